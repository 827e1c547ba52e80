"""The prefill GEMM's cut (host code): every plan it can return is one that the
kernel is built for, and fits the split-K workspace."""
import pytest

from tests.pf_gemm import (MAX_TILES, MIN_TILES, PART_TILES, SHAPE_NWR, library_part_tiles, part_tiles, plan,
                           tiles_per_group, units)


@pytest.mark.parametrize("n_cu", [256, 64])
@pytest.mark.parametrize("d,ffn", [(64, 64), (128, 352), (320, 832), (1024, 2816), (4096, 11008), (5120, 13824),
                                   (8192, 28672)])
def test_plans_are_valid(d, ffn, n_cu):
    for q8 in (False, True):
        if q8 and ffn % 64:
            continue
        for mt in range(MIN_TILES, 65):
            for nb, k in ((3 * d // 16, d), (d // 16, d), (ffn // 8, d), (d // 16, ffn)):
                p = plan(nb, mt, k, q8, n_cu)
                assert 0 <= p.shape < (2 if q8 else 3)
                assert 4 <= p.tt <= 8 and p.tt == tiles_per_group(mt, p.n_tt)
                # every token group has tt tiles or one less
                sizes = {(g + 1) * mt // p.n_tt - g * mt // p.n_tt for g in range(p.n_tt)}
                assert sizes <= {p.tt, p.tt - 1}
                # every K group of every range has a step
                steps, nkg = k // (64 if q8 else 32), 8 // SHAPE_NWR[p.shape]
                assert p.ks == 1 or p.ks * nkg <= steps
                assert library_part_tiles(nb, p) == part_tiles(nb, p)
                if p.ks > 1:
                    assert part_tiles(nb, p) <= PART_TILES and units(nb, p) // p.ks <= MAX_TILES
