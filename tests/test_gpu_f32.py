"""fp32 weights against the oracle at the sizes where the fp32 projection and
attention kernels change: 2- and 4-block row groups, K splits and their
remainders (d_ffn a multiple of 16 only), one to four token tiles, key splits
of one tile per wave and longer ones, and weights read from the caller's rows
when no packed copy is kept."""
import numpy as np
import pytest

import synth
from oracle import verify as ov
from tests.helpers import GpuCase, compare_step, small_cfg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

TOL = 1e-4   # the fp32 bar of the other parity tests


def _check(case, cfg, seed, p, m, depth):
    kv = case.new_kv(fill=float("nan"))
    kv_o = case.synthetic_context(kv, seed + 1, p)
    toks, par = synth.random_tree(seed + 2, m, depth, cfg.vocab)
    ref = ov.verify_step(case.w.oracle(), kv_o, toks, par)
    ref["tokens"], ref["parents"] = np.asarray(toks), np.asarray(par)
    acc, lg = case.step(kv, toks, par)
    compare_step(acc, lg, ref, TOL)
    acc2, lg2 = case.step(kv, toks, par)
    assert np.array_equal(lg.view(np.uint32), lg2.view(np.uint32))


@pytest.mark.parametrize("d,heads,ffn,p,m", [
    (64, 1, 80, 5, 3),            # waves without a step
    (1024, 8, 2832, 300, 1),      # 4-block groups, 177 FFN steps over the splits
    (1024, 16, 2816, 3000, 16),   # long key splits, two tiles in flight
    (1024, 8, 2816, 0, 17),
    (1088, 17, 2912, 90, 48),     # 34 row tiles: 2-block groups
    (2048, 16, 5504, 700, 64),    # the largest tree
])
def test_f32_step(d, heads, ffn, p, m):
    cfg = small_cfg(n_layers=1, d_model=d, n_heads=heads, head_dim=d // heads, d_ffn=ffn, vocab=2080,
                    init_std=0.09 * np.sqrt(256.0 / d))
    case = GpuCase(cfg, seed=7100, capacity=max(64, 32 * -(-(p + m) // 32)))
    try:
        _check(case, cfg, 7200, p, m, 6 if m > 1 else 1)
    finally:
        case.close()


def test_f32_without_packed_copy():
    """With less than twice the copy's bytes free, the kernels read the
    caller's rows; the sums are the same, so the results are too."""
    cfg = small_cfg(n_layers=1, d_model=1024, n_heads=8, head_dim=128, d_ffn=2816, vocab=32000,
                    init_std=0.045)
    packed = GpuCase(cfg, seed=7300, capacity=128)
    rows = fill = None
    try:
        torch.cuda.empty_cache()
        copy = 4 * (4 * 1024 * 1024 + 3 * 1024 * 2816 + 32000 * 1024)
        weights = packed.dev.nbytes()
        room = int(1.6 * copy) + weights
        fill = torch.empty(max(torch.cuda.mem_get_info()[0] - room, 0), dtype=torch.uint8, device="cuda:0")
        rows = GpuCase(cfg, seed=7300, capacity=128, weights=packed.w)
        assert torch.cuda.mem_get_info()[0] > copy   # the copy would have fitted
        out = []
        for case in (packed, rows):
            _check(case, cfg, 7400, 77, 16, 6)
            kv = case.new_kv()
            case.synthetic_context(kv, 7401, 77)
            toks, par = synth.random_tree(7402, 16, 6, cfg.vocab)
            out.append(case.step(kv, toks, par)[1])
        assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))
    finally:
        packed.close()
        if rows is not None:
            rows.close()
        del fill
        torch.cuda.empty_cache()
