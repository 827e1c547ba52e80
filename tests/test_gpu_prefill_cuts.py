"""Whole prefills at the lengths where the cut of the prefill GEMM changes: one
token group and several (even and uneven), one K range and several, row tiles
that end early, the smallest chunk (a prompt just above a small max_tree, and
the one-token rest of a 1025-token prompt), bf16 and int8 weights, on an empty
and on a cached prefix.  These small widths take few of the GEMM's
instantiations (128- and 256-row workgroups mostly); test_gpu_pf_gemm.py runs each.
Bars as in test_gpu_prefill.py, whose oracle comparison this reuses."""
import numpy as np
import pytest

import synth
from oracle import verify as ov
from tests.helpers import GpuCase, small_cfg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2412_18934_amd import dv  # noqa: E402
from tests.test_gpu_prefill import _check_next, _check_rows  # noqa: E402


def _case(dtype, d, heads, ffn, capacity, max_tree=64):
    cfg = small_cfg(n_layers=2, d_model=d, n_heads=heads, head_dim=d // heads, d_ffn=ffn, vocab=2048,
                    weight_dtype=dtype, init_std=0.09 * np.sqrt(256.0 / d))
    return GpuCase(cfg, seed=501, capacity=capacity, max_tree=max_tree)


def _check(case, n, p0, seed):
    kv = case.new_kv(fill=float("nan"))
    kv_o = case.synthetic_context(kv, seed, p0)
    prompt = synth.prompt(seed + 1, n, case.cfg.vocab)
    ref_kv, logits = ov.prefill(case.w.oracle(), prompt, kv=kv_o)
    nxt = dv.dv_prefill(case.h, prompt, kv.c)
    torch.cuda.synchronize()
    assert kv.len == p0 + n
    _check_rows(case, kv, ref_kv, p0, n)
    _check_next(nxt, logits[-1])
    first = [kv.layer_host(l, p0 + n) for l in range(case.cfg.n_layers)]
    kv.c.len = p0
    assert dv.dv_prefill(case.h, prompt, kv.c) == nxt
    for l, (k, v) in enumerate(first):
        k2, v2 = kv.layer_host(l, p0 + n)
        assert np.array_equal(k, k2) and np.array_equal(v, v2)


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("n,p0", [(65, 0), (97, 40), (130, 0), (200, 33), (500, 0), (1025, 7)])
def test_prefill_cuts(dtype, n, p0):
    case = _case(dtype, 1024, 8, 2816, 32 * -(-(n + p0) // 32))
    try:
        _check(case, n, p0, 5100 + n)
    finally:
        case.close()


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("n", [3, 17, 40])
def test_prefill_small_max_tree(dtype, n):
    case = _case(dtype, 320, 5, 832, 64, max_tree=2)   # 320: row tiles end early
    try:
        _check(case, n, 5, 5300 + n)
    finally:
        case.close()


@pytest.mark.parametrize("heads,n,p0", [(8, 70, 0), (8, 96, 5), (8, 65, 300), (4, 140, 1), (16, 130, 700)])
def test_prefill_attention_key_groups(heads, n, p0):
    """Few query blocks: two key groups per workgroup, with odd and even tile
    counts, a group without a tile for some waves, both head sizes."""
    case = _case("bf16", 512, heads, 1408, 32 * -(-(n + p0) // 32)) if heads != 16 else \
        _case("bf16", 1024, heads, 2816, 32 * -(-(n + p0) // 32))
    try:
        _check(case, n, p0, 5500 + n)
    finally:
        case.close()


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
def test_first_prefill_on_a_side_stream(dtype):
    """A handle bound to a non-blocking stream, whose first prefill cuts K: the
    same bytes as on the default stream."""
    case = _case(dtype, 1024, 8, 2816, 160)
    side = torch.cuda.Stream()
    h2 = dv.dv_verify_init(case.ccfg, case.dev.c, side.cuda_stream)
    try:
        prompt = synth.prompt(5700, 130, case.cfg.vocab)
        kv = [case.new_kv(fill=float("nan")) for _ in range(2)]
        torch.cuda.synchronize()
        nxt = dv.dv_prefill(h2, prompt, kv[0].c)
        assert dv.dv_prefill(case.h, prompt, kv[1].c) == nxt
        for l in range(case.cfg.n_layers):
            a, b = (x.layer_host(l, 130) for x in kv)
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    finally:
        dv.dv_verify_free(h2)
        case.close()
