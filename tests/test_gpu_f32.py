"""fp32 weights against the oracle at the sizes where the fp32 projection and
attention kernels change: 2- and 4-block row groups, K splits and their
remainders (d_ffn a multiple of 16 only), one to four token tiles, key splits
of one tile per wave and longer ones, and weights that change under the
handle."""
import numpy as np
import pytest

import synth
from oracle import verify as ov
from paper_2412_18934_amd import dv
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


def test_f32_weights_are_read_in_place():
    """A caller may write new values into its fp32 matrices: the next step uses
    them, as a handle made from them does."""
    cfg = small_cfg(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=688, vocab=1024, init_std=0.09)
    case = GpuCase(cfg, seed=7300, capacity=128)
    fresh = None
    try:
        kv = case.new_kv()
        case.synthetic_context(kv, 7301, 77)
        toks, par = synth.random_tree(7302, 16, 6, cfg.vocab)
        before = case.step(kv, toks, par)[1]
        for lay in case.dev.layers:
            for k in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down"):
                lay[k].mul_(1.25).add_(0.01)
        case.dev.lm_head.neg_()
        torch.cuda.synchronize()
        after = case.step(kv, toks, par)[1]
        fresh = dv.dv_verify_init(case.ccfg, case.dev.c)
        want = torch.empty((16, cfg.vocab), dtype=torch.float32, device="cuda:0")
        dv.dv_verify_step(fresh, toks, par, kv.c, want.data_ptr())
        assert np.array_equal(after.view(np.uint32), want.cpu().numpy().view(np.uint32))
        assert np.abs(after - before).max() > 0.1
    finally:
        case.close()
        if fresh is not None:
            dv.dv_verify_free(fresh)


@pytest.mark.parametrize("d,ffn", [(64, 16), (96 * 2, 48), (448, 1008), (320, 272)])
def test_f32_odd_steps(d, ffn):
    """Single last steps (an odd count of 16-column steps in the row or in a K
    split), whose pair would reach past the row."""
    cfg = small_cfg(n_layers=1, d_model=d, n_heads=d // 64, head_dim=64, d_ffn=ffn, vocab=96,
                    init_std=0.09 * np.sqrt(256.0 / d))
    case = GpuCase(cfg, seed=7600, capacity=64)
    try:
        for m in (1, 9, 33):
            _check(case, cfg, 7700 + m, 20, m, 5 if m > 1 else 1)
    finally:
        case.close()


@pytest.mark.parametrize("d,m", [(1024, 8), (2048, 16), (2048, 33)])
def test_f32_sums_are_eight_chains(d, m):
    """Every projection sum is added up in 8 chains of K / 8 fp32 products (two
    per wave).  A rounding is off by 0.42 2^-24 of the value (rms); over a chain
    of n, whose partial sums grow with the square root of its length, by 0.3 2^-24
    sqrt(n) of the result, and as much over 8 such chains.  The bar, on the
    values of layer 0 against 64 bits, is 1.2 times that, with 2^-24 for the
    norm; half as many chains miss it."""
    cfg = small_cfg(n_layers=1, d_model=d, n_heads=d // 128, head_dim=128, d_ffn=64, vocab=96)
    case = GpuCase(cfg, seed=7800, capacity=64)
    try:
        kv = case.new_kv()
        toks, par = synth.random_tree(7801, m, 4, cfg.vocab)
        case.step(kv, toks, par)
        got = kv.layer_host(0, m)[1].astype(np.float64).transpose(1, 0, 2).reshape(m, d)
        lay = case.w.layers[0]
        x = case.w.embed[np.asarray(toks)].astype(np.float64)
        u = x / np.sqrt((x * x).mean(1, keepdims=True) + cfg.rms_eps) * lay["attn_norm"].astype(np.float64)
        want = u @ lay["wv"].astype(np.float64).T
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        bar = 1.2 * 2.0 ** -24 * np.sqrt(0.3 ** 2 * d / 8 + 1)
        print("[f32] K = %d, %d nodes: %.3g, bar %.3g" % (d, m, err, bar), flush=True)
        assert err <= bar
    finally:
        case.close()
