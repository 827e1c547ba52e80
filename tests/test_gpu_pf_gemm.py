"""Every instantiation of the prefill GEMM (epilogue, workgroup shape, token
tiles per unit, one K range and several, bf16 and int8 weights) against
64 bits, on small matrices with ragged rows, tokens and steps: row tiles that
end early, a token group one tile short, padding tokens, K groups and ranges
that share the steps unevenly.

Operands are exact in the kernel's formats (the reference takes hi + lo of the
split activations), so an output is off by the sums' rounding and, where it is
stored in 16 bits, by that rounding.  One rounding is off by 0.42 2^-24 of the
value on average (rms); over a chain, whose partial sums grow with the square
root of its length, by 0.3 2^-24 of the result and root of their number.  A
bf16 matrix instruction rounds 4 times (measured: 6.4e-7 in a chain of 320, which
is 0.6 2^-24 sqrt(320)).  int8 QKV sums each 64-column step by itself first: one
rounding a step, and 1.2 2^-24 for what is inside the steps.  The bars are 1.3 times
that, with 2 2^-24 for the epilogues.
"""
import numpy as np
import pytest

from tests import pf_gemm as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

EPS = 1e-6
NAMES = {P.EPI_QKV: "qkv", P.EPI_RESID: "resid", P.EPI_SWIGLU: "swiglu", P.EPI_LOGITS: "logits"}


def _gen(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float32)


class Problem:
    """One GEMM: operands, buffers, and its results in 64 bits."""

    def __init__(self, epi, q8, nb, k, d, hd, mt, m, seed):
        self.epi, self.q8, self.nb, self.k, self.d, self.hd, self.mt, self.m = epi, q8, nb, k, d, hd, mt, m
        rn = _gen(seed)
        mp, n = 16 * mt, 16 * nb
        w = rn(n, k)
        self.scale = None
        if q8:
            code = (w * 32).round().clamp(-127, 127)
            self.scale = rn(n).abs() * 1e-3 + 1e-3
            self.packed, w64 = P.pack_rows(code.to(torch.int8), True), code.double() * self.scale.double()[:, None]
        else:
            wb = (w / np.sqrt(k)).to(torch.bfloat16)
            self.packed, w64 = P.pack_rows(wb, False), wb.double()
        self.xs, x64 = P.split(rn(mp, k))
        self.sums = x64 @ w64.T                                  # [mp][n], packed row order
        self.nsq = 5
        self.ssq = rn(mp, self.nsq).square() * (d / self.nsq) + 0.1
        self.rinv = 1.0 / torch.sqrt(self.ssq.double().sum(1) / d + EPS)
        self.p0, self.cap = 37, 32 * -(-(37 + mp) // 32)
        self.cos, self.sin = rn(self.cap, hd // 2), rn(self.cap, hd // 2)
        self.x0, self.gain = rn(mp, d), rn(d).to(torch.bfloat16)

    def args(self, p):
        nan = float("nan")
        mp, d, heads = 16 * self.mt, self.d, self.d // self.hd
        full = lambda *s, dt=torch.float32: torch.full(s, nan, dtype=dt, device="cuda")  # noqa: E731
        b = self.buf = {
            "q": full(mp, d), "k": full(heads, self.cap, self.hd, dt=torch.bfloat16),
            "v": full(heads, self.cap // 32, self.hd, 32, dt=torch.bfloat16),
            "hs": full(self.nb * 8 // 32 * 32 + 32, 2 * mp, dt=torch.bfloat16), "x": self.x0.clone(),
            "us": full(d, 2 * mp, dt=torch.bfloat16), "ssq": full(mp, d // 64),
            "logits": full(self.m * 16 * self.nb + 4), "av": full(self.m, -(-self.nb // 4)),
            "ai": torch.full((self.m, -(-self.nb // 4)), -1, dtype=torch.int32, device="cuda"),
            "part": full(max(P.part_tiles(self.nb, p), 1) * 256),
            "cnt": torch.zeros(P.MAX_TILES, dtype=torch.int32, device="cuda")}
        a = P.PfArgs()
        a.packed, a.xs = self.packed.data_ptr(), self.xs.data_ptr()
        a.scale = self.scale.data_ptr() if self.q8 else None
        a.NB, a.K, a.MT, a.n_tt, a.ks = self.nb, self.k, self.mt, p.n_tt, p.ks
        a.part, a.cnt = b["part"].data_ptr(), b["cnt"].data_ptr()
        a.M, a.P0, a.ssq_in, a.nsq_in, a.eps, a.d = self.m, self.p0, self.ssq.data_ptr(), self.nsq, EPS, d
        a.q, a.kc, a.vc, a.cap, a.hd = b["q"].data_ptr(), b["k"].data_ptr(), b["v"].data_ptr(), self.cap, self.hd
        a.rope_cos, a.rope_sin, a.hs = self.cos.data_ptr(), self.sin.data_ptr(), b["hs"].data_ptr()
        a.logits, a.arg_val, a.arg_idx = b["logits"].data_ptr(), b["av"].data_ptr(), b["ai"].data_ptr()
        a.x, a.gain, a.us, a.ssq_out = b["x"].data_ptr(), self.gain.data_ptr(), b["us"].data_ptr(), b["ssq"].data_ptr()
        return a

    def bar(self, p):
        parts = p.ks * (8 // P.SHAPE_NWR[p.shape])
        if self.q8 and self.epi == P.EPI_QKV:
            var = 0.3 ** 2 * (self.k / 64) / parts + 1.2 ** 2
        else:
            var = 0.6 ** 2 * 2 * (self.k / 32) / parts
        return 1.3 * 2.0 ** -24 * np.sqrt(var + 2 ** 2)

    def check(self, p):
        m, bar, b = self.m, self.bar(p), self.buf
        assert int(b["cnt"].abs().sum()) == 0
        return getattr(self, "_" + NAMES[self.epi])(m, bar, b)

    def _qkv(self, m, bar, b):
        mat, row = P.block_rows(P.EPI_QKV, self.nb, self.d, self.hd)
        y = torch.empty(3, m, self.d, dtype=torch.float64, device="cuda")
        y[torch.from_numpy(mat.ravel()), :, torch.from_numpy(row.ravel())] = (self.sums[:m] * self.rinv[:m, None]).T
        y = y.view(3, m, -1, self.hd)
        pos = slice(self.p0, self.p0 + m)
        c, s = self.cos[pos].double()[:, None], self.sin[pos].double()[:, None]
        a, z = y[..., :self.hd // 2], y[..., self.hd // 2:]
        rot = torch.cat([a * c - z * s, z * c + a * s], -1)
        errs = [_rel(b["q"][:m].double(), rot[0].reshape(m, -1), bar)]
        assert torch.isnan(b["q"][m:]).all()
        k = b["k"].transpose(0, 1)
        v = b["v"].permute(1, 3, 0, 2).reshape(self.cap, -1, self.hd)
        for got, want in ((k, rot[1]), (v, y[2])):
            # rounded to bf16 from the fp32 value
    
            rms = float(want.square().mean().sqrt())
            assert ((got[pos] - want).abs() <= 2.0 ** -8 * want.abs() + 8 * bar * rms).all()
            assert torch.isnan(got[:self.p0]).all() and torch.isnan(got[self.p0 + m:]).all()
        return errs

    def _swiglu(self, m, bar, b):
        y = (self.sums * self.rinv[:, None]).view(16 * self.mt, -1, 2, 16)
        g, u = y[:, :, 0].reshape(16 * self.mt, -1), y[:, :, 1].reshape(16 * self.mt, -1)
        want = torch.nn.functional.silu(g) * u
        f = want.shape[1]
        got = P.unsplit(b["hs"].view(torch.int16).flatten()[:f * 32 * self.mt], 16 * self.mt, f)
        assert (got[m:] == 0).all()
        return [_rel(got[:m], want[:m], 3 * bar + 2.0 ** -17)]  # hi + lo: 16 bits

    def _resid(self, m, bar, b):
        want = self.x0.double()[:m] + self.sums[:m]
        errs = [_rel(b["x"][:m].double(), want, bar)]
        assert torch.equal(b["x"][m:], self.x0[m:])
        got = P.unsplit(b["us"].view(torch.int16).flatten(), 16 * self.mt, self.d)
        errs.append(_rel(got[:m], want * self.gain.double(), bar + 2.0 ** -17))
        errs.append(_rel(b["ssq"][:m].double(), want.view(m, -1, 64).square().sum(2), 2 * bar + 2.0 ** -20))
        assert (got[m:] == 0).all() and (b["ssq"][m:] == 0).all()
        return errs

    def _logits(self, m, bar, b):
        n = 16 * self.nb
        want = self.sums[:m] * self.rinv[:m, None]
        off = (b["logits_at"] - b["logits"].data_ptr()) // 4 if b["logits_at"] else None
        errs = []
        if off is not None:
            got = b["logits"][off:off + m * n].view(m, n)
            errs.append(_rel(got.double(), want, bar))
            assert torch.isnan(b["logits"][:off]).all() and torch.isnan(b["logits"][off + m * n:]).all()
            parts = got.view(m, -1, 64)
            assert torch.equal(b["av"], parts.amax(2))
            idx = parts.argmax(2) + 64 * torch.arange(parts.shape[1], device="cuda")
            assert torch.equal(b["ai"].long(), idx)
        else:
            assert torch.isnan(b["logits"]).all()
            errs.append(_rel(b["av"].double(), want.view(m, -1, 64).amax(2), bar))
        return errs


def _rel(got, want, bar):
    e = float((got - want).norm() / want.norm())
    assert e <= bar, "relative error %.3g > %.3g" % (e, bar)
    return e


def _plan(shape, tt, n_tt, ks):
    return P.PfPlan(shape, tt, n_tt, ks)


@pytest.mark.parametrize("q8", [False, True], ids=["bf16", "i8"])
@pytest.mark.parametrize("epi", [P.EPI_QKV, P.EPI_RESID, P.EPI_SWIGLU], ids=["qkv", "resid", "swiglu"])
@pytest.mark.parametrize("shape", [0, 1, 2])
def test_every_instantiation(epi, q8, shape):
    if q8 and shape == 2:
        pytest.skip("not built")
    for tt in (4, 5, 6, 7, 8):
        for n_tt, ks in ((1, 1), (3, 1), (2, 3), (1, 2)):
            # the last group of several is one tile short (4 tiles are never less)
            mt = n_tt * tt - (1 if n_tt > 1 and tt > 4 else 0)
            if n_tt == 1 and ks == 1 and tt == 4:
                mt = 3                          # the smallest chunk: 3 tiles in a group of 4
            d, hd = (320, 64) if tt % 2 else (384, 128)
            k = {P.EPI_RESID: 1216 if q8 else 1120, P.EPI_QKV: d, P.EPI_SWIGLU: d}[epi]
            if epi != P.EPI_RESID and ks * (8 // P.SHAPE_NWR[shape]) > k // (64 if q8 else 32):
                ks = 1
            nb = {P.EPI_QKV: 3 * d // 16, P.EPI_RESID: d // 16, P.EPI_SWIGLU: 44}[epi]
            pr = Problem(epi, q8, nb, k, d, hd, mt, 16 * mt - 5, 1000 + 100 * shape + 10 * tt + n_tt)
            p = _plan(shape, tt, n_tt, ks)
            print("[pf] %s %s shape %d tt %d n_tt %d ks %d" % (NAMES[epi], "i8" if q8 else "bf16", shape, tt, n_tt, ks),
                  end="", flush=True)
            P.launch(pr.args(p), p, epi)
            torch.cuda.synchronize()
            print("  " + " ".join("%.2e" % e for e in pr.check(p)), "bar %.2e" % pr.bar(p), flush=True)


@pytest.mark.parametrize("q8", [False, True], ids=["bf16", "i8"])
@pytest.mark.parametrize("shape,tt,ks", [(0, 8, 1), (0, 8, 4), (1, 8, 1), (1, 7, 2), (2, 6, 1)])
def test_sums_over_a_whole_model_width(q8, shape, tt, ks):
    """K = 5120 (160 k-steps): the rounding of long chains, on the queries,
    which are stored in fp32."""
    if q8 and shape == 2:
        pytest.skip("not built")
    pr = Problem(P.EPI_QKV, q8, 960, 5120, 5120, 128, tt, 16 * tt, 2000 + tt)
    p = _plan(shape, tt, 1, ks)
    P.launch(pr.args(p), p, P.EPI_QKV)
    torch.cuda.synchronize()
    print("[pf] K = 5120 %s shape %d tt %d ks %d: " % ("i8" if q8 else "bf16", shape, tt, ks), pr.check(p),
          "bar %.2e" % pr.bar(p), flush=True)


@pytest.mark.parametrize("mt,m", [(3, 33), (3, 48), (4, 49), (4, 64)])
@pytest.mark.parametrize("out", ["aligned", "unaligned", "none"])
def test_logits(mt, m, out):
    """The wide trees' lm_head: vector and scalar stores, and no logits at all."""
    pr = Problem(P.EPI_LOGITS, False, 36, 320, 320, 64, mt, m, 3000 + m)
    p = _plan(2, 4, 1, 1)
    a = pr.args(p)
    a.logits = {"aligned": pr.buf["logits"].data_ptr(), "unaligned": pr.buf["logits"].data_ptr() + 4, "none": None}[out]
    pr.buf["logits_at"] = a.logits
    P.launch(a, p, P.EPI_LOGITS)
    torch.cuda.synchronize()
    pr.check(p)
