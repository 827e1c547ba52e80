"""The host engine (dv_engine.cpp) compiled for the CPU against a logging
stand-in for the HIP runtime and the kernel launchers (hipstub.cpp): the order of
clears, launches and waits, and what happens when memory runs out."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2412_18934_amd import dv

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2412_18934_amd", "csrc")
STREAM = 0x1230


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("engine") / "libengine.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "dv_engine.cpp"), os.path.join(HERE, "hipstub.cpp"), "-o", out], check=True)
    L = ctypes.CDLL(out)
    L.stub_log.restype = ctypes.c_char_p
    L.stub_reset.argtypes = [ctypes.c_size_t]
    L.stub_live.restype = ctypes.c_size_t
    L.dv_last_error.restype = ctypes.c_char_p
    L.dv_last_error.argtypes = [ctypes.c_void_p]
    return L


class Engine:
    def __init__(self, lib, dtype, n_layers=2, d=256, ffn=704, vocab=1024, max_ctx=4096, max_tree=8, stream=STREAM):
        self.lib = lib
        hd = 128 if d >= 1024 else 64
        cfg = dv.dv_config(n_layers=n_layers, d_model=d, n_heads=d // hd, head_dim=hd, d_ffn=ffn, vocab=vocab,
                           rms_eps=1e-6, rope_base=10000.0, weight_dtype=dtype, max_ctx=max_ctx, max_tree=max_tree)
        tab = ctypes.cast((ctypes.c_void_p * n_layers)(*([0x1000] * n_layers)), ctypes.POINTER(ctypes.c_void_p))
        w = dv.dv_weights(0x1000, 0x1000, 0x1000, *[tab] * 9, 0x1000, *[tab] * 7)
        self.h = ctypes.c_void_p()
        lib.stub_reset(2 ** 64 - 1)
        assert lib.dv_verify_init(ctypes.byref(cfg), ctypes.byref(w), ctypes.c_void_p(stream), ctypes.byref(self.h)) == 0
        self.init_log = self.log()
        self.kv = dv.dv_kv(0x1000, 0x1000, max_ctx, 0)

    def log(self):
        rows = [r.split() for r in self.lib.stub_log().decode().splitlines()]
        return [(what, int(stream, 16), int(n)) for what, stream, n in rows]

    def prefill(self, n, fail_at=2 ** 64 - 1):
        self.lib.stub_reset(fail_at)
        toks = np.zeros(n, np.int32)
        nxt = ctypes.c_int32()
        return self.lib.dv_prefill(self.h, toks.ctypes.data_as(ctypes.c_void_p), n, ctypes.byref(self.kv),
                                   ctypes.byref(nxt))

    def close(self):
        self.lib.dv_verify_free(self.h)


@pytest.fixture(params=[dv.DV_BF16, dv.DV_I8], ids=["bf16", "i8"])
def engine(request, lib):
    e = Engine(lib, request.param)
    yield e
    e.close()
    assert lib.stub_live() == 0


def test_clears_are_ordered_before_the_launches(engine):
    """A memset on the null stream is not ordered before launches on a
    non-blocking stream: either it goes on the handle's stream, or the device is
    synchronised in between."""
    assert engine.prefill(300) == 0
    pending = False
    for what, stream, _ in engine.log():
        if what == "memset" and stream != STREAM:
            pending = True
        elif what == "devsync":
            pending = False
        elif what in ("pf_embed", "pf_gemm", "causal", "gemm", "norm", "attention", "accept"):
            assert stream == STREAM
            assert not pending, what
    assert [w for w, _, _ in engine.log()].count("pf_gemm") == 4 * 2


def test_prefill_without_room_for_its_workspace(engine):
    """The prompt runs as chains then, and the failed allocation leaves nothing
    behind: no error for the next launch, and the workspace is made later."""
    live = engine.lib.stub_live()
    assert engine.prefill(300, fail_at=1 << 16) == 0
    names = [w for w, _, _ in engine.log()]
    assert engine.kv.len == 300 and "pf_gemm" not in names and names.count("accept") == 1
    assert names.count("attention") == 2 * -(-300 // 8)
    assert engine.lib.stub_live() == live
    engine.kv.len = 0
    assert engine.prefill(300) == 0
    assert [w for w, _, _ in engine.log()].count("pf_gemm") == 4 * 2
    # a longer prompt that needs more than there is keeps what it has
    live = engine.lib.stub_live()
    engine.kv.len = 0
    assert engine.prefill(1000, fail_at=1 << 16) == 0 and engine.kv.len == 1000
    assert engine.lib.stub_live() == live
    engine.kv.len = 0
    assert engine.prefill(300, fail_at=1 << 16) == 0
    assert [w for w, _, _ in engine.log()].count("pf_gemm") == 4 * 2


@pytest.mark.parametrize("d,ffn,max_tree,n,kept,chains", [
    (1536, 4224, 8, 10, 7909, True),      # a few tokens behind a long context
    (1024, 2816, 64, 65, 4000, True), (1024, 2816, 4, 5, 0, True),
    (1024, 2816, 64, 128, 0, False), (5120, 13824, 64, 65, 0, False), (5120, 13824, 64, 100, 2000, False),
    (1024, 2816, 8, 33, 4000, False),     # more than four chains
])
def test_int8_prompts_of_few_chains_take_the_faster_route(lib, d, ffn, max_tree, n, kept, chains):
    """Measured on both routes, us per layer, chains and causal: 115 / 272, 157 /
    217, 82 / 89, 171 / 113, 267 / 210, 363 / 301.  bf16 prompts take the causal
    pass as they always did."""
    for dtype in (dv.DV_I8, dv.DV_BF16):
        e = Engine(lib, dtype, n_layers=1, d=d, ffn=ffn, vocab=32, max_ctx=8192, max_tree=max_tree)
        e.kv.len = kept
        assert e.prefill(n) == 0 and e.kv.len == kept + n
        names = [w for w, _, _ in e.log()]
        took_chains = "pf_gemm" not in names
        assert took_chains == (chains and dtype == dv.DV_I8)
        e.close()


def test_workspaces_are_what_the_calls_use(lib):
    """The split-K partials are sized by the model's plans, and the rows of the
    one-workgroup sampling walk exist only for vocabularies that take it."""
    e = Engine(lib, dv.DV_BF16)
    try:
        small = lib.stub_live()
        assert e.prefill(1000) == 0
        # 63 tiles in 8 groups, d_model / 16 = 16 blocks and 3 or 5.5 times that, 2 ranges
        rows = 1024 * (4 * 256 * 4 + 704 * 4 + 4 * 5 + 4)
        part = 1024 * 96 * 8 * 2 * 8
        assert rows <= lib.stub_live() - small <= rows + part + (1 << 16)
    finally:
        e.close()
    allocations = []
    for vocab in (65536, 65568):
        e = Engine(lib, dv.DV_BF16, n_layers=1, vocab=vocab)
        allocations.append(sum(w == "malloc" for w, _, _ in e.init_log))
        e.close()
    assert allocations[1] == allocations[0] + 1


def test_fp32_weights_are_not_copied(lib):
    d, ffn, vocab, layers = 1024, 2816, 8192, 4
    e = Engine(lib, dv.DV_F32, n_layers=layers, d=d, ffn=ffn, vocab=vocab, max_ctx=64)
    try:
        assert not [r for r in e.init_log if r[0] == "pack"]
        assert lib.stub_live() < 4 * layers * (4 * d * d + 3 * d * ffn) / 4
    finally:
        e.close()
