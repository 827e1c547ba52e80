"""Compile libdv.so (HIP kernels + C ABI) for gfx950 with hipcc."""
import os
import shutil
import subprocess
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libdv.so")
SOURCES = ["dv_kernels.hip", "dv_prefill.hip", "dv_engine.cpp"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU ops stay off in every HIP build of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Always recompiles (the sources in parallel); writes libdv.so atomically
    next to this file."""
    with tempfile.TemporaryDirectory() as tmp:
        base = [hipcc()] + HIPCC_FLAGS + ["-I", INCLUDE, "-I", CSRC]
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        jobs = [subprocess.Popen(base + ["-c", os.path.join(CSRC, s), "-o", o], stdout=subprocess.PIPE,
                                 stderr=subprocess.STDOUT, text=True) for s, o in zip(SOURCES, objs)]
        logs = [j.communicate()[0] for j in jobs]
        if any(j.returncode for j in jobs):
            raise RuntimeError("hipcc failed:\n" + "".join(logs))
        out = LIB + ".tmp%d" % os.getpid()
        res = subprocess.run([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", out],
                             capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print("".join(logs) + res.stderr)
    os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
