"""The prefill GEMM's launcher by itself: its C++ symbols in libdv.so, the
argument struct read from the header that declares it, and the operand layouts
in torch (dv_internal.h)."""
import ctypes
import os
import re

import numpy as np

from paper_2412_18934_amd import dv

CSRC = os.path.join(os.path.dirname(os.path.abspath(dv.__file__)), "csrc")
EPI_QKV, EPI_RESID, EPI_SWIGLU, EPI_LOGITS = 0, 1, 2, 3
SHAPE_NWR = (8, 4, 2)   # row waves of 4 blocks each
PART_TILES, MAX_TILES, MIN_TILES = 65536, 1024, 3


def _struct(name):
    """The ctypes twin of a struct of pointers, ints and floats in dv_internal.h."""
    src = open(os.path.join(CSRC, "dv_internal.h")).read()
    body = re.search(r"struct %s \{(.*?)\n\};" % name, src, flags=re.S).group(1)
    body = re.sub(r"//.*", "", body)
    fields = []
    for decl in filter(None, (" ".join(d.split()) for d in body.split(";"))):
        base, rest = re.match(r"(?:const )?(\w+) (.*)", decl).groups()
        for var in rest.split(","):
            var = var.strip()
            if var.startswith("*"):
                fields.append((var[1:], ctypes.c_void_p))
            else:
                fields.append((var, {"int": ctypes.c_int, "float": ctypes.c_float}[base]))
    return type(name, (ctypes.Structure,), {"_fields_": fields})


PfArgs, PfPlan = _struct("PfArgs"), _struct("PfPlan")


def plan(nb, mt, k, q8, n_cu=256):
    f = dv.lib()._Z7pf_planiiibi
    f.restype, f.argtypes = PfPlan, [ctypes.c_int] * 3 + [ctypes.c_bool, ctypes.c_int]
    return f(nb, mt, k, q8, n_cu)


def tiles_per_group(mt, n_tt):
    return max(-(-mt // n_tt), 4)


def units(nb, p):
    return -(-nb // (4 * SHAPE_NWR[p.shape])) * p.n_tt * p.ks


def part_tiles(nb, p):
    return units(nb, p) * SHAPE_NWR[p.shape] * 4 * p.tt if p.ks > 1 else 0


def library_part_tiles(nb, p):
    f = dv.lib()._Z13pf_part_tilesiRK6PfPlan
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.POINTER(PfPlan)]
    return f(nb, ctypes.byref(p))


def launch(args, p, epi):
    f = dv.lib()._Z14launch_pf_gemmRK6PfArgsRK6PfPlaniP12ihipStream_t
    f.restype, f.argtypes = ctypes.c_int, [ctypes.POINTER(PfArgs), ctypes.POINTER(PfPlan), ctypes.c_int,
                                           ctypes.c_void_p]
    assert p.tt == tiles_per_group(args.MT, p.n_tt) and 0 < args.M <= 16 * args.MT
    rc = f(ctypes.byref(args), ctypes.byref(p), epi, None)
    assert rc == 0, "launch_pf_gemm: HIP error %d" % rc


def block_rows(epi, nb, d, hd):
    """Physical (matrix, row) of every packed row [nb][16]: QKV pairs dims j and
    j + hd/2 of a head, SWIGLU gate and up rows, else rows in order."""
    mat, row = np.zeros((nb, 16), np.int64), np.zeros((nb, 16), np.int64)
    r = np.arange(16)
    for gb in range(nb):
        t, half = divmod(gb, 2)
        if epi == EPI_QKV:
            seg, tt = divmod(t, d // 32)
            h, j = divmod(tt, hd // 32)
            mat[gb], row[gb] = seg, h * hd + 16 * j + half * (hd // 2) + r
        elif epi == EPI_SWIGLU:
            mat[gb], row[gb] = half, 16 * t + r
        else:
            row[gb] = 16 * gb + r
    return mat, row


def pack_rows(w, q8):
    """w [16 nb][K] in packed row order -> block order."""
    n, k = w.shape
    b = w.reshape(n // 16, 16, k // 64, 2, 4, 8) if q8 else w.reshape(n // 16, 16, k // 32, 4, 8)
    # int8: [pair][block][lane = 16 g + r][k-step half][8]; bf16: [k-step][block][lane][8]
    return b.permute(2, 0, 4, 1, 3, 5).contiguous() if q8 else b.permute(2, 0, 3, 1, 4).contiguous()


def split(x):
    """fp32 [16 MT][K] -> split layout, bf16 bits as int16 (hi truncated, lo
    rounded), and the value hi + lo in 64 bits."""
    import torch
    m, k = x.shape
    hi = (x.view(torch.int32) & -65536).view(torch.float32)
    lo = (x - hi).to(torch.bfloat16)
    both = torch.stack([hi.to(torch.bfloat16), lo])
    v = both.view(2, m // 16, 16, k // 32, 4, 8).permute(3, 1, 0, 4, 2, 5).contiguous()
    return v.view(torch.int16), hi.double() + lo.double()


def unsplit(s, m, k):
    """The 64-bit values of a split-layout buffer (int16 bits)."""
    import torch
    v = s.view(torch.bfloat16).view(k // 32, m // 16, 2, 4, 16, 8).permute(2, 1, 4, 0, 3, 5).reshape(2, m, k)
    return v[0].double() + v[1].double()
