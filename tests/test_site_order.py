"""The hop kernels' traversal order (host code, eofa::site_order): every site once;
the slabs of t dealt out to eight runs where eight windows of three slabs (or the
whole field) exceed the MALL (1.5 M 5D sites of a parity; 2 M in FP16S), and one run
through the lattice elsewhere, long thin lattices among them.
"""
import ctypes

import numpy as np
import pytest

from paper_1706_05843_amd import eofa


class Geometry(ctypes.Structure):
    _fields_ = [("L", ctypes.c_int * 4), ("Ls", ctypes.c_int), ("V", ctypes.c_int), ("Vh", ctypes.c_int)]


def order(dims, Ls, prec):
    f = getattr(eofa.lib(), "_ZN4eofa10site_orderERKNS_8GeometryEiPi")
    f.restype = None
    v = int(np.prod(dims))
    out = np.full(v // 2, -1, dtype=np.int32)
    f(ctypes.byref(Geometry((ctypes.c_int * 4)(*dims), Ls, v, v // 2)), prec, out.ctypes.data_as(ctypes.c_void_p))
    return out


@pytest.mark.parametrize("dims,Ls,dealt,dealt16", [
    ((24, 24, 24, 64), 12, True, True),      # slabs of 0.33 M 5D sites, 5.3 M in all
    ((16, 16, 16, 64), 16, True, True),      # 0.13 M, 2.1 M
    ((18, 14, 22, 26), 24, True, False),     # 0.13 M, 1.7 M
    ((16, 16, 16, 32), 16, False, False),    # 1.05 M in all
    ((8, 8, 8, 256), 32, False, False),      # 0.03 M, 2.1 M: windows of 0.8 M
    ((12, 12, 12, 128), 16, False, False),   # 0.055 M, 1.8 M: 1.3 M
    ((4, 4, 6, 10), 4, False, False),
])
@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32, eofa.FP16S])
def test_order(dims, Ls, dealt, dealt16, prec):
    o = order(dims, Ls, prec)
    assert np.array_equal(np.sort(o), np.arange(len(o)))
    t = o // (dims[0] // 2 * dims[1] * dims[2])
    eighth = t[:len(o) // 8]
    if dealt16 if prec == eofa.FP16S else dealt:
        assert np.array_equal(np.unique(eighth), np.arange(dims[3]))
    else:
        bt = 4 if dims[3] % 4 == 0 else 2
        assert np.all(np.diff(t // bt) >= 0)
