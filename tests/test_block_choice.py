"""The choice between the two binned kernels (no GPU): curves of far fewer points
than bins, whose boxes tie, stay with the kernel that scores every box, weighted
ones only with a minimum count that hardly a box reaches.  The calls are ones
where the other choice took at least a quarter as long again."""
import ctypes as C
import math
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1112_1701_amd", "libbls_mi355x.so")


class Shape(C.Structure):
    _fields_ = [(k, C.c_int64) for k in ("n_off", "n", "p_off", "r_off")] + \
               [(k, C.c_int32) for k in ("nperiods", "nbins", "kmin", "kmax")]


@pytest.mark.parametrize("n,periods,nbins,qmin,qmax,weighted,mip,want", [
    (3, 29400, 407, 0.0503, 0.49, False, 1, False),
    (6, 18040, 1393, 0.0236, 0.16, False, 1, False),
    (10, 18040, 1393, 0.0236, 0.16, False, 1, False),
    (40, 18040, 1393, 0.0236, 0.16, False, 1, True),
    (1000, 18040, 1393, 0.0236, 0.16, False, 1, True),
    (12, 3640, 2585, 0.01, 0.03, False, 1, False),
    (18, 11558, 2242, 0.0552, 0.49, False, 1, False),
    (22, 2295, 2291, 0.0456, 0.441, False, 1, False),
    (12, 20000, 1740, 0.015, 0.098, True, 1, True),
    (6, 32208, 1740, 0.015, 0.036, True, 3, False),
    (30, 32208, 1740, 0.015, 0.036, True, 3, True),
    (3, 113680, 771, 0.0038, 0.0363, True, 3, False),
    (28, 237120, 1581, 0.0285, 0.0828, True, 3, True),
    (7, 3283, 2648, 0.0435, 0.3513, True, 3, True),
    (8, 5474, 3328, 0.011, 0.1251, True, 3, True)])
def test_few_points(monkeypatch, n, periods, nbins, qmin, qmax, weighted, mip, want):
    import paper_1112_1701_amd._lib as L
    L.load()
    monkeypatch.delenv("BLS_BLOCK_SEARCH", raising=False)
    f = getattr(C.CDLL(LIB), "_ZN3bls11block_batchEPKNS_10CurveShapeEibibii")
    f.restype = C.c_bool
    s = Shape(0, n, 0, 0, periods, nbins, math.ceil(qmin * nbins - 0.5), int(qmax * nbins + 0.5))
    assert f(C.byref(s), 1, C.c_bool(weighted), mip, C.c_bool(False), 256, 160 * 1024) == want
