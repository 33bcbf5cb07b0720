"""The choice between the two binned kernels (no GPU): curves of far fewer points
than bins stay with the kernel that scores every box, but for weighted ones
without a minimum count."""
import ctypes as C
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1112_1701_amd", "libbls_mi355x.so")


class Shape(C.Structure):
    _fields_ = [(k, C.c_int64) for k in ("n_off", "n", "p_off", "r_off")] + \
               [(k, C.c_int32) for k in ("nperiods", "nbins", "kmin", "kmax")]


@pytest.mark.parametrize("n,weighted,mip,want", [
    (12, False, 1, False), (54, False, 1, False), (55, False, 1, True), (5000, False, 1, True),
    (12, True, 1, True), (12, True, 3, False), (55, True, 3, True)])
def test_few_points(monkeypatch, n, weighted, mip, want):
    import paper_1112_1701_amd._lib as L
    L.load()
    monkeypatch.delenv("BLS_BLOCK_SEARCH", raising=False)
    f = getattr(C.CDLL(LIB), "_ZN3bls11block_batchEPKNS_10CurveShapeEibibii")
    f.restype = C.c_bool
    kmax = 62 if weighted and mip > 1 else 170
    s = Shape(0, n, 0, 0, 20000, 1740, 26, kmax)
    assert f(C.byref(s), 1, C.c_bool(weighted), mip, C.c_bool(False), 256, 160 * 1024) == want


@pytest.mark.parametrize("n,want", [(3, False), (6, False), (10, False), (20, True), (40, True),
                                    (1000, True)])
def test_fewer_points_tie_more(monkeypatch, n, want):
    import paper_1112_1701_amd._lib as L
    L.load()
    monkeypatch.delenv("BLS_BLOCK_SEARCH", raising=False)
    f = getattr(C.CDLL(LIB), "_ZN3bls11block_batchEPKNS_10CurveShapeEibibii")
    f.restype = C.c_bool
    s = Shape(0, n, 0, 0, 4 * 4510, 1393, 33, 223)
    assert f(C.byref(s), 1, C.c_bool(False), 1, C.c_bool(False), 256, 160 * 1024) == want
