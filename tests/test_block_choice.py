"""The choice between the two binned kernels (no GPU): unit-weight curves of far
fewer points than bins stay with the kernel that scores every box."""
import ctypes as C
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1112_1701_amd", "libbls_mi355x.so")


class Shape(C.Structure):
    _fields_ = [(k, C.c_int64) for k in ("n_off", "n", "p_off", "r_off")] + \
               [(k, C.c_int32) for k in ("nperiods", "nbins", "kmin", "kmax")]


@pytest.mark.parametrize("n,weighted,want", [(12, False, False), (80, False, False),
                                             (81, False, True), (5000, False, True),
                                             (12, True, True)])
def test_few_points(monkeypatch, n, weighted, want):
    import paper_1112_1701_amd._lib as L
    L.load()
    monkeypatch.delenv("BLS_BLOCK_SEARCH", raising=False)
    f = getattr(C.CDLL(LIB), "_ZN3bls11block_batchEPKNS_10CurveShapeEibibii")
    f.restype = C.c_bool
    s = Shape(0, n, 0, 0, 20000, 2585, 15, 260)
    assert f(C.byref(s), 1, C.c_bool(weighted), 1, C.c_bool(False), 256, 160 * 1024) == want
