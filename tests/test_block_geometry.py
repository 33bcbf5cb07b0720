"""The block search's geometry (no GPU): every box within the width range is
in exactly one tested pair of blocks, and every index stays in its array."""
import ctypes as C
import os

import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1112_1701_amd", "libbls_mi355x.so")


class Geom(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("bsize", "nblocks", "omin", "omax", "magic")]


@pytest.fixture(scope="module")
def geometry():
    import paper_1112_1701_amd._lib as L
    L.load()
    f = getattr(C.CDLL(LIB), "_ZN3bls14block_geometryEiiiPNS_9BlockGeomE")
    f.restype = C.c_bool
    return f


@pytest.mark.parametrize("nbins", [2, 3, 4, 5, 16, 63, 64, 65, 100, 128, 193, 300, 321, 350, 577,
                                   1000, 2000, 4095, 4096])
def test_every_box_in_a_tested_pair(geometry, nbins):
    widths = sorted({1, 2, 3, 7, nbins // 200, nbins // 100, nbins // 20, nbins // 10, nbins // 4,
                     nbins // 2 - 1, nbins // 2} & set(range(1, nbins // 2 + 1)))
    g = Geom()
    assert not geometry(nbins, 1, nbins // 2 + 1, C.byref(g))
    for kmin in widths:
        for kmax in [k for k in widths if k >= kmin]:
            if not geometry(nbins, kmin, kmax, C.byref(g)):
                continue
            s, nb = g.bsize, g.nblocks
            assert s % 2 == 1 and s <= 64 and nb <= 256 and (nb - 1) * s < nbins <= nb * s
            assert 0 <= g.omin <= g.omax <= 255 and g.omax + 1 < nb
            i = np.arange(128 * s + 64)
            assert np.array_equal((i * g.magic) >> 20, i // s)   # the drain's division
            j = np.arange(nbins)[:, None]
            k = np.unique(np.linspace(kmin, kmax, 40).astype(int))[None, :]
            e = j + k
            b = np.where(e < nbins, e // s, nb + (e - nbins) // s)
            o = b - j // s
            assert o.min() >= g.omin and o.max() <= g.omax
            first = np.where(b < nb, b * s, nbins + (b - nb) * s)
            last = np.where(b < nb, np.minimum(first + s - 1, nbins - 1), first + s - 1)
            assert np.all((first <= e) & (e <= last))
