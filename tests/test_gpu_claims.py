"""Work items on both sides of the grid's size: every period of a single
curve is searched, once, whether its item is a workgroup's first, one of a
larger claim, or one of the last ones."""
import numpy as np
import pytest

import oracle
import synth
from tests.parity import check_curve
from tests.test_gpu_unbinned import _check, _gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


@pytest.mark.parametrize("m", [1, 2, 2048, 2049, 9000, 70000])
@pytest.mark.parametrize("kernel", ["0", "1"])
def test_binned_items(bls, monkeypatch, m, kernel):
    monkeypatch.setenv("BLS_TILE_CAP", "1")  # an item per period
    monkeypatch.setenv("BLS_BLOCK_SEARCH", kernel)
    lc = synth.small_curve(31, 40, nperiods=m, nbins=12, qmin=0.1, qmax=0.3)
    print("[case] claims", m, kernel, flush=True)
    with bls.Plan(max_curves=1, max_points=64, max_periods=m) as p:
        g = bls.bls_search(p.handle, lc.t, lc.x, None, lc.periods, 12, 0.1, 0.3)
    o = oracle.search(lc.t, lc.x, None, lc.periods, 12, 0.1, 0.3)
    check_curve(lc, g, o, label="claims %d" % m)


@pytest.mark.parametrize("m", [1, 1025, 40000])
def test_unbinned_items(bls, m):
    lc = synth.small_curve(32, 30, nperiods=m, nbins=12, qmin=0.05, qmax=0.3)
    print("[case] unbinned claims", m, flush=True)
    with bls.Plan(max_curves=1, max_points=64, max_periods=m) as p:
        g = _gpu(bls, p.handle, [(lc.t, lc.x, None)], [lc.periods], 0.05, 0.3)
    _check((lc.t, lc.x, None), lc.periods, g[:4],
           oracle.unbinned(lc.t, lc.x, None, lc.periods, 0.05, 0.3), "m%d" % m)
