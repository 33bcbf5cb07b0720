"""The unbinned search's screens by blocks of runs, at the sizes where their
layout changes: blocks that end early, quarters of the workgroup's prefix
sums, the three places of the per-point arrays, boxes of nearly a cycle,
equal phases and equal fluxes.  Against the FP64 oracle, with the tolerance
of the other unbinned tests."""
import numpy as np
import pytest

import oracle
import synth
from tests.test_gpu_unbinned import REL_TOL, _check, _gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,nper,qmin,qmax", [
    (3, 40, 0.01, 0.9), (7, 40, 0.01, 0.4), (8, 40, 0.01, 0.4), (9, 40, 0.2, 0.9),
    (17, 40, 0.05, 0.95), (111, 30, 0.01, 0.1), (113, 30, 0.01, 0.1), (512, 20, 0.3, 0.6),
    (1024, 20, 0.005, 0.05), (1025, 20, 0.005, 0.05), (2048, 6, 0.001, 0.95),
    (5000, 4, 0.001, 0.5), (32768, 2, 0.002, 0.01), (32769, 2, 0.002, 0.01),
])
def test_block_screens(bls, n, nper, qmin, qmax, weighted):
    lc = synth.small_curve(5000 + n, n, nperiods=nper, nbins=64, qmin=qmin, qmax=qmax,
                           weighted=weighted)
    t = lc.t.copy()
    t[n // 3:n // 2] = np.repeat(t[n // 3:n // 2:2], 2)[:n // 2 - n // 3]  # equal phases
    print("[case] unbinned blocks", n, nper, qmin, qmax, weighted, flush=True)
    with bls.Plan(max_curves=1, max_points=n, max_periods=nper) as p:
        g = _gpu(bls, p.handle, [(t, lc.x, lc.w)], [lc.periods], qmin, qmax)
    o = oracle.unbinned(t, lc.x, lc.w, lc.periods, qmin, qmax)
    _check((t, lc.x, lc.w), lc.periods, g[:4], o, "n%d" % n)
    top = o["sr"].max()
    assert g[4][0] == o["best_index"] or abs(g[0][g[4][0]] - top) <= REL_TOL * top


@pytest.mark.parametrize("n", [64, 300, 6000])
@pytest.mark.parametrize("flux", ["rounded", "outlier"])
def test_ties(bls, n, flux):
    rng = np.random.default_rng(n)
    t = np.sort(rng.uniform(0.0, 30.0, n))
    x = np.round(rng.normal(0.0, 1.0, n)) if flux == "rounded" else (np.arange(n) == n // 2) * 1.0
    per = synth.log_period_grid(0.3, 9.0, 12)
    print("[case] unbinned ties", n, flux, flush=True)
    with bls.Plan(max_curves=1, max_points=n, max_periods=12) as p:
        g = _gpu(bls, p.handle, [(t, x, None)], [per], 0.01, 0.1)
    _check((t, x, None), per, g[:4], oracle.unbinned(t, x, None, per, 0.01, 0.1), flux)
