"""One flux whose mean is not exact, over less than a period: boxes that hold
every point hold its whole remainder, but are not valid, and the block search
finds the best of those that are, as the kernel that scores every box does."""
import numpy as np
import pytest

import paper_1112_1701_amd as bls
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flux", [0.1, 1.0 / 3.0, 1e-5, 1e9 / 7.0])
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("n,nbins,qmin,qmax", [(566, 11, 0.06, 0.47), (700, 157, 0.036, 0.185),
                                               (60, 300, 0.01, 0.45), (5000, 1000, 0.005, 0.3)])
def test_one_flux(monkeypatch, flux, weights, flags, n, nbins, qmin, qmax):
    rng = np.random.default_rng(n)
    t = np.sort(rng.uniform(0.0, 2.5, n))
    x = np.full(n, flux)
    w = rng.uniform(0.5, 2.0, n) if weights else None
    per = synth.log_period_grid(0.1, 20.0, 300)
    res = []
    for env in ("0", "1"):
        monkeypatch.setenv("BLS_BLOCK_SEARCH", env)
        with bls.Plan(max_points=n, max_periods=per.size, flags=flags) as p:
            res.append(bls.bls_search(p.handle, t, x, w, per, nbins, qmin, qmax))
    for k in res[0]:
        assert np.array_equal(res[0][k], res[1][k], equal_nan=True), k
