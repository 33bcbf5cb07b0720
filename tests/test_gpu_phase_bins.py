"""The device's phase bins on a plan that takes far more points than trial
periods: the bins have a place per point."""
import numpy as np
import pytest

import oracle
import paper_1112_1701_amd as bls

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,max_periods", [(200, 1), (5000, 4), (20000, 33)])
def test_more_points_than_periods(n, max_periods):
    rng = np.random.default_rng(n)
    t = np.sort(rng.uniform(0.0, 40.0, n))
    x = rng.normal(1.0, 0.01, n)
    with bls.Plan(max_curves=1, max_points=n, max_periods=max_periods) as p:
        for period in (0.37, 5.1):
            for nbins in (100, 1000):
                g = bls.bls_debug_phase_bins(p.handle, t, period, nbins)
                o, *_ = oracle.bins(t, np.ones_like(t), None, period, nbins)
                assert np.array_equal(g, o), (n, period, nbins)
        per = np.linspace(0.5, 5.0, max_periods)
        r = bls.bls_search(p.handle, t, x, None, per, 100, 0.01, 0.1)
    with bls.Plan(max_curves=1, max_points=n, max_periods=max_periods) as p:
        s = bls.bls_search(p.handle, t, x, None, per, 100, 0.01, 0.1)
    for k in s:
        assert np.array_equal(r[k], s[k], equal_nan=True), k
