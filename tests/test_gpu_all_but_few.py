"""Dips that hold almost every point, beside a few far above them, on data that
cover part of the period.  W - R of such a box is a small difference of large
numbers; the block search finds it as the kernel that scores every box does."""
import numpy as np
import pytest

import paper_1112_1701_amd as bls
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 3000, 50000, 200000])
@pytest.mark.parametrize("few", [1, 2, 7])
@pytest.mark.parametrize("noise", [0.0, 1e-3])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("nbins,qmin,qmax", [(20, 0.2, 0.45), (40, 0.2, 0.45), (300, 0.2, 0.45),
                                             (1000, 0.25, 0.4)])
def test_all_but_few(monkeypatch, n, few, noise, weighted, nbins, qmin, qmax):
    rng = np.random.default_rng(n + few)
    t = np.concatenate([np.sort(rng.uniform(0.0, 2.0, n - few)), 2.4 + 0.01 * np.arange(few)])
    x = rng.normal(0.0, 1.0, n) * noise
    x[n - few:] += 5.0
    w = rng.uniform(0.5, 2.0, n) if weighted else None
    per = synth.log_period_grid(3.0, 12.0, 120)
    res = []
    for env in ("0", "1"):
        monkeypatch.setenv("BLS_BLOCK_SEARCH", env)
        with bls.Plan(max_points=n, max_periods=per.size, flags=1) as p:
            res.append(bls.bls_search(p.handle, t, x, w, per, nbins, qmin, qmax))
    for k in res[0]:
        assert np.array_equal(res[0][k], res[1][k], equal_nan=True), k
