"""The fold of a curve's points past its last whole chunk of 1024: merged or not,
the same bits, and on a dense cadence (runs of points in one bin) no slower than
a whole chunk."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


@pytest.mark.parametrize("n", [3, 5, 255, 257, 1000, 1023, 1024, 1025, 1290, 2047])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("block", ["0", "1"])
def test_merged_or_not(bls, monkeypatch, n, weighted, block):
    print("[case] rest", n, weighted, block, flush=True)
    rng = np.random.default_rng(n)
    t = np.arange(n) * 2.0 / 1440.0
    x, w = rng.normal(0.0, 1.0, n), rng.uniform(0.5, 2.0, n) if weighted else None
    if weighted:
        w[rng.random(n) < 0.1] = 0.0
        w[:2] = 1.0
    monkeypatch.setenv("BLS_BLOCK_SEARCH", block)
    got = []
    for merge in (None, "1", "0"):
        monkeypatch.setenv("BLS_FOLD_MERGE", merge) if merge else None
        with bls.Plan(max_points=1 << 12, max_periods=1 << 10) as p:
            got.append(bls.bls_search(p.handle, t, x, w, synth.log_period_grid(0.05, 20.0, 300), 90,
                                      0.02, 0.2))
    for g in got[1:]:
        for key in got[0]:
            assert np.array_equal(g[key], got[0][key], equal_nan=True), key


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("nbins", [24, 60])
def test_dense_cadence(bls, nbins, weighted):
    print("[case] dense rest", nbins, weighted, flush=True)
    nc, m, ms = 100, 4000, []
    for n in (1024, 1000):
        rng = np.random.default_rng(1)
        t = np.tile(np.arange(n) * 2.0 / 1440.0, nc)
        x, w = rng.normal(0.0, 1.0, nc * n), rng.uniform(0.5, 2.0, nc * n) if weighted else None
        with bls.Plan(max_curves=nc, max_points=nc * n, max_periods=nc * m) as p:
            for _ in range(5):
                bls.bls_search_batch(p.handle, np.arange(nc + 1) * n, t, x, w,
                                     synth.log_period_grid(0.5, 20.0, m), None, nbins, 0.05, 0.2)
            ms.append(min(bls.bls_kernel_times(p.handle)))
    print("[ms] 1024 points, 1000:", ms, flush=True)
    assert ms[1] <= 1.4 * ms[0], ms
