"""Curves without a signal (one flux throughout, a filled or saturated star):
no box or run of them has a value, and the searches' screens see that.  Their
kernels take no longer than on noise, within a factor that no screen passing
everything stays below."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


def _flux(kind, rng, n):
    """(flux, weights): noise, one flux (its mean exact or not), with weights."""
    x = rng.normal(0.0, 1.0, n) if kind[0] == "noise" else np.full(n, kind[0])
    return x, 10.0 ** rng.uniform(-1.0, 1.0, n) if kind[1] else None


# (a flux whose mean is not exact leaves a remainder of one sign: no dips)
@pytest.mark.parametrize("kind,flags", [((1.0, False), 0), ((1.0, True), 0), ((0.1, False), 1),
                                        ((0.1, True), 1)])
@pytest.mark.parametrize("n,m", [(1000, 2000), (5000, 400), (40000, 32)])
def test_unbinned(bls, kind, flags, n, m):
    import torch
    dev = lambda a: None if a is None else torch.tensor(a, device="cuda:0")
    print("[case] flat unbinned", kind, flags, n, m, flush=True)
    rng = np.random.default_rng(n)
    t = dev(np.sort(rng.uniform(0.0, 60.0, n)))
    per = dev(synth.log_period_grid(0.3, 9.0, m))
    out = [torch.empty(m, device="cuda:0", dtype=d) for d in (
        torch.float32, torch.float32, torch.int32, torch.int32)]
    best = torch.empty(1, device="cuda:0", dtype=torch.int64)
    ms = []
    for k in (("noise", kind[1]), kind):
        x, w = _flux(k, rng, n)
        x, w = dev(x), dev(w)
        torch.cuda.synchronize()
        with bls.Plan(max_points=n, max_periods=m, flags=flags) as p:
            for _ in range(4):
                bls.bls_search_unbinned_device(p.handle, np.array([0, n]), t, x, w, per, None,
                                               0.01, 0.1, *out, best)
                bls.bls_synchronize(p.handle)
            ms.append(min(bls.bls_kernel_times(p.handle)))
    print("[ms] noise, flat:", ms, flush=True)
    if kind[0] == 1.0 and not kind[1]:      # the mean is exact
        assert (out[0].cpu().numpy() == 0.0).all() and (out[2].cpu().numpy() == -1).all()
    assert ms[1] <= 2.0 * ms[0], ms


# The block search against the kernel that scores every box: no signal, one
# sign under BLS_DIP_ONLY, weights of any range, a minimum count that no box
# reaches (every box is then in question, or none).
@pytest.mark.parametrize("kind,flags,mip", [
    ("one", 0, 1), ("tenth", 1, 1), ("one, weights", 0, 1), ("tenth, weights", 1, 1),
    ("errors over 10", 0, 1), ("errors over 1000", 0, 1), ("errors over 1000", 1, 3),
    ("noise", 0, 100), ("two values", 0, 1)])
@pytest.mark.parametrize("n,m,nbins,qmin,qmax", [(300, 4000, 300, 0.01, 0.1),
                                                 (1000, 4000, 525, 0.005, 0.06),
                                                 (5000, 2000, 1000, 0.005, 0.05)])
def test_blocks(bls, monkeypatch, kind, flags, mip, n, m, nbins, qmin, qmax):
    print("[case] flat blocks", kind, flags, mip, n, nbins, flush=True)
    nc = 8
    rng = np.random.default_rng(n)
    t = np.sort(rng.uniform(0.0, 60.0, (nc, n)), axis=1)
    x, w = rng.normal(0.0, 1.0, (nc, n)), None
    if kind.startswith("errors"):
        s = np.log10(float(kind.split()[-1]))
        w = 10.0 ** rng.uniform(-s, s, (nc, n))      # weights: errors to the -2
        x /= np.sqrt(w)
    elif kind == "two values":
        x = (x > 1.0) * 1.0
    elif kind != "noise":
        x[:] = 1.0 if kind.startswith("one") else 0.1
        if kind.endswith("weights"):
            w = 10.0 ** rng.uniform(-1.0, 1.0, (nc, n))
    per = synth.log_period_grid(0.2, 10.0, m)
    got, ms = [], []
    for mode in ("0", "1"):
        monkeypatch.setenv("BLS_BLOCK_SEARCH", mode)
        with bls.Plan(max_curves=nc, max_points=nc * n, max_periods=nc * m, flags=flags,
                      min_in_points=mip) as p:
            for _ in range(4):
                r = bls.bls_search_batch(p.handle, np.arange(nc + 1) * n, t.ravel(), x.ravel(),
                                         None if w is None else w.ravel(), per, None, nbins,
                                         qmin, qmax)
            got.append(r)
            ms.append(min(bls.bls_kernel_times(p.handle)))
    print("[ms] every box, blocks:", ms, flush=True)
    for key in got[0]:
        assert np.array_equal(got[0][key], got[1][key], equal_nan=True), key
    assert ms[1] <= 4.0 * ms[0], ms


# Far fewer points than bins: many boxes hold the same points, and tie.  The
# first point is in bin 0 at every period, so that some of the boxes that tie
# with the one from there run past the end of the cycle.
@pytest.mark.parametrize("n,limit", [(4, 12.0), (12, 6.0), (50, 3.0), (200, 3.0)])
@pytest.mark.parametrize("nbins,qmin,qmax", [(300, 0.01, 0.1), (1000, 0.005, 0.05),
                                             (2585, 0.0058, 0.0454)])
@pytest.mark.parametrize("rounded", [False, True])
@pytest.mark.parametrize("weighted,flags", [(False, 0), (True, 1)])
def test_few_points(bls, monkeypatch, n, limit, nbins, qmin, qmax, rounded, weighted, flags):
    print("[case] few points", n, nbins, rounded, weighted, flags, flush=True)
    nc, m = 90, 40
    rng = np.random.default_rng(n)
    t = np.sort(rng.uniform(0.0, 60.0, (nc, n)), axis=1).ravel()
    x = rng.normal(0.0, 1.0, nc * n)
    x = np.round(x) if rounded else x
    w = rng.uniform(0.5, 2.0, nc * n) if weighted else None
    per = synth.log_period_grid(0.2, 20.0, m)
    got, ms = [], []
    for mode in ("0", "1"):
        monkeypatch.setenv("BLS_BLOCK_SEARCH", mode)
        with bls.Plan(max_curves=nc, max_points=nc * n, max_periods=nc * m, flags=flags) as p:
            for _ in range(5):
                r = bls.bls_search_batch(p.handle, np.arange(nc + 1) * n, t, x, w, per, None, nbins,
                                         qmin, qmax)
            got.append(r)
            ms.append(min(bls.bls_kernel_times(p.handle)))
    print("[ms] every box, blocks:", ms, flush=True)
    for key in got[0]:
        assert np.array_equal(got[0][key], got[1][key], equal_nan=True), key
    assert ms[1] <= limit * ms[0], ms


@pytest.mark.parametrize("n,step", [(1700, 0.05), (20000, 0.01)])
@pytest.mark.parametrize("weighted,flags", [(False, 0), (True, 0), (False, 1)])
def test_unbinned_equal_times(bls, n, step, weighted, flags):
    """Times on a coarse grid, several points a time: a run does not split equal
    phases, and the screens see only the edges that runs can have.  The search
    then takes what its sort takes, which is all that a flat curve on the same
    times needs."""
    import torch
    dev = lambda a: None if a is None else torch.tensor(a, device="cuda:0")
    print("[case] equal times", n, step, weighted, flags, flush=True)
    rng = np.random.default_rng(n)
    t = dev(np.round(np.sort(rng.uniform(0.0, 30.0, n)) / step) * step)
    x, w = rng.normal(0.0, 1.0, n), dev(rng.uniform(0.5, 2.0, n)) if weighted else None
    m = max(16, 300000 // n)
    per = dev(synth.log_period_grid(0.2, 20.0, m))
    out = [torch.empty(m, device="cuda:0", dtype=d) for d in (
        torch.float32, torch.float32, torch.int32, torch.int32)]
    best = torch.empty(1, device="cuda:0", dtype=torch.int64)
    ms = []
    for flux in (np.ones(n), x):
        flux = dev(flux)
        torch.cuda.synchronize()
        with bls.Plan(max_points=n, max_periods=m, flags=flags) as p:
            for _ in range(4):
                bls.bls_search_unbinned_device(p.handle, np.array([0, n]), t, flux, w, per, None,
                                               0.05, 0.28, *out, best)
                bls.bls_synchronize(p.handle)
            ms.append(min(bls.bls_kernel_times(p.handle)))
    print("[ms] flat, noise:", ms, flush=True)
    assert ms[1] <= 1.25 * ms[0], ms


# Periods longer than the data with boxes of much of the cycle: many boxes hold
# the same points, and a period's best stays in question until the list of
# candidates has been pruned many times.
@pytest.mark.parametrize("nc,n,m,nbins,qmin,qmax", [(8, 18000, 500, 1460, 0.046, 0.39),
                                                    (40, 2000, 500, 1460, 0.046, 0.39),
                                                    (46, 8000, 70, 2270, 0.041, 0.397)])
@pytest.mark.parametrize("weighted", [False, True])
def test_periods_beyond_the_data(bls, monkeypatch, nc, n, m, nbins, qmin, qmax, weighted):
    print("[case] beyond the data", nc, n, m, nbins, weighted, flush=True)
    rng = np.random.default_rng(n)
    t = np.sort(rng.uniform(0.0, 10.0, (nc, n)), axis=1).ravel()
    x = rng.normal(0.0, 1.0, nc * n)
    w = rng.uniform(0.5, 2.0, nc * n) if weighted else None
    per = synth.log_period_grid(0.2, 20.0, m)
    ms, res = [], []
    for env in ("0", "1"):
        monkeypatch.setenv("BLS_BLOCK_SEARCH", env)
        with bls.Plan(max_curves=nc, max_points=nc * n, max_periods=nc * m) as p:
            t_ = []
            for _ in range(4):
                r = bls.bls_search_batch(p.handle, np.arange(nc + 1) * n, t, x, w, per, None,
                                         nbins, qmin, qmax)
                t_.append(bls.bls_last_stats(p.handle)["search_ms"])
            ms.append(min(t_))
            res.append(r)
    print("[ms] every box, blocks:", ms, flush=True)
    for k in res[0]:
        assert np.array_equal(res[0][k], res[1][k], equal_nan=True), k
    assert ms[1] <= 2.0 * ms[0], ms
