"""Launches of the block search that mix curves: bin counts whose planes and
whose scratch are largest in different curves, in a plan's batch, the plan-free
search and a server's tick, and ticks that hold every kind of request.  The
results are the bits of the kernel that scores every box, one curve at a time.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

KEYS = ("sr", "jstart", "kwidth")


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


def _curves(nbins, qmax, weighted, m, n=800):
    return [synth.small_curve(400 + k, n + 13 * k, nperiods=m, nbins=nb, qmin=0.01, qmax=q,
                              weighted=weighted)
            for k, (nb, q) in enumerate(zip(nbins, qmax))]


def _alone(bls, monkeypatch, lcs):
    monkeypatch.setenv("BLS_BLOCK_SEARCH", "0")
    with bls.Plan(max_points=1 << 16, max_periods=1 << 14) as p:
        return [bls.bls_search(p.handle, lc.t, lc.x, lc.w, lc.periods, lc.nbins, lc.qmin, lc.qmax)
                for lc in lcs]


def _same(got, want, label):
    for key in KEYS:
        assert np.array_equal(np.asarray(got[key], np.float64),
                              np.asarray(want[key], np.float64)), (label, key)
    assert got["best_index"] == want["best_index"], label


# a plane of its own nearly fills the LDS with the first counts, the narrow
# curves' tiles hold four periods
@pytest.mark.parametrize("nbins,qmax,weighted", [((2500, 2500, 2500, 300), 0.15, True),
                                                 ((3500, 3500, 3500, 500), 0.3, True),
                                                 ((3949, 3949, 3949, 2801), 0.05, False)])
@pytest.mark.parametrize("path", ["plan", "noalloc"])
def test_batches_of_wide_and_narrow_grids(bls, monkeypatch, nbins, qmax, weighted, path):
    m = 500
    print("[case] mixed batch", nbins, qmax, weighted, path, flush=True)
    lcs = _curves(nbins, [qmax] * len(nbins), weighted, m)
    want = _alone(bls, monkeypatch, lcs)
    monkeypatch.setenv("BLS_BLOCK_SEARCH", "1")
    off = np.concatenate([[0], np.cumsum([lc.n for lc in lcs])])
    p_off = np.arange(len(lcs) + 1) * m
    cat = lambda a: np.concatenate([getattr(lc, a) for lc in lcs])
    t, x, w, per = cat("t"), cat("x"), cat("w") if weighted else None, cat("periods")
    if path == "plan":
        with bls.Plan(max_curves=8, max_points=1 << 16, max_periods=1 << 14) as p:
            r = bls.bls_search_batch(p.handle, off, t, x, w, per, p_off, np.array(nbins), 0.01,
                                     qmax)
    else:
        import torch
        dev = lambda a: None if a is None else torch.tensor(a, device="cuda:0")
        new = lambda d, k: torch.empty(k, device="cuda:0", dtype=d)
        r = dict(sr=new(torch.float32, 4 * m), depth=new(torch.float32, 4 * m),
                 jstart=new(torch.int32, 4 * m), kwidth=new(torch.int32, 4 * m),
                 best_index=new(torch.int64, 4))
        args = [dev(a) for a in (t, x, w, per)]
        torch.cuda.synchronize()
        bls.bls_search_device_noalloc(off, *args, p_off, np.array(nbins), 0.01, qmax,
                                      r["sr"], r["depth"], r["jstart"], r["kwidth"],
                                      r["best_index"])
        torch.cuda.synchronize()
        r = {k: v.cpu().numpy() for k, v in r.items()}
    for c, wc in enumerate(want):
        got = {k: r[k][c * m:(c + 1) * m] for k in KEYS}
        got["sr"] = np.float32(got["sr"])
        _same(dict(got, best_index=r["best_index"][c]), dict(wc, sr=np.float32(wc["sr"])), c)


@pytest.mark.parametrize("nbins,qmax,weighted", [
    ((2600, 300, 2600, 300), (0.1,) * 4, (True,) * 4),       # as above, one tick
    ((3949, 2801, 300, 300), (0.05,) * 4, (False,) * 4),
    # block search and every box (boxes above half the bins), with and without
    # weights
    ((300, 150, 400, 200, 1000, 120), (0.1, 0.7, 0.1, 0.7, 0.05, 0.6),
     (False, False, True, True, True, False)),
])
def test_ticks_of_every_kind(bls, monkeypatch, nbins, qmax, weighted):
    print("[case] mixed tick", nbins, qmax, weighted, flush=True)
    lcs = [_curves([nb], [q], wt, 2500, n=600 + 31 * k)[0]
           for k, (nb, q, wt) in enumerate(zip(nbins, qmax, weighted))]
    want = _alone(bls, monkeypatch, lcs)
    monkeypatch.setenv("BLS_BLOCK_SEARCH", "1")
    srv = bls.bls_server_create(max_slots=8, arena_bytes=64 << 20, tick_cost=2e8)
    try:
        tickets = [bls.bls_server_submit(srv, lc.t, lc.x, lc.w, lc.periods, lc.nbins, lc.qmin,
                                         lc.qmax) for lc in lcs]
        res = [bls.bls_server_wait(srv, tk, 60.0) for tk in tickets]
        stats = bls.bls_server_get_stats(srv)
    finally:
        bls.bls_server_destroy(srv)
    assert stats["completed"] == len(lcs) and stats["failed"] == 0
    for k, (r, wc) in enumerate(zip(res, want)):
        assert r["status"] == bls.BLS_OK
        _same(r, dict(wc, sr=np.float32(wc["sr"])), k)
