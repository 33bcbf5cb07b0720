"""Calls that reuse the last call's plan: the same batch again (new data in the
same arrays), and what comes between them.  The results are those of a plan
that reuses nothing."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_reused_plan():
    import torch

    import paper_1112_1701_amd as bls
    bls._lib.load()
    dev = lambda a: torch.tensor(a, device="cuda:0")
    n, m = 700, 600
    lcs = [synth.small_curve(60 + k, n, nperiods=m, nbins=150, qmin=0.02, qmax=0.1)
           for k in range(4)]
    per = dev(lcs[0].periods)
    t, x = dev(lcs[0].t), dev(lcs[0].x)
    out = [torch.empty(m, device="cuda:0", dtype=d) for d in (
        torch.float32, torch.float32, torch.int32, torch.int32)]
    out.append(torch.empty(1, device="cuda:0", dtype=torch.int64))

    def call(p, nbins=150):
        torch.cuda.synchronize()
        bls.bls_search_device(p.handle, [0, n], t, x, None, per, None, nbins, 0.02, 0.1, *out)
        bls.bls_synchronize(p.handle)
        return [o.cpu().numpy().copy() for o in out]

    with bls.Plan(max_curves=8, max_points=8 * n, max_periods=8 * m) as p, \
            bls.Plan(max_curves=1, max_points=n, max_periods=m, flags=bls.BLS_NO_GRAPH) as q:
        for k, between in enumerate([None, "host", "unbinned", "bins", "other", "data", None]):
            print("[case] replay", k, between, flush=True)
            lc = lcs[k % 4]
            t.copy_(dev(lc.t))
            x.copy_(dev(lc.x))
            if between == "host":
                bls.bls_search_batch(p.handle, np.arange(4) * n, np.tile(lc.t, 3),
                                     np.tile(lc.x, 3), None, lc.periods, None, 150, 0.02, 0.1)
            elif between == "unbinned":
                o = [torch.empty(m, device="cuda:0", dtype=d) for d in (
                    torch.float32, torch.float32, torch.int32, torch.int32)]
                b = torch.empty(1, device="cuda:0", dtype=torch.int64)
                bls.bls_search_unbinned_device(p.handle, np.array([0, n]), t, x, None, per, None,
                                               0.02, 0.1, *o, b)
                bls.bls_synchronize(p.handle)
            elif between == "bins":
                bls.bls_debug_phase_bins(p.handle, lc.t, 1.3, 100)
            elif between == "other":
                call(p, 90)
            elif between == "data":                     # an invalid curve, then this one
                x[3] = float("nan")
                with pytest.raises(bls.BlsError):
                    call(p)
                x.copy_(dev(lc.x))
            first = call(p)
            again = call(p)
            assert bls.bls_last_stats(p.handle)["graph_replayed"] == 1
            want = call(q)
            assert bls.bls_last_stats(q.handle)["graph_replayed"] == 0
            for a, b, c in zip(first, again, want):
                assert np.array_equal(a, c) and np.array_equal(b, c), (k, between)


@pytest.mark.parametrize("nc", [1, 5, 300])
def test_status_of_queued_calls(nc):
    """The status that a wait reports is that of the last call queued before
    it, whichever curve it is of."""
    import torch

    import paper_1112_1701_amd as bls
    bls._lib.load()
    dev = lambda a: torch.tensor(a, device="cuda:0")
    n, m = 70, 40
    lc = synth.small_curve(90, n, nperiods=m, nbins=50, qmin=0.02, qmax=0.2)
    t, good = dev(np.tile(lc.t, nc)), dev(np.tile(lc.x, nc))
    bad = good.clone()
    bad[(nc - 1) * n + 5] = float("inf")
    per, off = dev(lc.periods), np.arange(nc + 1) * n
    out = [torch.empty(nc * m, device="cuda:0", dtype=d) for d in (
        torch.float32, torch.float32, torch.int32, torch.int32)]
    best = torch.empty(nc, device="cuda:0", dtype=torch.int64)
    torch.cuda.synchronize()
    with bls.Plan(max_curves=nc, max_points=nc * n, max_periods=nc * m) as p:
        for x in ([good], [bad], [bad, good], [good, bad], [good]):
            print("[case] status", nc, len(x), flush=True)
            for v in x:
                bls.bls_search_device(p.handle, off, t, v, None, per, None, 50, 0.02, 0.2,
                                      *out, best)
            if x[-1] is good:
                bls.bls_synchronize(p.handle)
            else:
                with pytest.raises(bls.BlsError, match="curve %d" % (nc - 1)):
                    bls.bls_synchronize(p.handle)


@pytest.mark.parametrize("nc,m", [(1, 1), (1, 31), (3, 33), (70, 96), (2, 5000)])
@pytest.mark.parametrize("weighted", [False, True])
def test_host_results_where_the_kernels_write_them(monkeypatch, nc, m, weighted):
    """Results that the kernels write to pinned memory are those that a plan
    without it copies from the device."""
    import paper_1112_1701_amd as bls
    bls._lib.load()
    n = 90
    lcs = [synth.small_curve(70 + k, n, nperiods=m, nbins=60, qmin=0.02, qmax=0.2,
                             weighted=weighted) for k in range(nc)]
    t, x = (np.concatenate([getattr(c, a) for c in lcs]) for a in "tx")
    w = np.concatenate([c.w for c in lcs]) if weighted else None
    got = []
    for hook in (None, "pinned"):
        print("[case] host results", nc, m, weighted, hook, flush=True)
        monkeypatch.setenv("BLS_DEBUG_FAIL_ALLOC", hook) if hook else None
        with bls.Plan(max_curves=nc + 1, max_points=nc * n + 9, max_periods=nc * m + 5) as p:
            for _ in range(2):
                got.append(bls.bls_search_batch(p.handle, np.arange(nc + 1) * n, t, x, w,
                                                lcs[0].periods, None, 60, 0.02, 0.2))
    for g in got[1:]:
        for key in got[0]:
            assert np.array_equal(g[key], got[0][key], equal_nan=True), key
