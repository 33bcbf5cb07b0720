"""The eclipse window at cadence lengths on both sides of what a wave holds (1024
points), in calls of many periods: the counts are the oracle's, and longer
cadences, which a workgroup takes, cost no more than their points."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


@pytest.mark.parametrize("sizes", [(1, 63, 64, 65, 570, 1023, 1024), (1024, 1025), (2048, 2049, 3)])
@pytest.mark.parametrize("nphase,m", [(1, 2), (65, 1), (300, 2), (2400, 2)])
def test_lengths(bls, sizes, nphase, m):
    import torch
    dev = lambda a: torch.tensor(a, device="cuda:0")
    print("[case] window lengths", sizes, nphase, m, flush=True)
    rng = np.random.default_rng(sizes[-1])
    nper = 20000 // len(sizes) + 1
    ts = [synth.T_START + np.sort(rng.uniform(0.0, 40.0, n)) for n in sizes]
    n_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = (rng.random(int(n_off[-1])) > 0.2) * 1.0
    w[n_off[:-1]] = 1.0
    per = synth.log_period_grid(0.1, 10.0, nper)
    T, P = dev(np.concatenate(ts)), dev(per)
    for wt in (None, w):
        out = torch.empty(len(sizes) * nper, dtype=torch.int32, device="cuda:0")
        W = None if wt is None else dev(wt)
        torch.cuda.synchronize()
        with bls.Plan(max_curves=8, max_points=1 << 14, max_periods=1 << 16) as p:
            bls.bls_eclipse_window_device(p.handle, n_off, T, P, None, nphase, 0.05, m, out, weights=W)
        got = out.cpu().numpy().reshape(len(sizes), nper)
        some = np.unique(np.concatenate([np.arange(0, nper, 37), [nper - 1]]))
        for c, tc in enumerate(ts):
            wc = None if wt is None else wt[n_off[c]:n_off[c + 1]]
            o = oracle.eclipse_window(tc, wc, per[some], nphase, 0.05, m)
            assert np.array_equal(got[c, some], o), (c, sizes[c])


def test_beyond_a_wave(bls):
    import torch
    dev = lambda a: torch.tensor(a, device="cuda:0")
    print("[case] window beyond a wave", flush=True)
    nc, nper, ms = 24, 20000, []
    P = dev(synth.log_period_grid(0.1, 10.0, nper))
    for n in (1024, 1100):
        rng = np.random.default_rng(1)
        t = dev(np.tile(np.sort(rng.uniform(0.0, 90.0, n)), nc))
        w = dev((rng.random(nc * n) > 0.3) * 1.0)
        out = torch.empty(nc * nper, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        k = []
        with bls.Plan(max_curves=nc, max_points=nc * n, max_periods=nc * nper) as p:
            for _ in range(4):
                bls.bls_eclipse_window_device(p.handle, np.arange(nc + 1) * n, t, P, None, 300, 0.05,
                                              2, out, weights=w)
                k.append(bls.bls_last_stats(p.handle)["search_ms"])
        ms.append(min(k))
    print("[ms] 1024 points, 1100:", ms, flush=True)
    assert ms[1] <= 1.5 * ms[0], ms
