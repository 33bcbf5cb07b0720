"""The eclipse window with a wave per period (calls of many periods), at bin
counts and cadence lengths on both sides of its limits: the counts are the
oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nphase,dur,m", [(1, 0.02, 2), (2, 0.3, 2), (63, 0.02, 1), (65, 0.05, 2),
                                          (200, 0.02, 2), (1001, 0.3, 2), (2400, 0.02, 2),
                                          (2600, 0.02, 2)])
def test_wave_per_period(nphase, dur, m):
    import torch

    import paper_1112_1701_amd as bls
    bls._lib.load()
    rng = np.random.default_rng(nphase)
    sizes = [1, 2, 63, 64, 65, 570, 1024, 1025, 1500]
    ts = [synth.T_START + np.sort(rng.uniform(0.0, 40.0, n)) for n in sizes]
    n_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    t = np.concatenate(ts)
    w = (rng.random(t.size) > 0.1) * 1.0
    w[n_off[:-1]] = 1.0
    counts = [2000, 1999, 2003, 1998, 2001, 2100, 2000, 1997, 2500]  # 18598 periods
    grids = [synth.log_period_grid(0.1, 10.0, k) for k in counts]
    p_off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    dev = lambda a: torch.tensor(a, device="cuda:0")
    print("[case] window waves", nphase, dur, m, flush=True)
    for wt in (None, w):
        out = torch.empty(int(p_off[-1]), dtype=torch.int32, device="cuda:0")
        args = (dev(t), dev(np.concatenate(grids)))
        wd = None if wt is None else dev(wt)
        with bls.Plan(max_curves=16, max_points=1 << 14, max_periods=1 << 15) as p:
            torch.cuda.synchronize()
            bls.bls_eclipse_window_device(p.handle, n_off, *args, p_off, nphase, dur, m, out,
                                          weights=wd)
        got = out.cpu().numpy()
        for c, tc in enumerate(ts):
            wc = None if wt is None else wt[n_off[c]:n_off[c + 1]]
            o = oracle.eclipse_window(tc, wc, grids[c], nphase, dur, m)
            assert np.array_equal(got[p_off[c]:p_off[c + 1]], o), (c, sizes[c])
