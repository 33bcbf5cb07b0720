"""Cadences of more cycles than an int holds, in the eclipse window's two
kernels: refused, and nothing of them stays for the next call."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nper", [300, 20000])      # a workgroup, a wave per period
@pytest.mark.parametrize("cycles", [2.0**30, 2.0**31, 2.0**33, 2.0**63])
def test_cycles_beyond_int(nper, cycles):
    import torch

    import paper_1112_1701_amd as bls
    bls._lib.load()
    dev = lambda a: torch.tensor(a, device="cuda:0")
    per = synth.log_period_grid(0.2, 5.0, nper)
    good = np.sort(np.random.default_rng(1).uniform(0.0, 30.0, 90))
    far = good.copy()
    far[-1] = cycles * 0.2 * 1.01
    print("[case] window cycles", nper, cycles, flush=True)
    out = torch.empty(nper, dtype=torch.int32, device="cuda:0")
    P = dev(per)
    with bls.Plan(max_points=128, max_periods=nper) as p:
        for t in (far, good):
            T = dev(t)
            torch.cuda.synchronize()
            call = lambda: bls.bls_eclipse_window_device(p.handle, [0, 90], T, P, None, 200, 0.05,
                                                         2, out)
            if t is far:
                with pytest.raises(bls.BlsError) as e:
                    call()
                assert e.value.status == bls.BLS_ERR_CAPACITY
            else:
                call()
    assert np.array_equal(out.cpu().numpy(), oracle.eclipse_window(good, None, per, 200, 0.05, 2))
