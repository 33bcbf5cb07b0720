"""Clipped statistics at the bin sizes where a wave's share, or its LDS list,
ends: the flags, counts and statistics are the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stars", [1, 4, 255, 256, 257, 260, 1023, 1500, 4200])
def test_members_per_bin(stars):
    import torch

    import paper_1112_1701_amd as bls
    bls._lib.load()
    rng = np.random.default_rng(stars)
    n = np.full(2 * stars, 6)                        # two bins, interleaved
    n_off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    sig = np.where(rng.random(2 * stars) < 0.05, 0.5, 0.01 * rng.uniform(0.8, 1.2, 2 * stars))
    x = 15.0 + np.repeat(sig, 6) * rng.standard_normal(12 * stars)
    mag = 14.05 + 0.1 * (np.arange(2 * stars) % 2)
    chips = np.array([0, 2 * stars], np.int64)
    f64, i32 = torch.float64, torch.int32
    dev = lambda a: torch.tensor(a, device="cuda:0")
    out = {k: torch.empty(m, dtype=d, device="cuda:0") for k, m, d in (
        ("rms", 2 * stars, f64), ("bin", 2 * stars, i32), ("flag", 2 * stars, i32),
        ("bin_mean", 3, f64), ("bin_std", 3, f64), ("bin_count", 3, i32))}
    print("[case] variability bins", stars, flush=True)
    xd, md = dev(x), dev(mag)
    with bls.Plan(max_curves=2 * stars, max_points=1 << 16) as p:
        torch.cuda.synchronize()
        bls.bls_variability_device(p.handle, n_off, xd, None, md, chips, 3, out, origin=14.0)
    g = {k: v.cpu().numpy() for k, v in out.items()}
    o = oracle.variability(x, None, n_off, mag, chips, 3, origin=14.0)
    # FP64 sums of up to 4200 values in another order (5e-13 relative), the
    # deviation about a mean ten times its size
    for k, ko in (("bin", "bin"), ("flag", "flag"), ("bin_count", "count")):
        assert np.array_equal(g[k], np.ravel(o[ko])), k
    for k, ko in (("rms", "rms"), ("bin_mean", "mean"), ("bin_std", "std")):
        assert np.allclose(g[k], np.ravel(o[ko]), rtol=1e-10, atol=1e-13, equal_nan=True), k
