"""The block search (bls_blocks.hip) against the kernel that scores every box
and against the FP64 oracle.

Both kernels return the same boxes and the same bits: sizes where the block
layout changes (blocks of 1, 3, 5, 7 and more bins, one to four waves-full of
them, last blocks that end early, widths beyond a wave), and inputs whose
boxes tie (few points, few flux values, an outlier, no signal at all).
"""
import sys

import numpy as np
import pytest

import oracle
import synth
from tests.parity import check_curve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bls():
    import paper_1112_1701_amd as bls
    bls._lib.load()
    return bls


def _both(bls, monkeypatch, lc, **cfg):
    out = []
    for mode in ("0", "1"):
        monkeypatch.setenv("BLS_BLOCK_SEARCH", mode)
        with bls.Plan(max_points=1 << 16, max_periods=1 << 12, **cfg) as p:
            out.append(bls.bls_search(p.handle, lc.t, lc.x, lc.w, lc.periods, lc.nbins,
                                      lc.qmin, lc.qmax))
    for key in ("sr", "depth", "jstart", "kwidth"):
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key
    assert out[0]["best_index"] == out[1]["best_index"]
    return out[1]


@pytest.mark.parametrize("nbins,qmin,qmax,n", [
    (4, 0.1, 0.5, 50),            # fewest bins that have blocks to pair
    (64, 0.02, 0.2, 700),         # one bin per block
    (65, 0.02, 0.5, 700),         # blocks of three, the last one short
    (300, 0.01, 0.1, 2000),       # blocks of five, none short
    (321, 0.01, 0.1, 900),        # blocks of seven, the last one short
    (1000, 0.005, 0.05, 4000),    # three waves-full of blocks
    (1000, 0.1, 0.5, 1500),       # widths of up to eight waves
    (4096, 0.001, 0.1, 3000),     # most bins, larger blocks
])
@pytest.mark.parametrize("weighted,flags,mip", [(False, 0, 1), (True, 0, 1), (False, 1, 3),
                                                (True, 1, 3)])
def test_blocks_equal_every_box(bls, monkeypatch, nbins, qmin, qmax, n, weighted, flags, mip):
    lc = synth.small_curve(9000 + nbins, n, nperiods=60, nbins=nbins, qmin=qmin, qmax=qmax,
                           weighted=weighted)
    print("[case] blocks", nbins, qmin, qmax, n, weighted, flags, mip, flush=True)
    g = _both(bls, monkeypatch, lc, flags=flags, min_in_points=mip)
    o = oracle.search(lc.t, lc.x, lc.w, lc.periods, lc.nbins, lc.qmin, lc.qmax,
                      dip_only=bool(flags), min_in_points=mip)
    check_curve(lc, g, o, label="blocks %d" % nbins)


@pytest.mark.parametrize("kind", ["binary", "constant", "rounded", "outlier", "alternating"])
@pytest.mark.parametrize("n,nbins,weights", [(2, 10, None), (8, 50, "spread"),
                                             (60, 400, None), (300, 150, "few"),
                                             (3000, 64, None), (40, 63, "few"),
                                             (40, 64, "few"), (90, 100, "spread")])
def test_blocks_ties(bls, monkeypatch, kind, n, nbins, weights):
    rng = np.random.default_rng(n + nbins)
    t = np.sort(rng.uniform(0.0, 30.0, n))
    x = {"binary": (rng.random(n) < 0.2) * 1.0, "constant": np.ones(n),
         "rounded": np.round(rng.normal(0.0, 1.0, n)),
         "outlier": 1e-4 * rng.normal(0.0, 1.0, n) + (np.arange(n) == n // 2),
         "alternating": np.where(np.arange(n) % 2 == 0, 1.0, -1.0)}[kind]
    w = {None: None, "few": rng.choice([0.0, 1.0, 2.0, 4.0], n),
         "spread": 10.0 ** rng.uniform(-3.0, 3.0, n)}[weights]
    lc = synth.LightCurve(t, x, w, synth.log_period_grid(0.3, 9.0, 150), nbins, 0.02, 0.3)
    print("[case] ties", kind, n, nbins, weights, flush=True)
    for cfg in (dict(), dict(flags=bls.BLS_DIP_ONLY, min_in_points=2)):
        _both(bls, monkeypatch, lc, **cfg)


@pytest.mark.parametrize("nbins,qmin,qmax,n", [(64, 0.02, 0.2, 700), (1000, 0.005, 0.05, 4000)])
@pytest.mark.parametrize("weighted,flags", [(False, 0), (True, 0), (False, 1), (True, 1)])
def test_register_copies_agree(bls, monkeypatch, nbins, qmin, qmax, n, weighted, flags):
    """The copies of four and of more waves per SIMD, each forced, return the
    bits of the kernel that scores every box."""
    lc = synth.small_curve(9300 + nbins, n, nperiods=1500, nbins=nbins, qmin=qmin, qmax=qmax,
                           weighted=weighted)
    print("[case] copies", nbins, n, weighted, flags, flush=True)
    for wide in ("0", "1"):
        monkeypatch.setenv("BLS_WIDE_REGS", wide)
        _both(bls, monkeypatch, lc, flags=flags)
