"""Calls on both sides of the built-in tile table's line (1024 periods per
CU; tiles of at least four periods): the results do not
depend on the tile, and are the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from tests.parity import check_curve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("curves,nbins", [(25, 120), (26, 120), (26, 300), (26, 400), (26, 640)])
def test_tile_table(monkeypatch, curves, nbins, weighted):
    import paper_1112_1701_amd as bls
    bls._lib.load()
    n, m = 90, 10240                                # 26 curves: 1040 periods per CU
    lcs = [synth.small_curve(700 + c, n, nperiods=m, nbins=nbins, qmin=0.02, qmax=0.04,
                             weighted=weighted) for c in range(curves)]
    per = lcs[0].periods
    args = (np.arange(curves + 1) * n, np.concatenate([lc.t for lc in lcs]),
            np.concatenate([lc.x for lc in lcs]),
            np.concatenate([lc.w for lc in lcs]) if weighted else None, per, None, nbins, 0.02,
            0.04)
    print("[case] tiles", curves, nbins, weighted, flush=True)
    with bls.Plan(max_curves=curves, max_points=curves * n, max_periods=curves * m) as p:
        got = bls.bls_search_batch(p.handle, *args)
        monkeypatch.setenv("BLS_LDS_BUDGET", "32768")
        wide = bls.bls_search_batch(p.handle, *args)
    for key in ("sr", "depth", "jstart", "kwidth", "best_index"):
        assert np.array_equal(got[key], wide[key]), key
    c = curves - 1
    o = oracle.search(lcs[c].t, lcs[c].x, lcs[c].w, per, nbins, 0.02, 0.04)
    check_curve(lcs[c], {k: got[k][c * m:(c + 1) * m] if k != "best_index" else int(got[k][c])
                         for k in ("sr", "depth", "jstart", "kwidth", "best_index")}, o,
                label="tiles %d" % nbins)
