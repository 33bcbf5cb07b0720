"""Device memory of the host-array calls: the kernels write the results to the
plan's pinned memory, so the plan holds none of its results' size on the
device unless pinned memory is refused (run in a child process, whose device
memory is its own)."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r'''
import sys
import numpy as np
import torch
import paper_1112_1701_amd as bls
M = 1 << 25
rng = np.random.default_rng(2)
t = np.sort(rng.uniform(0.0, 30.0, 500))
x = rng.normal(1.0, 0.01, 500)
per = np.linspace(0.5, 5.0, 40)
with bls.Plan(max_curves=8, max_points=10000, max_periods=4000) as p:   # loads the kernels
    bls.bls_search(p.handle, t, x, None, per, 100, 0.01, 0.1)
with bls.Plan(max_curves=8, max_points=10000, max_periods=M) as p:
    before = torch.cuda.mem_get_info()[0]
    r = bls.bls_search(p.handle, t, x, None, per, 100, 0.01, 0.1)
    used = before - torch.cuda.mem_get_info()[0]
np.savez(sys.argv[1], used=used, periods=8 * M, results=16 * M, **r)
'''


@pytest.mark.parametrize("refused", [False, True])
def test_host_results_take_no_device_memory(tmp_path, refused):
    env = dict(os.environ, PYTHONPATH=ROOT)
    env.pop("BLS_DEBUG_FAIL_ALLOC", None)
    if refused:
        env["BLS_DEBUG_FAIL_ALLOC"] = "pinned"
    out = str(tmp_path / "r.npz")
    subprocess.check_call([sys.executable, "-c", CHILD, out], env=env, timeout=100)
    z = np.load(out)
    used, periods, results = int(z["used"]), int(z["periods"]), int(z["results"])
    # the inputs' block, and half a block of results either way
    if refused:
        assert used >= periods + results
    else:
        assert used < periods + results // 2
    assert np.all(np.isfinite(z["sr"])) and int(z["best_index"]) == int(np.argmax(z["sr"]))
