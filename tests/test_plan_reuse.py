"""Reuse of the last search's plan: planning another batch ends it, also where
that planning fails, because the descriptors and the places of the segments in
their block have changed by then."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1112_1701_amd", "csrc")
LIBDIR = os.path.join(ROOT, "paper_1112_1701_amd")

DRIVER = r'''
#include "bls_plan.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace bls;
int main() {
  bls_plan p;   // (host members only; nothing is queued)
  p.num_cus = 256;
  p.max_lds = 160 * 1024;
  std::vector<char> host(desc_bytes(8)), device(desc_bytes(8));
  p.h_curves = reinterpret_cast<CurveDesc *>(host.data());
  p.d_curves = reinterpret_cast<CurveDesc *>(device.data());
  place_desc(&p, 1);
  const void *before = p.d_seg_start;
  p.replay_valid = true;
  CurveShape s{};
  s.n = 100;
  s.nperiods = 5000;
  s.nbins = 1000;
  s.kmin = 5;
  s.kmax = 50;
  TileChoice tc;
  tc.lds_budget = 400000;   // tiles that no workgroup has room for
  PlannedBatch pb;
  const int st = plan_batch(&p, std::vector<CurveShape>(4, s), true, tc, pb);
  if (st != BLS_ERR_CAPACITY || p.d_seg_start == before) return 1;
  printf("%s\n", p.replay_valid ? "still reused" : "ended");
  return p.replay_valid;
}
'''


def test_failed_planning_ends_reuse():
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "t.cpp"), os.path.join(d, "t")
        open(src, "w").write(DRIVER)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__",
                               "-I/opt/rocm/include", "-I" + CSRC, src, "-o", exe,
                               os.path.join(LIBDIR, "libbls_mi355x.so"),
                               "-Wl,-rpath," + LIBDIR, "-L/opt/rocm/lib", "-lamdhip64",
                               "-Wl,-rpath,/opt/rocm/lib"])
        out = subprocess.run([exe], capture_output=True, text=True)
        assert out.returncode == 0 and out.stdout.strip() == "ended", out.stdout + out.stderr


@pytest.mark.gpu
def test_failing_call_between_two_like_calls(monkeypatch):
    """The same on the GPU: a device call, a host call of another number of
    curves that planning refuses, the device call again."""
    import numpy as np
    import torch

    import paper_1112_1701_amd as bls
    import synth
    bls._lib.load()
    n, m = 300, 200
    lc = synth.small_curve(61, n, nperiods=m, nbins=200, qmin=0.02, qmax=0.1)
    dev = lambda a: torch.tensor(a, device="cuda:0")
    t, x, per = dev(lc.t), dev(lc.x), dev(lc.periods)
    out = [torch.empty(m, device="cuda:0", dtype=d) for d in (
        torch.float32, torch.float32, torch.int32, torch.int32)]
    out.append(torch.empty(1, device="cuda:0", dtype=torch.int64))
    torch.cuda.synchronize()
    got = []
    with bls.Plan(max_curves=8, max_points=8 * n, max_periods=8 * m) as p:
        for _ in range(2):
            bls.bls_search_device(p.handle, [0, n], t, x, None, per, None, 200, 0.02, 0.1, *out)
            bls.bls_synchronize(p.handle)
            got.append([o.cpu().numpy().copy() for o in out])
            assert bls.bls_last_stats(p.handle)["graph_replayed"] == 0
            with monkeypatch.context() as mp:
                mp.setenv("BLS_LDS_BUDGET", "400000")
                mp.setenv("BLS_BLOCK_SEARCH", "0")
                with pytest.raises(bls.BlsError) as e:
                    bls.bls_search_batch(p.handle, np.arange(5) * n, np.tile(lc.t, 4),
                                         np.tile(lc.x, 4), np.ones(4 * n), lc.periods, None,
                                         1000, 0.005, 0.05)
                assert e.value.status == bls.BLS_ERR_CAPACITY
    for a, b in zip(*got):
        assert np.array_equal(a, b)
