"""The block search's LDS (no GPU): whatever curves share a launch, it needs no
more than a workgroup has.  The planning functions of the library, run on the
host over batches whose planes and whose scratch are largest in different
curves."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1112_1701_amd", "csrc")
LIBDIR = os.path.join(ROOT, "paper_1112_1701_amd")

DRIVER = r'''
#include "bls_plan.h"
#include <cstdio>
#include <vector>
using namespace bls;
namespace {
constexpr int kLds = 160 * 1024, kCus = 256;
int g_bad = 0, g_block = 0;
CurveShape shape(int nbins, double qmax) {
  CurveShape s{};
  s.n = 3000;
  s.nperiods = 4000;
  s.nbins = nbins;
  bls_width_range(nbins, 0.01, qmax, &s.kmin, &s.kmax);
  return s;
}
// LDS of the curves in one launch, each with its own budget.
void launch(const char *what, const std::vector<CurveShape> &v, bool weighted,
            const std::vector<int> &budget, double qmax) {
  LdsLayout lds;
  for (size_t c = 0; c < v.size(); ++c) {
    TileChoice tc;
    tc.lds_budget = budget[c];
    tc.tile_cap = 4;
    tc.block = true;
    CurveDesc d;
    fill_curve_desc(v[c], weighted, tc, false, true, d);
    lds.add(d, true);
  }
  ++g_block;
  if (lds.total() + kBlockStaticLds > kLds && g_bad++ < 20)
    printf("%s: weighted %d qmax %g bins %d .. %d: %d bytes\n", what, (int)weighted, qmax,
           v.front().nbins, v.back().nbins, lds.total());
}
}  // namespace
int main() {
  bls_plan p;
  p.num_cus = kCus;
  p.max_lds = kLds;
  p.cfg.flags = BLS_NO_AUTOTUNE;
  for (int weighted = 0; weighted < 2; ++weighted)
    for (double qmax : {0.05, 0.1, 0.15, 0.3, 0.5})
      for (int wide = 300; wide <= 4096; wide += 41)
        for (int narrow = 100; narrow < wide; narrow += 73) {
          const CurveShape a = shape(wide, qmax), b = shape(narrow, qmax);
          // a plan's batch (budget of the median curve), the plan-free search
          // (of the widest), and two requests of a server's tick (each its own)
          const std::vector<CurveShape> v = {a, a, a, b};
          if (block_batch(v.data(), 4, weighted, 1, false, kCus, kLds)) {
            const TileChoice tc = choose_tiles(&p, v, weighted);
            if (tc.block) launch("plan", v, weighted, std::vector<int>(4, tc.lds_budget), qmax);
            launch("noalloc", v, weighted,
                   std::vector<int>(4, block_lds_budget(a, weighted, kLds)), qmax);
          }
          if (block_batch(&a, 1, weighted, 1, false, kCus, kLds) &&
              block_batch(&b, 1, weighted, 1, false, kCus, kLds))
            launch("server", {a, b}, weighted,
                   {block_lds_budget(a, weighted, kLds), block_lds_budget(b, weighted, kLds)},
                   qmax);
        }
  printf("%d launches, %d too large\n", g_block, g_bad);
  return g_bad != 0 || g_block < 1000;
}
'''


def test_mixed_launches_fit_the_lds():
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "t.cpp"), os.path.join(d, "t")
        open(src, "w").write(DRIVER)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__",
                               "-I/opt/rocm/include", "-I" + CSRC, src, "-o", exe,
                               os.path.join(LIBDIR, "libbls_mi355x.so"),
                               "-Wl,-rpath," + LIBDIR, "-L/opt/rocm/lib", "-lamdhip64",
                               "-Wl,-rpath,/opt/rocm/lib"])
        out = subprocess.run([exe], capture_output=True, text=True)
        assert out.returncode == 0, out.stdout + out.stderr
