"""The strides of the search kernel's period planes: the one of the fewest bank
conflicts, as counted access by access, and found once for curves of one shape
(a call without a plan fits every curve's tile anew)."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1112_1701_amd", "csrc")
LIBDIR = os.path.join(ROOT, "paper_1112_1701_amd")

DRIVER = r'''
#include "bls_plan.h"
#include <algorithm>
#include <chrono>
#include <cstdio>
using namespace bls;

// 64-bit reads of lanes (start bin, period) = divmod(task, tile), served 16
// lanes at a time from 32 banks of 4 bytes
static int cycles(long stride, int tile, int nbins) {
  int total = 0;
  for (int g = 0; g < 64; ++g) {
    int bank[32] = {0}, worst = 0;
    for (int l = 0; l < 16; ++l) {
      const long q = g * 16 + l, j = q / tile, t = q % tile;
      if (j >= nbins) continue;
      const long word = 2 * (t * stride + j);
      worst = std::max(worst, ++bank[word % 32]);
      worst = std::max(worst, ++bank[(word + 1) % 32]);
    }
    total += worst;
  }
  return total;
}

int main() {
  for (int pass = 0; pass < 2; ++pass)  // computed, then kept or computed again
    for (int nb : {2, 3, 7, 16, 51, 100, 333, 1023, 1024, 1025, 4096})
      for (int tile = 1; tile <= kTileMax; ++tile)
        for (int w = 1; w <= 2; ++w) {
          const int kmax = std::max(1, nb / 10), hb = hist_words(nb, kmax);
          int best = hb, least = 0;
          for (int hs = hb; hs < hb + 16; ++hs) {
            const int c = cycles((long)hs * w, tile, nb);
            if (hs == hb || c < least) best = hs, least = c;
          }
          if (hist_stride(nb, kmax, tile, w == 2) != best) {
            printf("stride of %d bins, %d periods\n", nb, tile);
            return 1;
          }
        }
  typedef std::chrono::steady_clock clock;
  double once = 0, again = 1e30;
  int T, hs;
  for (int k = 0; k < 5; ++k) {
    const auto t0 = clock::now();
    fit_tile(140 + k, 14, 5000, 25000, kTileMax, true, &T, &hs);
    const auto t1 = clock::now();
    for (int i = 0; i < 200; ++i) fit_tile(140 + k, 14, 5000, 25000, kTileMax, true, &T, &hs);
    const auto t2 = clock::now();
    once = std::max(once, std::chrono::duration<double>(t1 - t0).count());
    again = std::min(again, std::chrono::duration<double>(t2 - t1).count());
  }
  printf("%g %g\n", once * 1e6, again * 1e6);
  if (again > 50 * once) return 1;  // 200 fits, each a part of the first
  double first = 0;                 // and for a batch of many bin counts
  again = 1e30;
  for (int pass = 0; pass < 6; ++pass) {
    const auto t0 = clock::now();
    for (int nb = 1100; nb < 1300; ++nb) fit_tile(nb / 4, nb / 40, 5000, 25000, kTileMax, true, &T, &hs);
    for (int nb = 200; nb < 400; ++nb) fit_tile(nb, nb / 10, 5000, 21200, kTileMax, false, &T, &hs);
    const double s = std::chrono::duration<double>(clock::now() - t0).count();
    if (pass == 0) first = s;
    else again = std::min(again, s);
  }
  printf("%g %g\n", first * 1e6, again * 1e6);
  return again > 0.3 * first;
}
'''


def test_strides():
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
        print(out.stdout)
