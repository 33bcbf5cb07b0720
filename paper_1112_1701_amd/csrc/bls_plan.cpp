// Host runtime of the BLS library: plan creation, validation, planning of
// (curve, period tile) work items, launch sequencing, reuse of plans and
// the C ABI of include/bls.h.
//
// The operation and its conventions are those stated in include/bls.h (Law
// et al. 2011, section 2.2.2, and the box-least-squares statistic it cites).
#include "bls_plan.h"

#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <new>
#include <numeric>
#include <thread>

namespace bls {
namespace {

// Message of the calling thread's last error without a plan (plan creation,
// the plan-free search); a fixed buffer, so that recording it allocates
// nothing.
thread_local char g_create_error[256];
std::atomic<long long> g_alloc_count{0};

uint64_t fnv1a(uint64_t h, const void *data, size_t bytes) {
  const unsigned char *p = static_cast<const unsigned char *>(data);
  for (size_t i = 0; i < bytes; ++i) {
    h ^= p[i];
    h *= 1099511628211ull;
  }
  return h;
}

template <class T>
uint64_t mix(uint64_t h, const T &v) {
  return fnv1a(h, &v, sizeof(T));
}

int cbits_of(int64_t n) {
  int b = 0;
  while (b < 63 && (int64_t(1) << b) <= n) ++b;
  return b;  // bit length of n
}

void free_dev(void *p) {
  if (p) (void)hipFree(p);
}

}  // namespace

hipError_t device_alloc(void **ptr, size_t bytes) {
  *ptr = nullptr;
  const long long k = ++g_alloc_count;
  const char *hook = getenv("BLS_DEBUG_FAIL_ALLOC");
  if (hook && *hook) {
    // "N": the N-th device allocation of the process fails; "all": every one
    // ("pinned" leaves device allocations alone and refuses the host-array
    // path's pinned staging instead).
    if (strcmp(hook, "all") == 0 || atoll(hook) == k) return hipErrorOutOfMemory;
  }
  return hipMalloc(ptr, bytes > 0 ? bytes : 1);
}

int set_error(bls_plan *p, int status, const std::string &msg) {
  if (p)
    p->last_error = msg;
  else
    snprintf(g_create_error, sizeof g_create_error, "%s", msg.c_str());
  return status;
}

int set_error_noplan(int status, const char *msg) {
  snprintf(g_create_error, sizeof g_create_error, "%s", msg);
  return status;
}

int hip_error(bls_plan *p, hipError_t e, const char *what) {
  std::string m = std::string(what) + ": " + hipGetErrorString(e);
  return set_error(p, e == hipErrorOutOfMemory ? BLS_ERR_NO_MEMORY : BLS_ERR_DEVICE, m);
}

int width_range(int32_t nbins, double qmin, double qmax, int32_t *kmin, int32_t *kmax) {
  if (nbins < 2 || !(qmin > 0.0) || !(qmax < 1.0) || !(qmin <= qmax)) return BLS_ERR_INVALID_ARG;
  long lo = lround(qmin * (double)nbins);
  long hi = lround(qmax * (double)nbins);
  if (lo < 1) lo = 1;
  if (hi > nbins - 1) hi = nbins - 1;
  if (kmin) *kmin = (int32_t)lo;
  if (kmax) *kmax = (int32_t)hi;
  return lo <= hi ? BLS_OK : BLS_ERR_INVALID_ARG;
}

namespace {

// Cycles the scan's 64-bit LDS reads take for the first rounds of lane tasks
// of one workgroup when consecutive periods' planes are S float2 apart.  The
// LDS serves such reads 16 lanes at a time from 32 banks of 4 bytes: a group
// of 16 lanes takes as many cycles as the busiest bank has accesses.  Lane
// task q is (start bin, period) = divmod(q, tile); every lane reads at the
// same offset m past its own start, which moves all banks alike, so m = 0.
// Both banks of a read are an even one and the next, so pairs of them are
// counted.
int scan_read_cycles(int S, int tile, int nbins) {
  const int tasks = std::min(4 * kBlock, nbins * tile);
  int cycles = 0, t = 0, pair = 0;
  for (int q = 0; q < tasks; q += 16) {
    uint8_t count[16] = {0};
    int worst = 0;
    for (int l = q; l < std::min(q + 16, tasks); ++l) {
      worst = std::max<int>(worst, ++count[pair & 15]);
      const bool next = ++t == tile;  // the next start bin
      pair += next ? 1 - (tile - 1) * S : S;
      t = next ? 0 : t;
    }
    cycles += worst;
  }
  return cycles;
}

}  // namespace

int hist_words(int nbins, int kmax) {
  // widths above nbins / 2 are scanned through their complement, so no
  // read reaches more than min(kmax, nbins / 2) - 1 bins past the end
  return nbins + std::max(std::min(kmax, nbins / 2) - 1, 1);
}

// Banks depend on the stride mod 16 and on no start bin past the first rounds',
// so the padding does too.  It is kept where its key falls in a fixed table,
// without a lock or heap use: found anew it takes 33 us (59 equal curves in a
// call without a plan, which kept none and tried up to three tiles each, 3.1
// ms; 101 curves of 101 bin counts whose 16 costs each did not fit a table of
// 4096, 0.55).
int hist_stride(int nbins, int kmax, int tile, bool weighted) {
  constexpr int kBits = 14;
  static std::atomic<uint32_t> kept[1 << kBits];  // key << 4 | padding
  const int hb = hist_words(nbins, kmax);
  const int nb = std::min(nbins, 4 * kBlock);
  const uint32_t key = (uint32_t)nb << 11 | (uint32_t)(tile - 1) << 5 | (uint32_t)(hb & 15) << 1 |
                       (weighted ? 1u : 0u);
  static_assert(kTileMax <= 64 && 4 * kBlock < 1 << 17, "fields of the key");
  std::atomic<uint32_t> &place = kept[(key * 0x9E3779B1u) >> (32 - kBits)];
  const uint32_t k = place.load(std::memory_order_relaxed);
  if (k >> 4 == key) return hb + (int)(k & 15);
  const int wpb = weighted ? 2 : 1;  // the scan reads the first plane of wpb
  int best = 0, best_cost = 0;
  for (int pad = 0; pad < 16; ++pad) {
    const int c = scan_read_cycles(((hb + pad) * wpb) & 15, tile, nb);
    if (pad == 0 || c < best_cost) {
      best = pad;
      best_cost = c;
    }
  }
  place.store(key << 4 | (uint32_t)best, std::memory_order_relaxed);
  return hb + best;
}

void fit_tile(int nbins, int kmax, int64_t nperiods, int lds_budget, int tile_cap,
              bool weighted, int *tile, int *stride) {
  const int wpb = weighted ? 2 : 1;
  int T = std::max(1, lds_budget / (hist_words(nbins, kmax) * 8 * wpb));
  T = std::min(T, std::min(tile_cap, kTileMax));
  T = (int)std::min<int64_t>(T, std::max<int64_t>(nperiods, 1));
  T = std::max(T, 1);
  int hs = hist_stride(nbins, kmax, T, weighted);
  while (T > 1 && T * hs * 8 * wpb > lds_budget) {
    --T;
    hs = hist_stride(nbins, kmax, T, weighted);
  }
  *tile = T;
  *stride = hs;
}

namespace {
// Message sink of validate_batch_into: a caller-owned character buffer.
struct ErrBuf {
  char *buf;
  size_t len;
  ErrBuf &operator=(const char *m) {
    if (buf && len) snprintf(buf, len, "%s", m);
    return *this;
  }
};
}  // namespace

// Block size: odd (the lanes' strides then spread over the LDS banks), so
// that r = 1 .. 4 waves-full of blocks cover the bins, r by the estimated
// cost: r rounds of pair tests per offset, and the boxes of the pairs that
// pass (about 25 and one per 22 bins of them on noise), a lane per start.
bool block_geometry(int nbins, int kmin, int kmax, BlockGeom *out) {
  if (2 * kmax > nbins || kmin > kmax) return false;
  double best = 0.0;
  for (int r = 1; r <= kMaxBlocks / 64; ++r) {
    BlockGeom g;
    g.bsize = (nbins + 64 * r - 1) / (64 * r) | 1;
    g.nblocks = (nbins + g.bsize - 1) / g.bsize;
    const int pad = g.nblocks * g.bsize - nbins;
    g.omin = kmin >= g.bsize ? kmin / g.bsize : 0;  // least o with o s + s - 1 >= kmin
    if (g.omin * g.bsize + g.bsize - 1 < kmin) ++g.omin;
    g.omax = (kmax + g.bsize - 1 + pad) / g.bsize;
    g.magic = ((1 << 20) + g.bsize - 1) / g.bsize;
    if (g.omax + 1 >= g.nblocks || g.omax > 255 || g.bsize > 64) continue;
    const int rounds = (g.nblocks + 63) / 64;
    const double pairs = 25.0 + nbins / 22.0;
    const double cost = rounds * (g.omax + 1) * 35.0 +
                        ceil(pairs * g.bsize / 64.0) * (20.0 + 13.0 * g.bsize) +
                        rounds * g.bsize * 25.0;
    if (best == 0.0 || cost < best) {
      best = cost;
      *out = g;
    }
  }
  return best > 0.0;
}

// Periods per work item of the block search and the workgroups that share a
// CU: as many periods in hand per CU as its LDS allows (a wave works on one),
// and of equal choices the largest tile with at least four workgroups per CU
// (they load the points for more periods at once), else the smallest tile.
// One-period-per-wave tiles also beat larger ones (uniform batch, 300 bins:
// tiles of 1, 2, 3, 4, 8 took 14.2, 8.6, 7.0, 6.1, 6.4 ms; 1000 bins, 600
// points: 8.3, 5.6, 5.0, 4.9 ms for 1 to 4; 2000 bins: 3.4, 3.8, 4.0, 6.1).
int block_tile(int nbins, int kmax, bool weighted, int max_lds, const BlockGeom &g, int *groups) {
  const int cap = weighted ? 5 : 6;  // workgroups per CU that the registers allow
  int best = 0, best_periods = 0, best_groups = 0;
  for (int T = 1; T <= 4; ++T) {
    const int bytes = block_tile_bytes(T, nbins, kmax, weighted, g) + kBlockStaticLds;
    const int w = std::min(cap, max_lds / bytes);
    if (w < 1) break;
    const int periods = T * w;
    if (periods > best_periods || (periods == best_periods && w >= 4)) {
      best = T;
      best_periods = periods;
      best_groups = w;
    }
  }
  if (groups) *groups = best_groups;
  return best;
}

// Whether the block search is the faster kernel for a batch, in instructions
// per period after the fold, which both share.  Scoring every box: a lane per
// start bin, three quarters as many again for weights, and twice that where a
// box that passes the screen has its points counted (weighted, a minimum of two
// or more); 0.8 to 0.9 of it where the call's tiles are tuned or let eight (six)
// workgroups share a CU (untuned_lds_budget).  The block search: its parts for
// the curve's geometry, 1.4 times that for weights, more where the LDS holds
// fewer than 20 periods per CU (its root: with the power 0.8 that calls of up to
// 1000 bins had suggested, calls of 1000 to 4096 lost 10% and up to a factor of
// seven).  The constants are from both kernels' times over some 9000 calls of
// noise, 1 to 200 curves, 100 to 60000 periods.  On 3042 others, percent above
// the faster kernel of each call by the choice, by blocks always and by blocks
// never: 140 to 50000 points, 100 to 1000 bins, unit weights 4.5, 20 and 18,
// weighted 1.1, 36 and 4, with a minimum of three 3.0, 27 and 25; 1000 to 4096
// bins 4.3, 3 and 85, 4.0, 10 and 45, 1.5, 3 and 253.
//
// A curve of few points for its bins has boxes that tie over many start bins,
// each of which is scored: up to several times the other kernel's time, in
// proportion to the bins per point (weighted curves only with a minimum count
// that hardly a box reaches; where boxes do, the other kernel's counting of their
// points costs more).  3 to 120 points, 150 to 3500 bins: unit weights 1.7, 85 and
// 8 percent, weighted 11, 11 and 91, with a minimum of three 5.3, 41 and 90; 4 x
// 4510 periods x 1393 bins, 0.024 to 0.16, of 6, 10, 20 and 40 points 1.46 / 2.70
// ms, 1.33 / 1.75, 1.13 / 0.94 and 0.95 / 0.46; weighted with a minimum of three,
// 132 x 244 x 1740, 0.015 to 0.036, of 6 and 30 points 6.1 / 13.4 and 6.5 / 1.5.
//
// The rule sees sizes and not the data, on which the block search's time
// depends more than the other's: narrow boxes and weights over four decades
// (105 x 500 points x 192 periods x 2000 bins, 0.0038 to 0.046) 1.03 / 1.76 ms
// where weights within a factor of four take 0.95 / 0.88; periods beyond
// the data with wide boxes (39 x 215 x 62 x 2235, 0.046 to 0.35, periods to 20 d
// in 10 d) 0.80 / 2.6 where 60 d take 0.79 / 0.49; dips alone beside rare
// points far above them (1 x 1214 x 19830 x 743, 0.003 to 0.047, 0.5% of the
// points 500 sigma up) 0.24 / 0.36 where noise takes 0.20 / 0.18.
namespace {
double every_box_cost(const CurveShape &s, bool weighted, bool counts, bool eight) {
  const double instr = s.nbins / 64.0 * (2.0 * s.kmin + 7.0 * (s.kmax - s.kmin + 1) + 30.0);
  return instr * (!weighted ? (eight ? 0.9 : 1.0) : counts ? 3.0 : eight ? 1.25 : 1.55);
}
double block_cost(const CurveShape &s, bool weighted, int counts, const BlockGeom &g,
                  int periods_per_cu, double every) {
  const int rounds = (g.nblocks + 63) / 64, per = 64 / g.bsize;
  const double batches = ceil((20.0 + s.nbins / 25.0) / per);
  const double instr = 330.0 + rounds * (60.0 + 24.0 * g.bsize + 27.0 * (g.omax - g.omin + 1)) +
                       batches * (32.0 + 13.5 * g.bsize);
  const bool empty = counts > 1 && 10.0 * s.n * s.kmax < (double)counts * s.nbins;
  const double ties = (!weighted ? 0.012 : empty ? 0.01 : 0.0) * s.nbins / (double)s.n;
  return instr * (weighted ? 1.4 : 1.0) * std::max(1.0, sqrt(20.0 / periods_per_cu)) +
         ties * every;
}
}  // namespace

bool block_batch(const CurveShape *shapes, int n, bool weighted, int min_in_points, bool tuned,
                 int num_cus, int max_lds) {
  const char *e = getenv("BLS_BLOCK_SEARCH");  // 0: never, 1: wherever it can run
  if (e && atoi(e) == 0) return false;
  double every = 0.0, block = 0.0;
  int64_t periods = 0;
  for (int c = 0; c < n; ++c) periods += shapes[c].nperiods;
  for (int c = 0; c < n; ++c) {
    const CurveShape &s = shapes[c];
    BlockGeom g;
    if (!block_geometry(s.nbins, s.kmin, s.kmax, &g)) return false;
    int groups = 0;
    const int T = block_tile(s.nbins, s.kmax, weighted, max_lds, g, &groups);
    if (T < 1) return false;
    const bool eight = tuned || untuned_lds_budget(s, periods, weighted, num_cus) <
                                    default_tiles(weighted).lds_budget;
    const double boxes = every_box_cost(s, weighted, min_in_points > 1, eight);
    every += (double)s.nperiods * boxes;
    block += (double)s.nperiods * block_cost(s, weighted, min_in_points, g, T * groups, boxes);
  }
  // Fewer periods than seven waves per CU: a period takes a wave 25 us or more,
  // and the four of a workgroup less (461 bins, 1497 periods 44 / 35 us; 400
  // bins, 2000 periods 43 / 52).
  if (e == nullptr && periods < 7 * (int64_t)num_cus) return false;
  return e != nullptr || block < every;
}

// LDS budget of the block search for a batch whose typical curve is `rep`:
// its best tile's share of a CU, so that larger curves take smaller tiles
// and the launch keeps that tile's workgroups.
int block_lds_budget(const CurveShape &rep, bool weighted, int max_lds) {
  BlockGeom g;
  int groups = 1;
  if (!block_geometry(rep.nbins, rep.kmin, rep.kmax, &g) ||
      block_tile(rep.nbins, rep.kmax, weighted, max_lds, g, &groups) < 1)
    return max_lds - kBlockStaticLds;
  return max_lds / groups - kBlockStaticLds;
}

void fit_block_tile(int nbins, int kmin, int kmax, int64_t nperiods, int lds_budget, int tile_cap,
                    bool weighted, int *tile, int *stride, BlockGeom *g) {
  block_geometry(nbins, kmin, kmax, g);
  // at most one period per wave (block_tile)
  int T = (int)std::min<int64_t>(std::min(tile_cap, 4), std::max<int64_t>(nperiods, 1));
  while (T > 1 && block_tile_bytes(T, nbins, kmax, weighted, *g) > lds_budget) --T;
  *tile = std::max(T, 1);
  *stride = block_plane_words(nbins, kmax, *g);
}

void set_block_layout(CurveDesc &d, const BlockGeom &g) {
  d.bsize = g.bsize;
  d.nblocks = g.nblocks;
  d.omin = g.omin;
  d.omax = g.omax;
  d.bmagic = g.magic;
  d.scr_offset = (d.tile * d.hstride * 8 * (d.weighted ? 2 : 1) + 15) & ~15;
  d.scr_bytes = block_scratch_bytes(d.nbins, g);
}

void LdsLayout::add(const CurveDesc &d, bool block) {
  bytes = std::max(bytes, block ? d.scr_offset + std::min(d.tile, 4) * d.scr_bytes
                                : d.tile * d.hstride * 8 * (d.weighted ? 2 : 1));
}

void fill_curve_desc(const CurveShape &s, bool weighted, const TileChoice &tc,
                     bool check_periods, bool block, CurveDesc &d) {
  memset(&d, 0, sizeof d);
  d.n_off = s.n_off;
  d.n = s.n;
  d.p_off = s.p_off;
  d.r_off = s.r_off;
  d.nperiods = s.nperiods;
  d.nbins = s.nbins;
  d.kmin = s.kmin;
  d.kmax = s.kmax;
  const int cb = cbits_of(s.n);
  d.shift = 64 - cb;
  d.qbits = std::min(kQBitsMax, 63 - 2 * cb);
  d.weighted = weighted ? 1 : 0;
  d.check_periods = check_periods ? 1 : 0;
  // bins, then the clamp word / wrap-around copy, per period and plane,
  // padded against LDS bank conflicts, as the kernel lays them out
  int T = 1, hs = 0;
  BlockGeom g;
  if (block)
    fit_block_tile(s.nbins, s.kmin, s.kmax, s.nperiods, tc.lds_budget, tc.tile_cap, weighted, &T,
                   &hs, &g);
  else
    fit_tile(s.nbins, s.kmax, s.nperiods, tc.lds_budget, tc.tile_cap, weighted, &T, &hs);
  d.tile = T;
  d.hstride = hs;
  if (block) set_block_layout(d, g);
}

int validate_batch_into(const bls_plan_config &cfg, const bls_batch &b, bool check_data,
                        CurveShape *shapes, int shapes_cap, char *err_buf, size_t err_len,
                        bool binned) {
  ErrBuf err{err_buf, err_len};
  char msg[256];
  if (b.ncurves < 1 || b.n_off == nullptr || b.times == nullptr || b.flux == nullptr ||
      b.periods == nullptr) {
    err = "batch needs ncurves >= 1 and non-NULL n_off, times, flux, periods";
    return BLS_ERR_INVALID_ARG;
  }
  if (b.ncurves > cfg.max_curves) {
    snprintf(msg, sizeof msg, "%d curves exceed the plan's max_curves %d", b.ncurves,
             cfg.max_curves);
    err = msg;
    return BLS_ERR_CAPACITY;
  }
  if (b.n_off[0] != 0) {
    err = "n_off[0] must be 0";
    return BLS_ERR_INVALID_ARG;
  }
  if (b.p_off == nullptr && b.nperiods_shared < 1) {
    err = "shared period grid needs nperiods_shared >= 1";
    return BLS_ERR_INVALID_ARG;
  }
  if (b.p_off != nullptr && b.p_off[0] != 0) {
    err = "p_off[0] must be 0";
    return BLS_ERR_INVALID_ARG;
  }
  if (shapes_cap < b.ncurves) {
    err = "shape buffer smaller than the batch";
    return BLS_ERR_CAPACITY;
  }
  int64_t total_results = 0;
  for (int c = 0; c < b.ncurves; ++c) {
    CurveShape &s = shapes[c];
    s.n_off = b.n_off[c];
    s.n = b.n_off[c + 1] - b.n_off[c];
    if (s.n < 2) {
      snprintf(msg, sizeof msg, "curve %d has %lld points (need >= 2)", c, (long long)s.n);
      err = msg;
      return BLS_ERR_INVALID_ARG;
    }
    if (s.n > (int64_t(1) << 24)) {
      snprintf(msg, sizeof msg, "curve %d has %lld points (at most 2^24)", c, (long long)s.n);
      err = msg;
      return BLS_ERR_CAPACITY;
    }
    int64_t np;
    if (b.p_off) {
      s.p_off = b.p_off[c];
      np = b.p_off[c + 1] - b.p_off[c];
      s.r_off = s.p_off;
    } else {
      s.p_off = 0;
      np = b.nperiods_shared;
      s.r_off = (int64_t)c * b.nperiods_shared;
    }
    if (np < 1 || np > INT32_MAX) {
      snprintf(msg, sizeof msg, "curve %d has %lld trial periods", c, (long long)np);
      err = msg;
      return BLS_ERR_INVALID_ARG;
    }
    s.nperiods = (int32_t)np;
    total_results += np;
    const double qmin = b.qmin ? b.qmin[c] : b.qmin_all;
    const double qmax = b.qmax ? b.qmax[c] : b.qmax_all;
    if (!binned) {
      s.nbins = 0;
      s.kmin = s.kmax = 0;
      if (!(qmin > 0.0) || !(qmax < 1.0) || !(qmin <= qmax)) {
        snprintf(msg, sizeof msg, "curve %d: bad duty-cycle range [%g, %g]", c, qmin, qmax);
        err = msg;
        return BLS_ERR_INVALID_ARG;
      }
      if (s.n > kUnbinnedMaxPointsGlobal) {
        snprintf(msg, sizeof msg, "curve %d has %lld points (the unbinned search takes at most %d)",
                 c, (long long)s.n, kUnbinnedMaxPointsGlobal);
        err = msg;
        return BLS_ERR_CAPACITY;
      }
      continue;
    }
    s.nbins = b.nbins ? b.nbins[c] : b.nbins_all;
    if (s.nbins < 2) {
      snprintf(msg, sizeof msg, "curve %d: nbins %d < 2", c, s.nbins);
      err = msg;
      return BLS_ERR_INVALID_ARG;
    }
    if (s.nbins > cfg.max_nbins) {
      snprintf(msg, sizeof msg, "curve %d: nbins %d exceeds max_nbins %d", c, s.nbins,
               cfg.max_nbins);
      err = msg;
      return BLS_ERR_CAPACITY;
    }
    if (width_range(s.nbins, qmin, qmax, &s.kmin, &s.kmax) != BLS_OK) {
      snprintf(msg, sizeof msg, "curve %d: bad duty-cycle range [%g, %g] for %d bins", c, qmin,
               qmax, s.nbins);
      err = msg;
      return BLS_ERR_INVALID_ARG;
    }
  }
  const int64_t total_points = b.n_off[b.ncurves];
  if (total_points > cfg.max_points) {
    snprintf(msg, sizeof msg, "%lld points exceed the plan's max_points %lld",
             (long long)total_points, (long long)cfg.max_points);
    err = msg;
    return BLS_ERR_CAPACITY;
  }
  if (total_results > cfg.max_periods) {
    snprintf(msg, sizeof msg, "%lld results exceed the plan's max_periods %lld",
             (long long)total_results, (long long)cfg.max_periods);
    err = msg;
    return BLS_ERR_CAPACITY;
  }
  if (!check_data) return BLS_OK;

  // Host data: periods, then points (zero-weight points are dropped first).
  const int64_t nper_total = b.p_off ? b.p_off[b.ncurves] : b.nperiods_shared;
  for (int64_t i = 0; i < nper_total; ++i) {
    const double P = b.periods[i];
    if (!isfinite(P) || !(P > 0.0)) {
      snprintf(msg, sizeof msg, "trial period %lld is %g (must be finite and > 0)",
               (long long)i, P);
      err = msg;
      return BLS_ERR_INVALID_ARG;
    }
  }
  for (int c = 0; c < b.ncurves; ++c) {
    const CurveShape &s = shapes[c];
    int64_t kept = 0;
    double W = 0.0;
    for (int64_t i = s.n_off; i < s.n_off + s.n; ++i) {
      const double w = b.weights ? b.weights[i] : 1.0;
      if (!(w >= 0.0) || isinf(w)) {
        snprintf(msg, sizeof msg, "curve %d point %lld: weight %g (must be finite, >= 0)", c,
                 (long long)(i - s.n_off), w);
        err = msg;
        return BLS_ERR_INVALID_ARG;
      }
      if (w == 0.0) continue;
      if (!isfinite(b.times[i]) || !isfinite(b.flux[i])) {
        snprintf(msg, sizeof msg, "curve %d point %lld: non-finite time or flux", c,
                 (long long)(i - s.n_off));
        err = msg;
        return BLS_ERR_INVALID_ARG;
      }
      ++kept;
      W += w;
    }
    if (kept < 2 || !(W > 0.0) || !isfinite(W)) {
      snprintf(msg, sizeof msg, "curve %d: %lld points with positive weight (need >= 2)", c,
               (long long)kept);
      err = msg;
      return BLS_ERR_INVALID_ARG;
    }
  }
  return BLS_OK;
}

int validate_batch(const bls_plan_config &cfg, const bls_batch &b, bool check_data,
                   std::vector<CurveShape> &shapes, std::string &err, bool binned) {
  if (b.ncurves >= 1 && b.ncurves <= cfg.max_curves) shapes.resize(b.ncurves);
  char buf[256] = "";
  const int st = validate_batch_into(cfg, b, check_data, shapes.data(), (int)shapes.size(), buf,
                                     sizeof buf, binned);
  if (st != BLS_OK) err = buf;
  return st;
}

// Segments of the batch, grouped by work partition.  Curves go to the
// partitions round-robin in descending cost, so each partition (one per XCD:
// the device dispatches workgroups to its XCDs round-robin) gets a similar
// share, largest first, and every curve's period tiles stay in one XCD's L2:
// the curve is fetched by one L2 and adjacent tiles' partial result lines
// merge there before write-back.
void layout_partitions(bls_plan *p, const std::vector<double> &cost,
                       const std::vector<int64_t> &items_of, PlannedBatch &out) {
  const int nc = (int)cost.size();
  p->order.resize(nc);
  std::iota(p->order.begin(), p->order.end(), 0);
  std::stable_sort(p->order.begin(), p->order.end(),
                   [&](int a, int b) { return cost[a] > cost[b]; });
  // Few curves (fewer than two per XCD) share one partition: splitting them
  // would only make most workgroups probe empty partitions first.
  const int np =
      (p->num_cus > 0 && p->num_cus % kMaxParts == 0 && nc >= 2 * kMaxParts) ? kMaxParts : 1;
  int64_t items = 0;
  int s = 0;
  for (int x = 0; x < np; ++x) {
    out.part_begin[x] = items;
    for (int k = x; k < nc; k += np) {
      const int c = p->order[k];
      p->h_seg_start[s] = items;
      p->h_seg_curve[s] = c;
      p->h_seg_tile0[s] = 0;
      items += items_of[c];
      ++s;
    }
  }
  for (int x = np; x <= kMaxParts; ++x) out.part_begin[x] = items;
  p->h_seg_start[nc] = items;
  out.nparts = np;
  out.nseg = nc;
  out.nitems = items;
}

int item_group(const bls_plan *p, const std::vector<CurveShape> &shapes) {
  if (const char *e = getenv("BLS_ITEM_GROUP")) {
    const int g = atoi(e);  // 0: one tile per item; kGroupMax: groups
    return g == kGroupMax ? kGroupMax : 0;
  }
  int64_t periods = 0;
  for (const CurveShape &s : shapes) periods += s.nperiods;
  // at least four groups per workgroup of a full grid (eight per CU)
  const int64_t want = (int64_t)kGroupMax * 4 * 8 * std::max(p->num_cus, 1);
  return periods >= want ? kGroupMax : 0;
}

int plan_batch(bls_plan *p, const std::vector<CurveShape> &shapes, bool weighted,
               const TileChoice &tc, PlannedBatch &out) {
  const int nc = (int)shapes.size();
  // The descriptors and the places of the segments change from here on, also
  // where planning fails: the last search's plan goes stale.
  p->replay_valid = false;
  // queued copies may still read the pinned descriptors
  const int ws = desc_wait(p);
  if (ws != BLS_OK) return ws;
  place_desc(p, nc);
  out = PlannedBatch{};
  out.ncurves = nc;
  out.weighted = weighted;

  // Work items: groups of kGroupMax consecutive periods, aligned to whole
  // result lines and written out together, when the batch has enough of
  // them for several items per resident workgroup; one tile each otherwise.
  const int G = item_group(p, shapes);
  // Per-curve tile: as many periods as fit the LDS budget, at least one.
  const bool block = tc.block;
  LdsLayout lds;
  std::vector<double> item_cost(nc);
  for (int c = 0; c < nc; ++c) {
    const CurveShape &s = shapes[c];
    CurveDesc &d = p->h_curves[c];
    // each distinct period range is checked once (a shared grid by curve 0)
    fill_curve_desc(s, weighted, tc, c == 0 || s.p_off != shapes[0].p_off, block, d);
    const int T = d.tile;
    if (G > 0) {
      d.group = G;
      d.galign = (int32_t)(s.r_off % G);
    }
    lds.add(d, block);
    const double nw = (double)(s.kmax - s.kmin + 1);
    item_cost[c] = (double)(G > 0 ? G : T) * ((double)s.n + 1.6 * (double)s.nbins * nw);
    out.total_points += s.n;
    out.total_results += s.nperiods;
    out.trial_points += (double)s.n * (double)s.nperiods;
    out.box_evals += (double)s.nbins * nw * (double)s.nperiods;
  }
  const int hist_bytes = lds.total();
  if (hist_bytes > p->max_lds - 1024) {
    return set_error(p, BLS_ERR_CAPACITY,
                     "one period's histogram needs " + std::to_string(hist_bytes) +
                         " bytes of LDS, more than a workgroup has");
  }

  // Largest items first within each XCD partition, so the persistent grid
  // drains evenly.
  std::vector<int64_t> items_of(nc);
  for (int c = 0; c < nc; ++c) {
    const CurveDesc &d = p->h_curves[c];
    items_of[c] = d.group > 0 ? ((int64_t)d.nperiods + d.galign + d.group - 1) / d.group
                              : (d.nperiods + d.tile - 1) / d.tile;
  }
  layout_partitions(p, item_cost, items_of, out);
  const int64_t items = out.nitems;
  out.hist_bytes = hist_bytes;
  out.block = block;

  int per_cu = 0;
  hipError_t e = (hipError_t)search_blocks_per_cu(weighted, (p->cfg.flags & BLS_DIP_ONLY) != 0, block,
                                                  hist_bytes, &per_cu);
  if (e != hipSuccess) return hip_error(p, e, "occupancy query");
  if (per_cu < 1) return set_error(p, BLS_ERR_CAPACITY, "search kernel does not fit a CU");
  if (tc.occupancy > 0) per_cu = std::min(per_cu, tc.occupancy);
  const int64_t grid = std::min<int64_t>(items, (int64_t)p->num_cus * per_cu);
  out.grid = (int32_t)std::max<int64_t>(grid, 1);
  return BLS_OK;
}

int desc_wait(bls_plan *p) {
  if (!p->desc_pending) return BLS_OK;
  hipError_t e = hipEventSynchronize(p->ev_desc);
  if (e != hipSuccess) return hip_error(p, e, "wait for descriptor uploads");
  p->desc_pending = false;
  return BLS_OK;
}

// One block holds a call's descriptors: the curves', then their segments'
// (first items, curves, first tiles), so that one copy uploads them.
size_t desc_bytes(int nc) {
  static_assert(sizeof(CurveDesc) % 8 == 0, "the segments' 64-bit items follow the curves");
  return sizeof(CurveDesc) * nc + 8 * ((size_t)nc + 1) + 4 * (size_t)nc * 2;
}

void place_desc(bls_plan *p, int nc) {
  for (int dev = 0; dev < 2; ++dev) {
    unsigned char *b = reinterpret_cast<unsigned char *>(dev ? p->d_curves : p->h_curves);
    int64_t *start = reinterpret_cast<int64_t *>(b + sizeof(CurveDesc) * nc);
    int32_t *curve = reinterpret_cast<int32_t *>(start + nc + 1);
    (dev ? p->d_seg_start : p->h_seg_start) = start;
    (dev ? p->d_seg_curve : p->h_seg_curve) = curve;
    (dev ? p->d_seg_tile0 : p->h_seg_tile0) = curve + nc;
  }
}

int desc_mark(bls_plan *p) {
  hipError_t e = hipEventRecord(p->ev_desc, p->stream);
  if (e != hipSuccess) return hip_error(p, e, "event record");
  p->desc_pending = true;
  return BLS_OK;
}

int ring_begin(bls_plan *p) {
  const int slot = (int)(p->k_recorded % bls_plan::kTimeRing);
  hipError_t e = hipEventRecord(p->ev_k0[slot], p->stream);
  return e == hipSuccess ? BLS_OK : hip_error(p, e, "event record");
}

int ring_end(bls_plan *p) {
  const int slot = (int)(p->k_recorded % bls_plan::kTimeRing);
  hipError_t e = hipEventRecord(p->ev_k1[slot], p->stream);
  if (e != hipSuccess) return hip_error(p, e, "event record");
  ++p->k_recorded;
  return BLS_OK;
}

int enqueue_pre(bls_plan *p, const PlannedBatch &pb, const double *t, const double *x,
                const double *w, const double *periods, int64_t *best, bool upload) {
  hipStream_t st = p->stream;
  hipError_t e;
  const int nc = pb.ncurves;
  if (upload) {
    e = hipMemcpyAsync(p->d_curves, p->h_curves, desc_bytes(nc), hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return hip_error(p, e, "upload descriptors");
  }

  PrepArgs pa;
  pa.curves = p->d_curves;
  pa.periods = periods;
  pa.ncurves = nc;
  pa.t = t;
  pa.x = x;
  pa.w = w;
  pa.dt = p->d_dt;
  pa.q = p->d_q;
  pa.qw = p->d_qw;
  pa.counter = p->d_counter;
  pa.keys = reinterpret_cast<unsigned long long *>(best);
  pa.status = p->status_dev;
  e = (hipError_t)launch_prep(pa, st);
  if (e != hipSuccess) return hip_error(p, e, "launch prep");
  return BLS_OK;
}

int enqueue_kernel(bls_plan *p, const PlannedBatch &pb, const double *periods, float *sr,
                   float *depth, int32_t *js, int32_t *ks, int64_t *best, bool unbinned) {
  SearchArgs sa;
  sa.curves = p->d_curves;
  sa.periods = periods;
  sa.dt = p->d_dt;
  sa.q = p->d_q;
  sa.qw = pb.weighted ? p->d_qw : nullptr;
  sa.seg_start = p->d_seg_start;
  sa.seg_curve = p->d_seg_curve;
  sa.seg_tile0 = p->d_seg_tile0;
  sa.nseg = pb.nseg;
  sa.min_in_points = p->cfg.min_in_points;
  sa.nitems = pb.nitems;
  sa.counter = p->d_counter;
  sa.sr = sr;
  sa.depth = depth;
  sa.jstart = js;
  sa.kwidth = ks;
  sa.best_key = reinterpret_cast<unsigned long long *>(best);
  sa.hist_bytes = pb.hist_bytes;
  sa.block = pb.block ? 1 : 0;
  sa.ucap = pb.ucap;
  sa.uws = pb.uws;
  sa.uws_stride = pb.uws_stride;
  sa.fold_policy = 0;
  sa.seed_unit = 1;
  if (const char *fm = getenv("BLS_FOLD_MERGE")) sa.fold_policy = atoi(fm) == 1 ? 1 : 2;
  if (const char *su = getenv("BLS_SEED_UNIT")) sa.seed_unit = atoi(su) != 0 ? 1 : 0;
  sa.nparts = pb.nparts;
  for (int x = 0; x <= kMaxParts; ++x) sa.part_begin[x] = pb.part_begin[x];
  const bool dip = (p->cfg.flags & BLS_DIP_ONLY) != 0;
  hipError_t e = unbinned ? (hipError_t)launch_unbinned(sa, pb.weighted, dip, pb.grid, p->stream)
                          : (hipError_t)launch_search(sa, pb.weighted, dip, pb.grid, p->stream);
  if (e != hipSuccess) return hip_error(p, e, "launch search");
  return BLS_OK;
}

int enqueue_post(bls_plan *p, const PlannedBatch &pb, const int64_t *keys, int64_t *best) {
  hipError_t e = (hipError_t)launch_best_index(reinterpret_cast<const unsigned long long *>(keys),
                                               reinterpret_cast<unsigned long long *>(best),
                                               pb.ncurves, p->stream);
  if (e != hipSuccess) return hip_error(p, e, "launch best index");
  return BLS_OK;
}

int enqueue_search(bls_plan *p, const PlannedBatch &pb, const double *t, const double *x,
                   const double *w, const double *periods, float *sr, float *depth, int32_t *js,
                   int32_t *ks, int64_t *best, bool unbinned, bool upload, int64_t *keys) {
  if (!keys) keys = best;
  int st = enqueue_pre(p, pb, t, x, w, periods, keys, upload);
  if (st == BLS_OK && upload) st = desc_mark(p);
  if (st == BLS_OK) st = ring_begin(p);
  if (st == BLS_OK) st = enqueue_kernel(p, pb, periods, sr, depth, js, ks, keys, unbinned);
  if (st == BLS_OK) st = ring_end(p);
  if (st == BLS_OK) st = enqueue_post(p, pb, keys, best);
  return st;
}

TileChoice default_tiles(bool weighted) {
  TileChoice tc;
  // The same 32 KB for both paths: one-curve calls on uneven weighted curves
  // ran at 1.97e11 trial-period points/s with it, against 1.92e11 with 40 KB
  // and 1.94e11 with 24 KB.
  (void)weighted;
  tc.lds_budget = 32768;
  tc.tile_cap = kTileMax;
  tc.occupancy = 0;
  return tc;
}

// Calls with many periods per workgroup keep the chip full whatever the tile,
// and are fastest with the tile that lets eight unit-weight (or six weighted)
// workgroups share a CU; smaller calls gain more from fewer, larger items.
// Search kernel, 32 KB against 21 KB (weighted 25 KB): 192 curves x 2000
// points x 20000 periods x 300 bins 11.34 / 8.51 ms; 384 x 600 x 20000 x 300
// 20.4 / 14.6; 64 x 600 x 5000 x 300 1.04 / 0.87; 128 x 600 x 20000 x 200
// 4.56 / 3.55; weighted 64 x 250 x 12000 x 200 2.06 / 1.77, 64 x 2000 x 12000
// x 350 4.61 / 3.78; but 16 x 600 x 5000 x 300 0.371 / 0.399, weighted 16 x
// 2000 x 5000 x 200 0.403 / 0.442, and 64 x 2000 x 2000 x 500 0.638 / 0.660.
// Wide grids, whose tile would drop below four periods, keep 32 KB (weighted
// 166 x 1106 x 2787 x 402 took 3.46 ms with it, 3.63 with tiles of three).
int untuned_lds_budget(const CurveShape &rep, int64_t periods, bool weighted, int num_cus) {
  const int small = weighted ? 25000 : 21200, wide = default_tiles(weighted).lds_budget;
  if (periods < (int64_t)1024 * std::max(num_cus, 1)) return wide;
  return small / (hist_words(rep.nbins, rep.kmax) * 8 * (weighted ? 2 : 1)) >= 4 ? small : wide;
}

double last_kernel_ms(bls_plan *p) {
  if (p->k_recorded == 0) return 0.0;
  const int slot = (int)((p->k_recorded - 1) % bls_plan::kTimeRing);
  float ms = 0.f;
  if (hipEventElapsedTime(&ms, p->ev_k0[slot], p->ev_k1[slot]) != hipSuccess) return 0.0;
  return ms;
}

void fill_stats(bls_plan *p, const PlannedBatch &pb, bool replayed) {
  p->stats.trial_points = pb.trial_points;
  p->stats.box_evals = pb.box_evals;
  p->stats.work_items = pb.nitems;
  p->stats.grid = pb.grid;
  p->stats.block = kBlock;
  p->stats.lds_bytes = pb.hist_bytes;
  p->stats.graph_replayed = replayed ? 1 : 0;
}

// Elements of a result array in a block of them: whole lines.
static size_t result_stride(int64_t n) { return ((size_t)n + 31) & ~(size_t)31; }

int ensure_staging(bls_plan *p) {
  if (p->d_t) return BLS_OK;
  const size_t np = (size_t)p->cfg.max_points, nr = (size_t)p->cfg.max_periods,
               nc = (size_t)p->cfg.max_curves;
  // One block, for one copy; a call lays its inputs out compactly from the
  // block's start (host_search), the other users have them at the plan's
  // capacities.  The best keys follow on a line of their own.
  const size_t in = (3 * np + nr + 15) & ~(size_t)15;
  const hipError_t e = device_alloc((void **)&p->d_t, (in + nc) * 8);
  if (e != hipSuccess) {
    p->d_t = nullptr;
    return hip_error(p, e, "allocate host-path staging");
  }
  p->d_x = p->d_t + np;
  p->d_w = p->d_x + np;
  p->d_periods = p->d_w + np;
  p->d_best = reinterpret_cast<int64_t *>(p->d_t + in);
  return BLS_OK;
}

int ensure_result_staging(bls_plan *p) {
  if (p->d_sr) return BLS_OK;
  const size_t nrp = result_stride(p->cfg.max_periods);
  const hipError_t e = device_alloc((void **)&p->d_sr, nrp * 16);
  if (e != hipSuccess) {
    p->d_sr = nullptr;
    return hip_error(p, e, "allocate host-path staging");
  }
  p->d_depth = p->d_sr + nrp;
  p->d_j = reinterpret_cast<int32_t *>(p->d_depth + nrp);
  p->d_k = p->d_j + nrp;
  return BLS_OK;
}

// Waits for the stream; the curves' status is then in p->h_status.
int wait_for_status(bls_plan *p) {
  const hipError_t e = hipStreamSynchronize(p->stream);
  return e == hipSuccess ? BLS_OK : hip_error(p, e, "synchronize");
}

int check_device_status(bls_plan *p, int ncurves) {
  const int32_t *status = p->h_status;
  for (int c = 0; c < ncurves; ++c) {
    if (status[c] != kCurveOk) {
      char msg[160];
      snprintf(msg, sizeof msg, "curve %d: %s", c,
               status[c] == kCurveBadData
                   ? "non-finite time/flux of a kept point, or a negative/non-finite weight"
               : status[c] == kCurveBadPeriod
                   ? "a trial period is not finite and > 0"
                   : "fewer than two points with positive weight");
      return set_error(p, BLS_ERR_INVALID_ARG, msg);
    }
  }
  return BLS_OK;
}

// Per-curve validity flags of the last prep (1 where the curve's data or
// trial periods were invalid); the prep kernel writes them to host memory.
int device_status_flags(bls_plan *p, int ncurves, int32_t *bad) {
  const int st = wait_for_status(p);
  if (st != BLS_OK) return st;
  for (int c = 0; c < ncurves; ++c) bad[c] = p->h_status[c] != kCurveOk ? 1 : 0;
  return BLS_OK;
}

int ensure_detect_buffers(bls_plan *p) {
  if (p->d_detect_desc) return BLS_OK;
  hipError_t e;
  if ((e = device_alloc((void **)&p->d_detect_desc, sizeof(DetectDesc) * p->cfg.max_curves)) ||
      (e = device_alloc((void **)&p->d_detect_out, sizeof(bls_detection) * p->cfg.max_curves))) {
    if (p->d_detect_desc) (void)hipFree(p->d_detect_desc);
    p->d_detect_desc = nullptr;
    p->d_detect_out = nullptr;
    return hip_error(p, e, "allocate detection buffers");
  }
  return BLS_OK;
}

int enqueue_detect_shared(bls_plan *p, int ncurves, const double *periods, int64_t nperiods,
                          const float *sr, int max_peaks, double window, double threshold) {
  int st = ensure_detect_buffers(p);
  if (st != BLS_OK) return st;
  std::vector<DetectDesc> dd(ncurves);
  for (int c = 0; c < ncurves; ++c) {
    dd[c].p_off = 0;
    dd[c].r_off = (int64_t)c * nperiods;
    dd[c].nperiods = nperiods;
  }
  hipStream_t s = p->stream;
  // a synchronous upload: dd lives on this function's stack
  hipError_t e = hipMemcpyAsync(p->d_detect_desc, dd.data(), sizeof(DetectDesc) * ncurves,
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_error(p, e, "upload detection descriptors");
  DetectArgs a;
  a.desc = p->d_detect_desc;
  a.periods = periods;
  a.sr = sr;
  a.out = p->d_detect_out;
  a.ncurves = ncurves;
  a.max_peaks = max_peaks;
  a.window = window;
  a.threshold = threshold;
  if ((e = (hipError_t)launch_detect(a, s)) != hipSuccess) return hip_error(p, e, "launch detection");
  return BLS_OK;
}

int ensure_recovery_buffers(bls_plan *p) {
  if (p->d_inj) return BLS_OK;
  hipError_t e;
  if ((e = device_alloc((void **)&p->d_inj, 32 * (size_t)p->cfg.max_curves)) ||
      (e = device_alloc((void **)&p->d_inj_t0, sizeof(double)))) {
    if (p->d_inj) (void)hipFree(p->d_inj);
    p->d_inj = nullptr;
    p->d_inj_t0 = nullptr;
    return hip_error(p, e, "allocate injection buffers");
  }
  return BLS_OK;
}

}  // namespace bls

using namespace bls;

namespace {

// f(i0, i1) over [0, n) in contiguous pieces on up to 16 host threads, one
// piece per `grain` items at least (the calling thread takes the last).
template <class F>
void par_ranges(int64_t n, int64_t grain, F f) {
  const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
  const int64_t nt = std::max<int64_t>(
      1, std::min<int64_t>((int64_t)std::min(hw, 16u), n / std::max<int64_t>(grain, 1)));
  std::vector<std::thread> th;
  int64_t i0 = 0;
  for (int64_t t = 0; t + 1 < nt; ++t) {
    const int64_t i1 = n * (t + 1) / nt;
    try {
      th.emplace_back(f, i0, i1);
    } catch (...) {
      f(i0, i1);  // no thread: this one does the piece
    }
    i0 = i1;
  }
  f(i0, n);
  for (auto &x : th) x.join();
}

// Copy of `bytes` between host buffers on several threads (a single thread
// copies at a fraction of the memory bandwidth).
void par_copy(void *dst, const void *src, size_t bytes) {
  par_ranges((int64_t)bytes, int64_t(8) << 20, [&](int64_t i0, int64_t i1) {
    memcpy((char *)dst + i0, (const char *)src + i0, (size_t)(i1 - i0));
  });
}

// Pinned staging for the host API, sized once for the plan's limits: the
// inputs (times, flux, weights, periods) or the results (SR, depth, first
// and last bin, best index), whichever is larger.  False if pinned memory
// is not available (the host API then copies from pageable memory).
bool ensure_host_stage(bls_plan *p) {
  if (p->h_stage) return true;
  // BLS_DEBUG_FAIL_ALLOC=pinned: behave as if pinned memory were refused
  const char *hook = getenv("BLS_DEBUG_FAIL_ALLOC");
  if (hook && strcmp(hook, "pinned") == 0) return false;
  const size_t np = (size_t)p->cfg.max_points, nr = (size_t)p->cfg.max_periods,
               nc = (size_t)p->cfg.max_curves;
  const size_t in = 3 * np * 8 + nr * 8 + 256, res = 16 * result_stride((int64_t)nr) + nc * 8;
  const size_t bytes = std::max(in, res);
  if (hipHostMalloc((void **)&p->h_stage, bytes, 0) != hipSuccess) {
    p->h_stage = nullptr;
    return false;
  }
  p->h_stage_bytes = bytes;
  return true;
}

// Host-array search of a validated batch (shared by bls_search and
// bls_search_batch).
int host_search(bls_plan *p, const bls_batch &b, const std::vector<CurveShape> &shapes,
                const bls_results &out) {
  int st = ensure_staging(p);
  if (st != BLS_OK) return st;
  const bool weighted = b.weights != nullptr;
  TileChoice tc = choose_tiles(p, shapes, weighted);
  PlannedBatch pb;
  st = plan_batch(p, shapes, weighted, tc, pb);
  if (st != BLS_OK) return st;

  const int64_t npts = b.n_off[b.ncurves];
  const int64_t nper = b.p_off ? b.p_off[b.ncurves] : b.nperiods_shared;
  hipStream_t s = p->stream;
  hipError_t e;
  // Inputs through the pinned staging when there is one: a threaded copy
  // into it, then DMA (pageable copies run at a fraction of that rate).  The
  // previous call's copies from or into it ended with that call.
  const bool pinned = ensure_host_stage(p);
  if (!pinned && (st = ensure_result_staging(p)) != BLS_OK) return st;
  const double *src_t = b.times, *src_x = b.flux, *src_w = b.weights, *src_p = b.periods;
  if (pinned) {
    double *st = reinterpret_cast<double *>(p->h_stage);
    double *sx = st + npts, *sw = sx + npts, *sp = sw + (weighted ? npts : 0);
    par_copy(st, b.times, (size_t)npts * 8);
    par_copy(sx, b.flux, (size_t)npts * 8);
    if (weighted) par_copy(sw, b.weights, (size_t)npts * 8);
    par_copy(sp, b.periods, (size_t)nper * 8);
    src_t = st;
    src_x = sx;
    src_w = weighted ? sw : nullptr;
    src_p = sp;
  }
  if ((e = hipEventRecord(p->ev_begin, s)) != hipSuccess) return hip_error(p, e, "event");
  // on the device as in the staging: arrays one after the other
  double *d_t = p->d_t, *d_x = d_t + npts, *d_w = d_x + npts,
         *d_per = weighted ? d_w + npts : d_w;
  if (pinned) {
    if ((e = hipMemcpyAsync(d_t, src_t, (npts * (weighted ? 3 : 2) + nper) * 8,
                            hipMemcpyHostToDevice, s)) != hipSuccess)
      return hip_error(p, e, "upload inputs");
  } else if ((e = hipMemcpyAsync(d_t, src_t, npts * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
             (e = hipMemcpyAsync(d_x, src_x, npts * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
             (weighted && (e = hipMemcpyAsync(d_w, src_w, npts * 8, hipMemcpyHostToDevice, s)) !=
                              hipSuccess) ||
             (e = hipMemcpyAsync(d_per, src_p, nper * 8, hipMemcpyHostToDevice, s)) !=
                 hipSuccess) {
    return hip_error(p, e, "upload inputs");
  }
  const int64_t nres = pb.total_results;
  const size_t nrp = result_stride(nres);
  float *d_sr = p->d_sr;
  // With pinned staging the kernels write the results there themselves (the
  // inputs' upload from it has ended by then: same stream), and only the best
  // keys, which they update by atomics, stay in device memory.  A copy after
  // the search took, 5000 periods of one star 143 us a call / 132 so; 192 x 600
  // points x 20000 periods 15.8 / 14.9 ms; 64 x 250 x 12000 the same.
  if (pinned && (e = hipHostGetDevicePointer((void **)&d_sr, p->h_stage, 0)) != hipSuccess)
    return hip_error(p, e, "address of the results");
  float *d_depth = d_sr + nrp;
  int32_t *d_j = reinterpret_cast<int32_t *>(d_depth + nrp), *d_k = d_j + nrp;
  int64_t *d_best = pinned ? reinterpret_cast<int64_t *>(d_k + nrp) : p->d_best;
  st = enqueue_search(p, pb, d_t, d_x, weighted ? d_w : nullptr, d_per, d_sr, d_depth, d_j, d_k,
                      d_best, false, true, p->d_best);
  if (st != BLS_OK) return st;
  if ((e = hipEventRecord(p->ev_end, s)) != hipSuccess) return hip_error(p, e, "event");

  // Results in the pinned staging, else into pageable vectors.
  std::vector<float> v_sr, v_depth;
  std::vector<int32_t> v_js, v_ks;
  std::vector<int64_t> v_best;
  float *sr, *depth;
  int32_t *js, *ks;
  int64_t *best;
  if (pinned) {
    sr = reinterpret_cast<float *>(p->h_stage);
    depth = sr + nrp;
    js = reinterpret_cast<int32_t *>(depth + nrp);
    ks = js + nrp;
    best = reinterpret_cast<int64_t *>(ks + nrp);
  } else {
    v_sr.resize(nres);
    v_depth.resize(nres);
    v_js.resize(nres);
    v_ks.resize(nres);
    v_best.resize(b.ncurves);
    sr = v_sr.data();
    depth = v_depth.data();
    js = v_js.data();
    ks = v_ks.data();
    best = v_best.data();
  }
  if (!pinned &&
      ((e = hipMemcpyAsync(sr, d_sr, nres * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
       (e = hipMemcpyAsync(depth, d_depth, nres * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
       (e = hipMemcpyAsync(js, d_j, nres * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
       (e = hipMemcpyAsync(ks, d_k, nres * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
       (e = hipMemcpyAsync(best, d_best, b.ncurves * 8, hipMemcpyDeviceToHost, s)) != hipSuccess))
    return hip_error(p, e, "download results");
  st = wait_for_status(p);
  if (st == BLS_OK) st = check_device_status(p, b.ncurves);
  if (st != BLS_OK) return st;

  float ms = 0.f;
  p->stats.search_ms = last_kernel_ms(p);
  (void)hipEventElapsedTime(&ms, p->ev_begin, p->ev_end);
  p->stats.total_ms = ms;
  fill_stats(p, pb, false);

  // Results: (value, box) per period at r_off; phase and duration from j, k.
  // Up to 40 B are written per result: host threads take contiguous curve
  // ranges.
  par_ranges(b.ncurves, std::max<int64_t>(1, (int64_t)b.ncurves * (int64_t(1) << 20) /
                                                 std::max<int64_t>(nres, 1)),
             [&](int64_t c0, int64_t c1) {
    for (int64_t c = c0; c < c1; ++c) {
      const CurveShape &cs = shapes[c];
      const double *per = b.periods + cs.p_off;
      for (int32_t i = 0; i < cs.nperiods; ++i) {
        const int64_t r = cs.r_off + i;
        const bool none = ks[r] < 0;
        if (out.sr) out.sr[r] = (double)sr[r];
        if (out.depth) out.depth[r] = none ? NAN : (double)depth[r];
        if (out.jstart) out.jstart[r] = js[r];
        if (out.kwidth) out.kwidth[r] = ks[r];
        if (out.phase) out.phase[r] = none ? NAN : (double)js[r] / (double)cs.nbins;
        if (out.duration) out.duration[r] = none ? NAN : (double)ks[r] * per[i] / (double)cs.nbins;
      }
      if (out.best_index) out.best_index[c] = best[c];
    }
  });
  p->last = pb;
  return BLS_OK;
}

uint64_t batch_signature(const bls_plan *p, const bls_batch &b, const bls_device_results &o) {
  uint64_t h = 1469598103934665603ull;
  h = mix(h, b.ncurves);
  h = mix(h, b.times);
  h = mix(h, b.flux);
  h = mix(h, b.weights);
  h = mix(h, b.periods);
  h = mix(h, b.nperiods_shared);
  h = mix(h, b.nbins_all);
  h = mix(h, b.qmin_all);
  h = mix(h, b.qmax_all);
  h = fnv1a(h, b.n_off, sizeof(int64_t) * (b.ncurves + 1));
  if (b.p_off) h = fnv1a(h, b.p_off, sizeof(int64_t) * (b.ncurves + 1));
  if (b.nbins) h = fnv1a(h, b.nbins, sizeof(int32_t) * b.ncurves);
  if (b.qmin) h = fnv1a(h, b.qmin, sizeof(double) * b.ncurves);
  if (b.qmax) h = fnv1a(h, b.qmax, sizeof(double) * b.ncurves);
  h = mix(h, o.sr);
  h = mix(h, o.depth);
  h = mix(h, o.jstart);
  h = mix(h, o.kwidth);
  h = mix(h, o.best_index);
  h = mix(h, p->cfg.flags);
  h = mix(h, p->cfg.min_in_points);
  return h;
}

}  // namespace

extern "C" {

void bls_plan_config_init(bls_plan_config *cfg) {
  if (!cfg) return;
  memset(cfg, 0, sizeof *cfg);
  cfg->device = 0;
  cfg->max_curves = 1;
  cfg->max_points = int64_t(1) << 20;
  cfg->max_periods = int64_t(1) << 20;
  cfg->max_nbins = BLS_MAX_NBINS;
  cfg->min_in_points = 1;
  cfg->flags = 0;
  cfg->hip_stream = nullptr;
}

int bls_plan_create(bls_plan **out, const bls_plan_config *cfg_in) {
  if (!out) return set_error(nullptr, BLS_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  bls_plan_config cfg;
  if (cfg_in)
    cfg = *cfg_in;
  else
    bls_plan_config_init(&cfg);
  if (cfg.min_in_points <= 0) cfg.min_in_points = 1;
  if (cfg.max_curves < 1 || cfg.max_points < 2 || cfg.max_periods < 1 || cfg.max_nbins < 2 ||
      cfg.max_nbins > BLS_MAX_NBINS || cfg.max_curves > (1 << 30))
    return set_error(nullptr, BLS_ERR_INVALID_ARG, "bad plan capacities");
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess || ndev <= 0)
    return set_error(nullptr, BLS_ERR_DEVICE, "no HIP device available");
  if (cfg.device < 0 || cfg.device >= ndev)
    return set_error(nullptr, BLS_ERR_INVALID_ARG, "device ordinal out of range");

  bls_plan *p = new (std::nothrow) bls_plan();
  if (!p) return set_error(nullptr, BLS_ERR_NO_MEMORY, "host allocation");
  p->cfg = cfg;
  p->device = cfg.device;
  auto fail = [&](int st) {
    snprintf(g_create_error, sizeof g_create_error, "%s", p->last_error.c_str());
    bls_plan_destroy(p);
    return st;
  };
  if ((e = hipSetDevice(p->device)) != hipSuccess) return fail(hip_error(p, e, "set device"));
  hipDeviceProp_t prop;
  if ((e = hipGetDeviceProperties(&prop, p->device)) != hipSuccess)
    return fail(hip_error(p, e, "device properties"));
  p->num_cus = prop.multiProcessorCount;
  p->max_lds = (int)prop.sharedMemPerBlock;
  if (cfg.hip_stream) {
    p->stream = (hipStream_t)cfg.hip_stream;
  } else {
    if ((e = hipStreamCreateWithFlags(&p->stream, hipStreamNonBlocking)) != hipSuccess)
      return fail(hip_error(p, e, "create stream"));
    p->own_stream = true;
  }
  for (hipEvent_t *ev : {&p->ev_begin, &p->ev_search0, &p->ev_search1, &p->ev_end, &p->ev_desc})
    if ((e = hipEventCreate(ev)) != hipSuccess) return fail(hip_error(p, e, "create event"));
  for (int i = 0; i < bls_plan::kTimeRing; ++i)
    if ((e = hipEventCreate(&p->ev_k0[i])) != hipSuccess ||
        (e = hipEventCreate(&p->ev_k1[i])) != hipSuccess)
      return fail(hip_error(p, e, "create event"));

  const size_t nc = (size_t)cfg.max_curves, npt = (size_t)cfg.max_points;
  struct {
    void **ptr;
    size_t bytes;
  } req[] = {{(void **)&p->d_curves, desc_bytes((int)nc)},
             {(void **)&p->d_dt, 8 * npt},
             {(void **)&p->d_q, 4 * npt},
             {(void **)&p->d_qw, 4 * npt},
             {(void **)&p->d_counter, 64}};
  for (auto &r : req)
    if ((e = device_alloc(r.ptr, r.bytes)) != hipSuccess)
      return fail(hip_error(p, e, "allocate plan buffers"));
  if ((e = hipHostMalloc((void **)&p->h_curves, desc_bytes((int)nc), 0)) != hipSuccess ||
      (e = hipHostMalloc((void **)&p->h_status, 4 * nc, hipHostMallocCoherent)) != hipSuccess ||
      (e = hipHostGetDevicePointer((void **)&p->status_dev, p->h_status, 0)) != hipSuccess)
    return fail(hip_error(p, e, "allocate pinned descriptors"));
  static_assert(kCurveOk == 0, "a status not yet written is that of a valid curve");
  memset(p->h_status, 0, 4 * nc);
  *out = p;
  return BLS_OK;
}

int bls_plan_destroy(bls_plan *p) {
  if (!p) return BLS_OK;
  if (p->stream) (void)hipStreamSynchronize(p->stream);
  for (void *d : {(void *)p->d_detect_desc, (void *)p->d_detect_out,
                  (void *)p->d_window_desc, (void *)p->d_window_flag,
                  (void *)p->d_var_noff, (void *)p->d_var_alive, (void *)p->d_var_chip,
                  (void *)p->d_uws})
    free_dev(d);
  for (void *d : {(void *)p->d_curves, (void *)p->d_dt, (void *)p->d_q, (void *)p->d_qw,
                  (void *)p->d_counter, (void *)p->d_t, (void *)p->d_sr})
    free_dev(d);
  for (void *h : {(void *)p->h_curves, (void *)p->h_status, (void *)p->h_stage})
    if (h) (void)hipHostFree(h);
  for (hipEvent_t ev : {p->ev_begin, p->ev_search0, p->ev_search1, p->ev_end, p->ev_desc})
    if (ev) (void)hipEventDestroy(ev);
  for (int i = 0; i < bls_plan::kTimeRing; ++i) {
    if (p->ev_k0[i]) (void)hipEventDestroy(p->ev_k0[i]);
    if (p->ev_k1[i]) (void)hipEventDestroy(p->ev_k1[i]);
  }
  if (p->own_stream && p->stream) (void)hipStreamDestroy(p->stream);
  delete p;
  return BLS_OK;
}

int bls_search(bls_plan *p, const double *times, const double *flux, const double *weights,
               int64_t n, const double *periods, int64_t nperiods, int32_t nbins, double qmin,
               double qmax, double *sr, double *phase, double *duration, double *depth,
               int32_t *jstart, int32_t *kwidth, int64_t *best_index) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (n < 0 || nperiods < 1)
    return set_error(p, BLS_ERR_INVALID_ARG, "need n >= 2 and nperiods >= 1");
  int64_t n_off[2] = {0, n};
  bls_batch b;
  memset(&b, 0, sizeof b);
  b.ncurves = 1;
  b.n_off = n_off;
  b.times = times;
  b.flux = flux;
  b.weights = weights;
  b.p_off = nullptr;
  b.periods = periods;
  b.nperiods_shared = nperiods;
  b.nbins_all = nbins;
  b.qmin_all = qmin;
  b.qmax_all = qmax;
  bls_results o{sr, phase, duration, depth, jstart, kwidth, best_index};
  return bls_search_batch(p, &b, &o);
}

int bls_search_batch(bls_plan *p, const bls_batch *b, const bls_results *out) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (!b || !out) return set_error(p, BLS_ERR_INVALID_ARG, "batch and out must be non-NULL");
  p->last_error.clear();
  std::string err;
  int st = validate_batch(p->cfg, *b, true, p->shapes, err);
  if (st != BLS_OK) return set_error(p, st, err);
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  return host_search(p, *b, p->shapes, *out);
}

int bls_search_device(bls_plan *p, const bls_batch *b, const bls_device_results *o) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (!b || !o || !o->sr || !o->depth || !o->jstart || !o->kwidth || !o->best_index)
    return set_error(p, BLS_ERR_INVALID_ARG, "batch and every device result array are required");
  p->last_error.clear();
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  // A call like the last one finds its plan made and its descriptors uploaded.
  const bool reuse = (p->cfg.flags & BLS_NO_GRAPH) == 0;
  const uint64_t sig = batch_signature(p, *b, *o);
  if (reuse && p->replay_valid && sig == p->replay_sig) {
    if ((e = hipEventRecord(p->ev_begin, p->stream)) != hipSuccess) return hip_error(p, e, "event");
    const int st = enqueue_search(p, p->last, b->times, b->flux, b->weights, b->periods, o->sr,
                                  o->depth, o->jstart, o->kwidth, o->best_index, false, false);
    if (st != BLS_OK) return st;
    if ((e = hipEventRecord(p->ev_end, p->stream)) != hipSuccess) return hip_error(p, e, "event");
    fill_stats(p, p->last, true);
    return BLS_OK;
  }
  std::string err;
  int st = validate_batch(p->cfg, *b, false, p->shapes, err);
  if (st != BLS_OK) return set_error(p, st, err);
  const bool weighted = b->weights != nullptr;
  TileChoice tc = choose_tiles(p, p->shapes, weighted);
  PlannedBatch pb;
  st = plan_batch(p, p->shapes, weighted, tc, pb);
  if (st != BLS_OK) return st;
  p->last = pb;
  if ((e = hipEventRecord(p->ev_begin, p->stream)) != hipSuccess) return hip_error(p, e, "event");
  st = enqueue_search(p, pb, b->times, b->flux, b->weights, b->periods, o->sr, o->depth,
                      o->jstart, o->kwidth, o->best_index);
  if (st != BLS_OK) return st;
  p->replay_sig = sig;
  p->replay_valid = reuse;
  if ((e = hipEventRecord(p->ev_end, p->stream)) != hipSuccess) return hip_error(p, e, "event");
  fill_stats(p, pb, false);
  return BLS_OK;
}

int bls_search_unbinned_device(bls_plan *p, const bls_batch *b, const bls_unbinned_results *o) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (!b || !o || !o->sr || !o->depth || !o->first_point || !o->last_point || !o->best_index)
    return set_error(p, BLS_ERR_INVALID_ARG, "batch and every device result array are required");
  p->last_error.clear();
  std::string err;
  int st = validate_batch(p->cfg, *b, false, p->shapes, err, false);
  if (st != BLS_OK) return set_error(p, st, err);
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  const bool weighted = b->weights != nullptr;
  const int nc = b->ncurves;
  PlannedBatch pb;
  pb.ncurves = nc;
  pb.weighted = weighted;
  std::vector<double> cost(nc);
  int ucap = 1;
  // the pinned descriptors are rewritten: the last search's plan goes stale,
  // and queued copies may still read them
  p->replay_valid = false;
  st = desc_wait(p);
  if (st != BLS_OK) return st;
  place_desc(p, nc);
  for (int c = 0; c < nc; ++c) {
    const CurveShape &s = p->shapes[c];
    CurveDesc &d = p->h_curves[c];
    memset(&d, 0, sizeof d);
    d.n_off = s.n_off;
    d.n = s.n;
    d.p_off = s.p_off;
    d.r_off = s.r_off;
    d.nperiods = s.nperiods;
    d.nbins = 0;
    const int cb = cbits_of(s.n);
    d.shift = 64 - cb;
    d.qbits = std::min(kQBitsMax, 63 - 2 * cb);
    d.weighted = weighted ? 1 : 0;
    d.check_periods = (c == 0 || s.p_off != p->shapes[0].p_off) ? 1 : 0;
    d.tile = 1;
    d.qlo = b->qmin ? b->qmin[c] : b->qmin_all;
    d.qhi = b->qmax ? b->qmax[c] : b->qmax_all;
    ucap = std::max<int>(ucap, (int)s.n);
    // a start's run covers about qhi * n points
    cost[c] = (double)s.n * (1.0 + d.qhi * (double)s.n);
    pb.total_points += s.n;
    pb.total_results += s.nperiods;
    pb.trial_points += (double)s.n * (double)s.nperiods;
    pb.box_evals += (double)s.n * d.qhi * (double)s.n * (double)s.nperiods;
  }
  std::vector<int64_t> items_of(nc);
  for (int c = 0; c < nc; ++c) items_of[c] = p->h_curves[c].nperiods;
  layout_partitions(p, cost, items_of, pb);
  const int64_t items = pb.nitems;
  pb.ucap = ucap;
  const bool glob = unbinned_mode(ucap) != kUnbLds;
  const int64_t arrays = unbinned_array_bytes(ucap, weighted);
  pb.hist_bytes = unbinned_lds_bytes(ucap, weighted);
  if (pb.hist_bytes > p->max_lds - 2048)
    return set_error(p, BLS_ERR_CAPACITY, "curve too long for the unbinned search's LDS");
  int per_cu = 0;
  if ((e = (hipError_t)unbinned_blocks_per_cu(weighted, (p->cfg.flags & BLS_DIP_ONLY) != 0, ucap,
                                              &per_cu)) != hipSuccess)
    return hip_error(p, e, "occupancy query");
  if (per_cu < 1) return set_error(p, BLS_ERR_CAPACITY, "unbinned kernel does not fit a CU");
  int64_t grid = std::min<int64_t>(items, (int64_t)p->num_cus * per_cu);
  if (glob) {
    // at most about 1 GiB of workspace (at least 32 workgroups)
    const int64_t stride = (arrays + 255) & ~(int64_t)255;
    grid = std::min<int64_t>(grid, std::max<int64_t>(32, ((int64_t)1 << 30) / stride));
    const int64_t need = grid * stride;
    if (need > p->uws_bytes) {
      // queued unbinned searches may still use the old workspace
      if ((e = hipStreamSynchronize(p->stream)) != hipSuccess) return hip_error(p, e, "synchronize");
      free_dev(p->d_uws);
      p->d_uws = nullptr;
      p->uws_bytes = 0;
      if ((e = device_alloc((void **)&p->d_uws, (size_t)need)) != hipSuccess)
        return hip_error(p, e, "allocate unbinned workspace");
      p->uws_bytes = need;
    }
    pb.uws = p->d_uws;
    pb.uws_stride = stride;
  }
  pb.grid = (int32_t)std::max<int64_t>(1, grid);
  p->last = pb;
  if ((e = hipEventRecord(p->ev_begin, p->stream)) != hipSuccess) return hip_error(p, e, "event");
  st = enqueue_search(p, pb, b->times, b->flux, b->weights, b->periods, o->sr, o->depth,
                      o->first_point, o->last_point, o->best_index, true);
  if (st != BLS_OK) return st;
  if ((e = hipEventRecord(p->ev_end, p->stream)) != hipSuccess) return hip_error(p, e, "event");
  fill_stats(p, pb, false);
  return BLS_OK;
}

int bls_detect_device(bls_plan *p, const bls_batch *b, const float *sr, int32_t max_peaks,
                      double window, double sde_threshold, bls_detection *out) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (!b || !sr || !out || max_peaks < 0 || max_peaks > BLS_MAX_PEAKS || !(window >= 0.0) ||
      !isfinite(window) || isnan(sde_threshold))
    return set_error(p, BLS_ERR_INVALID_ARG,
                     "need batch, sr, out, 0 <= max_peaks <= 16, finite window >= 0");
  std::string err;
  std::vector<CurveShape> shapes;
  int st = validate_batch(p->cfg, *b, false, shapes, err);
  if (st != BLS_OK) return set_error(p, st, err);
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  const int nc = b->ncurves;
  std::vector<DetectDesc> dd(nc);
  for (int c = 0; c < nc; ++c) {
    dd[c].p_off = shapes[c].p_off;
    dd[c].r_off = shapes[c].r_off;
    dd[c].nperiods = shapes[c].nperiods;
  }
  st = ensure_detect_buffers(p);
  if (st != BLS_OK) return st;
  hipStream_t s = p->stream;
  if ((e = hipMemcpyAsync(p->d_detect_desc, dd.data(), sizeof(DetectDesc) * nc,
                          hipMemcpyHostToDevice, s)))
    return hip_error(p, e, "upload detection descriptors");
  DetectArgs a;
  a.desc = p->d_detect_desc;
  a.periods = b->periods;
  a.sr = sr;
  a.out = p->d_detect_out;
  a.ncurves = nc;
  a.max_peaks = max_peaks;
  a.window = window;
  a.threshold = sde_threshold;
  if ((e = hipEventRecord(p->ev_search0, s)) != hipSuccess) return hip_error(p, e, "event");
  if ((e = (hipError_t)launch_detect(a, s))) return hip_error(p, e, "launch detection");
  if ((e = hipEventRecord(p->ev_search1, s)) != hipSuccess) return hip_error(p, e, "event");
  if ((e = hipMemcpyAsync(out, p->d_detect_out, sizeof(bls_detection) * nc,
                          hipMemcpyDeviceToHost, s)) ||
      (e = hipStreamSynchronize(s)))
    return hip_error(p, e, "detection");
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, p->ev_search0, p->ev_search1);
  p->stats = bls_call_stats{};
  p->stats.search_ms = p->stats.total_ms = ms;
  double m_total = 0.0;
  for (int c = 0; c < nc; ++c) m_total += (double)dd[c].nperiods;
  p->stats.trial_points = m_total;
  p->stats.block = kBlock;
  p->stats.grid = nc;
  return BLS_OK;
}

int bls_eclipse_window_device(bls_plan *p, const bls_batch *b, int32_t nphase, double duration,
                              int32_t min_eclipses, int32_t *observed) {
  if (!p) return BLS_ERR_INVALID_ARG;
  char msg[200];
  if (!b || !observed || b->ncurves < 1 || !b->n_off || !b->times || !b->periods)
    return set_error(p, BLS_ERR_INVALID_ARG,
                     "need a batch with ncurves >= 1, n_off, times, periods, and observed");
  if (nphase < 1 || nphase > BLS_MAX_NBINS || !(duration > 0.0) || !isfinite(duration) ||
      (min_eclipses != 1 && min_eclipses != 2))
    return set_error(p, BLS_ERR_INVALID_ARG,
                     "need 1 <= nphase <= 4096, finite duration > 0, min_eclipses 1 or 2");
  if (b->ncurves > p->cfg.max_curves) return set_error(p, BLS_ERR_CAPACITY, "too many cadences");
  if (b->n_off[0] != 0 || (b->p_off && b->p_off[0] != 0) ||
      (!b->p_off && b->nperiods_shared < 1))
    return set_error(p, BLS_ERR_INVALID_ARG, "n_off[0] and p_off[0] must be 0, grid non-empty");
  const int nc = b->ncurves;
  // up to 32 KB of LDS per workgroup: five workgroups per CU
  int tile = std::max(
      1, std::min(kTileMax, ((32 << 10) - kWindowStaticLds - 8 * window_pad(nphase)) /
                                (8 * nphase)));
  // A wave per period where the LDS then holds two workgroups' bins and the
  // call has periods for four rounds of them (call, the workgroup on a period
  // / a wave each: 24 x 100000 periods, 200 bins 2.00 / 1.79 ms, 1000 bins 3.13
  // / 2.64; 24 x 50000, 2000 bins 4.89 / 3.06; 12 x 50000, 3000 bins, one
  // workgroup per CU, 3.27 / 3.82; 4 x 20000, 1000 bins 0.212 / 0.189, but 2 x
  // 4500 0.097 / 0.100), up to eight periods per wave and item; and where the
  // waves hold every cadence in registers: read again for each period, 24 x
  // 20000 periods of 1100 weighted points, 300 bins 0.51 / 0.85 ms, 10 x 2725 of
  // 20000 points, 2000 bins 0.52 / 1.18.
  const double waves = std::max(p->num_cus, 1) * 4.0 * (kBlock / 64);
  double periods = 0.0;  // (checked below)
  int64_t longest = 0;
  for (int c = 0; c < nc; ++c) {
    periods += b->p_off ? (double)b->p_off[c + 1] - (double)b->p_off[c] : (double)b->nperiods_shared;
    longest = std::max(longest, b->n_off[c + 1] - b->n_off[c]);
  }
  const bool per_wave = 2 * window_lds_bytes(tile, nphase, true) <= p->max_lds &&
                        periods >= 4 * waves && longest <= kWindowWavePoints;
  if (per_wave) tile = (int)std::min(8.0, periods / waves) * (kBlock / 64);
  std::vector<WindowDesc> wd(nc);
  int64_t items = 0, results = 0;
  for (int c = 0; c < nc; ++c) {
    WindowDesc &d = wd[c];
    memset(&d, 0, sizeof d);
    d.n_off = b->n_off[c];
    d.n = b->n_off[c + 1] - b->n_off[c];
    const int64_t np = b->p_off ? b->p_off[c + 1] - b->p_off[c] : b->nperiods_shared;
    if (d.n < 1 || np < 1 || np > INT32_MAX) {
      snprintf(msg, sizeof msg, "cadence %d has %lld points and %lld periods (need >= 1 each)", c,
               (long long)d.n, (long long)np);
      return set_error(p, BLS_ERR_INVALID_ARG, msg);
    }
    d.p_off = b->p_off ? b->p_off[c] : 0;
    d.r_off = b->p_off ? b->p_off[c] : (int64_t)c * b->nperiods_shared;
    d.nperiods = (int32_t)np;
    d.check_periods = (b->p_off || c == 0) ? 1 : 0;
    d.item0 = items;
    items += (np + tile - 1) / tile;
    results += np;
  }
  if (b->n_off[nc] > p->cfg.max_points || results > p->cfg.max_periods)
    return set_error(p, BLS_ERR_CAPACITY, "points or periods exceed the plan's limits");
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  if (!p->d_window_desc) {
    if ((e = device_alloc((void **)&p->d_window_desc, sizeof(WindowDesc) * p->cfg.max_curves)) ||
        (e = device_alloc((void **)&p->d_window_flag, sizeof(unsigned int)))) {
      if (p->d_window_desc) (void)hipFree(p->d_window_desc);
      p->d_window_desc = nullptr;
      p->d_window_flag = nullptr;
      return hip_error(p, e, "allocate eclipse-window buffers");
    }
  }
  const int lds = window_lds_bytes(tile, nphase, per_wave);
  int per_cu = 0;
  if ((e = (hipError_t)window_blocks_per_cu(per_wave, min_eclipses, lds, &per_cu)) != hipSuccess)
    return hip_error(p, e, "window occupancy");
  const int64_t grid = std::min<int64_t>(items, (int64_t)std::max(per_cu, 1) * p->num_cus * 4);
  hipStream_t s = p->stream;
  const unsigned int zero = 0;
  if ((e = hipMemcpyAsync(p->d_window_desc, wd.data(), sizeof(WindowDesc) * nc,
                          hipMemcpyHostToDevice, s)) ||
      (e = hipMemcpyAsync(p->d_window_flag, &zero, sizeof zero, hipMemcpyHostToDevice, s)))
    return hip_error(p, e, "upload window descriptors");
  WindowArgs a;
  a.desc = p->d_window_desc;
  a.ncurves = nc;
  a.tile = tile;
  a.nitems = items;
  a.t = b->times;
  a.w = b->weights;
  a.periods = b->periods;
  a.observed = observed;
  a.nphase = nphase;
  a.min_eclipses = min_eclipses;
  a.duration = duration;
  a.overflow = p->d_window_flag;
  a.per_wave = per_wave;
  if ((e = hipEventRecord(p->ev_search0, s)) != hipSuccess) return hip_error(p, e, "event");
  if ((e = (hipError_t)launch_window(a, (int)grid, s))) return hip_error(p, e, "launch window");
  if ((e = hipEventRecord(p->ev_search1, s)) != hipSuccess) return hip_error(p, e, "event");
  unsigned int flag = 0;
  if ((e = hipMemcpyAsync(wd.data(), p->d_window_desc, sizeof(WindowDesc) * nc,
                          hipMemcpyDeviceToHost, s)) ||
      (e = hipMemcpyAsync(&flag, p->d_window_flag, sizeof flag, hipMemcpyDeviceToHost, s)) ||
      (e = hipStreamSynchronize(s)))
    return hip_error(p, e, "eclipse window");
  {
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, p->ev_search0, p->ev_search1);
    p->stats = bls_call_stats{};
    p->stats.search_ms = p->stats.total_ms = ms;
    double pp = 0.0, dec = 0.0;
    for (int c = 0; c < nc; ++c) {
      pp += (double)wd[c].n * (double)wd[c].nperiods;
      dec += (double)wd[c].nperiods * (double)nphase;
    }
    p->stats.trial_points = pp;
    p->stats.box_evals = dec;
    p->stats.work_items = items;
    p->stats.grid = (int32_t)grid;
    p->stats.block = kBlock;
    p->stats.lds_bytes = lds;
  }
  for (int c = 0; c < nc; ++c) {
    if (wd[c].status != kCurveOk) {
      snprintf(msg, sizeof msg, "cadence %d: %s", c,
               wd[c].status == kCurveBadData     ? "non-finite kept time or a bad weight"
               : wd[c].status == kCurveBadPeriod ? "a trial period is not finite and > 0"
                                                 : "no point with positive weight");
      return set_error(p, BLS_ERR_INVALID_ARG, msg);
    }
  }
  if (flag)
    return set_error(p, BLS_ERR_CAPACITY, "a cadence spans more than 2^29 cycles of a period");
  return BLS_OK;
}

int bls_variability_device(bls_plan *p, const bls_batch *b, const bls_variability_config *cfg,
                           const bls_variability_results *o) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (!b || !cfg || !o || !b->n_off || !b->flux || !cfg->chip_off || !cfg->mag || !o->rms ||
      !o->bin || !o->flag || !o->bin_mean || !o->bin_std || !o->bin_count)
    return set_error(p, BLS_ERR_INVALID_ARG,
                     "need batch (n_off, flux), config (chip_off, mag) and every result array");
  const int nc = b->ncurves, nk = cfg->nchips;
  if (nc < 1 || nk < 1 || cfg->nmagbins < 1 || !(cfg->width > 0.0) || !isfinite(cfg->width) ||
      !isfinite(cfg->origin) || !(cfg->clip_sigma > 0.0) || !(cfg->flag_sigma >= 0.0) ||
      cfg->max_iter < 0 || cfg->min_stars < 1)
    return set_error(p, BLS_ERR_INVALID_ARG,
                     "need ncurves, nchips, nmagbins >= 1, finite origin, width > 0, "
                     "clip_sigma > 0, flag_sigma >= 0, max_iter >= 0, min_stars >= 1");
  if (nc > p->cfg.max_curves || cfg->nmagbins > kVarMaxBins || cfg->max_iter > kVarMaxIter)
    return set_error(p, BLS_ERR_CAPACITY,
                     "more curves than max_curves, nmagbins > 4096 or max_iter > 64");
  if (b->n_off[0] != 0 || cfg->chip_off[0] != 0 || cfg->chip_off[nk] != nc)
    return set_error(p, BLS_ERR_INVALID_ARG, "n_off[0], chip_off[0] must be 0; "
                                             "chip_off[nchips] must equal ncurves");
  for (int c = 0; c < nc; ++c)
    if (b->n_off[c + 1] < b->n_off[c])
      return set_error(p, BLS_ERR_INVALID_ARG, "n_off must be non-decreasing");
  for (int k = 0; k < nk; ++k)
    if (cfg->chip_off[k + 1] < cfg->chip_off[k])
      return set_error(p, BLS_ERR_INVALID_ARG, "chip_off must be non-decreasing");
  if (b->n_off[nc] > p->cfg.max_points)
    return set_error(p, BLS_ERR_CAPACITY, "points exceed the plan's max_points");
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  if (!p->d_var_noff) {
    const size_t mc = (size_t)p->cfg.max_curves;
    if ((e = device_alloc((void **)&p->d_var_noff, 8 * (mc + 1))) ||
        (e = device_alloc((void **)&p->d_var_alive, mc))) {
      free_dev(p->d_var_noff);
      free_dev(p->d_var_alive);
      p->d_var_noff = nullptr;
      p->d_var_alive = nullptr;
      return hip_error(p, e, "allocate variability scratch");
    }
  }
  if (nk > p->var_chip_cap) {
    free_dev(p->d_var_chip);
    p->d_var_chip = nullptr;
    p->var_chip_cap = 0;
    if ((e = device_alloc((void **)&p->d_var_chip, 8 * ((size_t)nk + 1))))
      return hip_error(p, e, "allocate chip offsets");
    p->var_chip_cap = nk;
  }
  hipStream_t s = p->stream;
  if ((e = hipMemcpyAsync(p->d_var_noff, b->n_off, 8 * ((size_t)nc + 1), hipMemcpyHostToDevice,
                          s)) ||
      (e = hipMemcpyAsync(p->d_var_chip, cfg->chip_off, 8 * ((size_t)nk + 1),
                          hipMemcpyHostToDevice, s)))
    return hip_error(p, e, "upload offsets");
  VarArgs a;
  memset(&a, 0, sizeof a);
  a.ncurves = nc;
  a.nchips = nk;
  a.nmagbins = cfg->nmagbins;
  a.max_iter = cfg->max_iter;
  a.min_stars = cfg->min_stars;
  a.n_off = p->d_var_noff;
  a.chip_off = p->d_var_chip;
  a.x = b->flux;
  a.w = b->weights;
  a.mag = cfg->mag;
  a.origin = cfg->origin;
  a.width = cfg->width;
  a.clip_sigma = cfg->clip_sigma;
  a.flag_sigma = cfg->flag_sigma;
  a.rms = o->rms;
  a.bin = o->bin;
  a.flag = o->flag;
  a.bin_mean = o->bin_mean;
  a.bin_std = o->bin_std;
  a.bin_count = o->bin_count;
  a.alive = p->d_var_alive;
  if ((e = hipEventRecord(p->ev_search0, s)) != hipSuccess) return hip_error(p, e, "event");
  if ((e = (hipError_t)launch_variability(a, s))) return hip_error(p, e, "launch variability");
  if ((e = hipEventRecord(p->ev_search1, s)) != hipSuccess) return hip_error(p, e, "event");
  if ((e = hipStreamSynchronize(s))) return hip_error(p, e, "variability");
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, p->ev_search0, p->ev_search1);
  p->stats = bls_call_stats{};
  p->stats.search_ms = p->stats.total_ms = ms;
  p->stats.trial_points = (double)b->n_off[nc];
  p->stats.box_evals = (double)nc;
  p->stats.block = kBlock;
  return BLS_OK;
}

int bls_debug_phase_bins(bls_plan *p, const double *times, int64_t n, double period,
                         int32_t nbins, int32_t *bins) {
  if (!p) return BLS_ERR_INVALID_ARG;
  if (!times || !bins || n < 2 || !isfinite(period) || !(period > 0.0) || nbins < 2)
    return set_error(p, BLS_ERR_INVALID_ARG, "need times, bins, n >= 2, period > 0, nbins >= 2");
  if (n > p->cfg.max_points || n > (int64_t(1) << 24))
    return set_error(p, BLS_ERR_CAPACITY, "n exceeds the plan's max_points");
  for (int64_t i = 0; i < n; ++i)
    if (!isfinite(times[i])) return set_error(p, BLS_ERR_INVALID_ARG, "non-finite time");
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  int st = ensure_staging(p);
  if (st != BLS_OK) return st;
  p->replay_valid = false;
  st = desc_wait(p);
  if (st != BLS_OK) return st;
  CurveDesc &d = p->h_curves[0];
  memset(&d, 0, sizeof d);
  d.n = n;
  d.nperiods = 1;
  d.nbins = nbins;
  const int cb = cbits_of(n);
  d.shift = 64 - cb;
  d.qbits = std::min(kQBitsMax, 63 - 2 * cb);
  hipStream_t s = p->stream;
  if ((e = hipMemcpyAsync(p->d_curves, p->h_curves, sizeof(CurveDesc), hipMemcpyHostToDevice,
                          s)) != hipSuccess ||
      (e = hipMemcpyAsync(p->d_t, times, n * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
      (e = hipMemcpyAsync(p->d_periods, &period, 8, hipMemcpyHostToDevice, s)) != hipSuccess)
    return hip_error(p, e, "upload");
  if ((st = desc_mark(p)) != BLS_OK) return st;
  PrepArgs pa;
  pa.curves = p->d_curves;
  pa.periods = p->d_periods;
  pa.ncurves = 1;
  pa.t = p->d_t;
  pa.x = p->d_t;  // any finite flux: only the time offsets are used
  pa.w = nullptr;
  pa.dt = p->d_dt;
  pa.q = p->d_q;
  pa.qw = p->d_qw;
  if ((e = (hipError_t)launch_prep(pa, s)) != hipSuccess) return hip_error(p, e, "launch prep");
  // into the encoded fluxes, which hold max_points values and are not needed
  if ((e = (hipError_t)launch_bins(p->d_dt, n, p->d_periods, nbins, p->d_q, s)) != hipSuccess)
    return hip_error(p, e, "launch bins");
  if ((e = hipMemcpyAsync(bins, p->d_q, n * 4, hipMemcpyDeviceToHost, s)) != hipSuccess)
    return hip_error(p, e, "download bins");
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_error(p, e, "synchronize");
  return BLS_OK;
}

int bls_synchronize(bls_plan *p) {
  if (!p) return BLS_ERR_INVALID_ARG;
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  // one wait for the results and the curves' status
  const int st = wait_for_status(p);
  if (st != BLS_OK) return st;
  float ms = 0.f;
  if (hipEventElapsedTime(&ms, p->ev_begin, p->ev_end) == hipSuccess) p->stats.total_ms = ms;
  p->desc_pending = false;
  p->stats.search_ms = last_kernel_ms(p);
  return p->last.ncurves > 0 ? check_device_status(p, p->last.ncurves) : BLS_OK;
}

int bls_get_stream(const bls_plan *p, void **stream) {
  if (!p || !stream) return BLS_ERR_INVALID_ARG;
  *stream = (void *)p->stream;
  return BLS_OK;
}

int bls_width_range(int32_t nbins, double qmin, double qmax, int32_t *kmin, int32_t *kmax) {
  return width_range(nbins, qmin, qmax, kmin, kmax);
}

int bls_last_error(const bls_plan *p, char *buf, size_t len) {
  if (!buf || len == 0) return BLS_ERR_INVALID_ARG;
  const char *m = p ? p->last_error.c_str() : g_create_error;
  const size_t n = std::min(len - 1, strlen(m));
  memcpy(buf, m, n);
  buf[n] = '\0';
  return BLS_OK;
}

const char *bls_status_string(int status) {
  switch (status) {
    case BLS_OK: return "ok";
    case BLS_ERR_INVALID_ARG: return "invalid argument";
    case BLS_ERR_NO_MEMORY: return "out of memory";
    case BLS_ERR_DEVICE: return "device (HIP) error";
    case BLS_ERR_CAPACITY: return "exceeds plan capacity";
    case BLS_ERR_BUSY: return "not ready";
    case BLS_ERR_TIMEOUT: return "timed out";
    default: return "unknown status";
  }
}

int bls_last_stats(const bls_plan *p, bls_call_stats *out) {
  if (!p || !out) return BLS_ERR_INVALID_ARG;
  *out = p->stats;
  return BLS_OK;
}

int bls_kernel_times(bls_plan *p, float *ms, int32_t max, int32_t *count) {
  if (!p || !count || max < 0 || (max > 0 && !ms)) return BLS_ERR_INVALID_ARG;
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return hip_error(p, e, "set device");
  if ((e = hipStreamSynchronize(p->stream)) != hipSuccess) return hip_error(p, e, "synchronize");
  const int64_t avail = std::min<int64_t>(p->k_recorded - p->k_base, bls_plan::kTimeRing);
  const int64_t n = std::min<int64_t>(avail, max);
  // the most recent n launches, oldest first
  for (int64_t i = 0; i < n; ++i) {
    const int64_t k = p->k_recorded - n + i;
    const int slot = (int)(k % bls_plan::kTimeRing);
    float v = 0.f;
    if ((e = hipEventElapsedTime(&v, p->ev_k0[slot], p->ev_k1[slot])) != hipSuccess)
      return hip_error(p, e, "event timing");
    ms[i] = v;
  }
  *count = (int32_t)n;
  return BLS_OK;
}

int bls_kernel_times_reset(bls_plan *p) {
  if (!p) return BLS_ERR_INVALID_ARG;
  p->k_base = p->k_recorded;
  return BLS_OK;
}

}  // extern "C"
