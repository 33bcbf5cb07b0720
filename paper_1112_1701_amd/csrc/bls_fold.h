// The fold shared by the search kernels: phases and bins of a tile of periods
// accumulated exactly in LDS (one 64-bit atomic per point and period), and the
// decoding of a bin word.
//
// No FP contraction anywhere (-ffp-contract=off): the phase is computed with
// exactly the FP64 operation sequence of its definition so that every point
// falls into the same bin as in an FP64 evaluation.
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "bls_device.h"

namespace bls {
namespace {

// One bin word holds (count << shift) + sum of signed fixed-point values.
// |sum| < 2^46 < 2^(shift - 1), so the sum is the sign-extended low field
// and the count is what remains above it.
struct BinWord {
  long long sum;
  unsigned count;
};

__device__ inline BinWord decode_word(unsigned long long u, int shift) {
  BinWord w;
  const int hi = 64 - shift;
  w.sum = ((long long)(u << hi)) >> hi;
  // a negative sum borrowed one from the count field
  w.count = (unsigned)(u >> shift) - (unsigned)(w.sum >> 63);
  return w;
}

// Correctly rounded float of an integer with |v| < 2^47: both halves convert
// exactly and the fused multiply-add rounds once.
__device__ inline float int47_to_float(long long v) {
  const int hi = (int)(v >> 24);
  const unsigned lo = (unsigned)v & 0xFFFFFFu;
  return fmaf((float)hi, 16777216.0f, (float)lo);
}

// trunc(frac(d f) nbins) with the FP64 operation order of the definition.
// For finite c >= 0, c - floor(c) is exact and below 1, so v_fract_f64
// returns exactly that value.  The result lies in [0, nbins]; nbins itself
// (phase so close to 1 that the product rounds up) is the clamp case of the
// definition.
__device__ inline int raw_bin(double d, double f, double nbd) {
  const double c = d * f;
  const double ph = __builtin_amdgcn_fract(c);
  return (int)(ph * nbd);
}

__device__ inline int phase_bin(double d, double f, double nbd, unsigned nbm1) {
  return (int)min((unsigned)raw_bin(d, f, nbd), nbm1);
}

// A 64-bit value every lane holds alike, moved to scalar registers.
__device__ inline int64_t uniform_i64(int64_t v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((uint64_t)v & 0xFFFFFFFFu));
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Lane spacing of the fold for one work item, in units of kPPT points:
// 1, 2 or 4 (a chunk is kBlock / 64 = 4 waves of 64 lanes).  On a dense
// cadence, points close in time fall into one bin at long periods, and
// lanes of one LDS atomic on the same word are serialised.  The gap is
// the smallest that puts adjacent lanes half a bin apart in phase at the
// tile's longest period (fmin = its smallest frequency); cadence is the
// curve's median time step.  Where lanes are that far apart already, the
// contiguous layout (gap 1) is the faster one.
static_assert(kBlock == 256 && kPPT == 4, "the fold's lane layout assumes 4 waves of 4 points");

__device__ inline int fold_lane_gap(double fmin, int nbins, float cadence) {
  // x = (lane step in time) / (bin width in time at the longest period)
  const double x = fmin * (double)nbins * (double)kPPT * (double)cadence;
  return !(x < 0.5) || !(x > 0.0) ? 1 : x >= 0.25 ? 2 : 4;
}

// Whether a tile's fold merges a thread's consecutive same-bin points: when
// one cadence step advances the phase by less than 0.3 bins at the tile's
// longest period (frequency fmin), so that runs of about three points or
// more share a bin, unless the launch fixes the choice (policy 1: always,
// 2: never).  The merge costs VALU operations on every point and saves one
// LDS atomic per point it joins; shorter runs do not repay it.  A weighted
// point saves two atomics, and there the merge pays from one bin per step.
// The block search, whose VALU is the busier, merges unit-weight points from
// 0.15 bins per step (1000 bins, 1-minute cadence, 8 curves x 40000 periods of
// 1.5 to 3 days: 7.2 ms merged, 6.8 not; 6 to 20 days: 7.4 and 7.9).
// The points past the last whole chunk follow the same rule: merged always, 550
// points took 1.5% longer and 240 weighted curves of about 2500 2.3%; never,
// 100 curves of 1000 points 2 minutes apart x 4000 periods x 24 bins 2.13 ms
// instead of 0.76 (weighted), 3000 points a minute apart x 10000 x 250 1.55 / 1.26.
// Any answer is correct; this one only picks the faster fold.
__device__ inline bool fold_merges(double fmin, int nbins, float cadence, int policy,
                                   bool weighted, double from = 0.3) {
  if (policy != 0) return policy == 1;
  const double x = fmin * (double)nbins * (double)cadence;
  return !(x >= (weighted ? 1.0 : from));
}

// Fold and bin one chunk of kBlock * kPPT points into the tile's histograms.
// Each thread takes kPPT consecutive points, so the 64 lanes of one atomic
// instruction hold points kPPT apart in time: their phases (hence bins and
// LDS banks) are far less correlated than those of 64 consecutive points of
// a sorted light curve, which cuts same-bin and same-bank collisions.
// Each period's histogram plane starts HS words after the previous one: nb
// bins, the word after them (it catches the clamp case and is added to bin
// nb - 1 when the histogram is decoded, later the start of the wrap-around
// copy), and padding that keeps the scan's reads free of bank conflicts.
// Weighted curves use two such planes per period, A (count, weight) then B
// (weighted signal), each contiguous so that the lanes of one atomic spread
// over all LDS banks.
// MERGE: consecutive points of a thread that share a bin are summed first;
// without it every point is one atomic (tiles whose periods are short
// against the cadence, where neighbours almost never share a bin).
// A thread's points of one chunk as they are loaded: time offsets, encoded
// values and weights (weighted curves).
struct FoldRegs {
  double d[kPPT];
  int32_t q[kPPT], qw[kPPT];
};

// Offset of the thread's first point in a chunk.  The lanes of a wave are
// kPPT gap points apart and the waves interleave (gap 1, 2 or 4).
__device__ inline int fold_offset(int gap) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  return kPPT * (l * gap + (w & (gap - 1))) + 64 * kPPT * gap * (w >> (gap >> 1));
}

// The points of a whole chunk (off: its first point in the packed arrays).
template <bool WEIGHTED>
__device__ inline void fold_load(const SearchArgs &a, int64_t off, int k0, FoldRegs &p) {
#pragma unroll
  for (int r = 0; r < kPPT; ++r) {
    p.d[r] = a.dt[off + k0 + r];
    p.q[r] = a.q[off + k0 + r];
    p.qw[r] = WEIGHTED ? a.qw[off + k0 + r] : 0;
  }
}

// Bin a thread's kPPT loaded points at the tile's np periods.  MERGE:
// consecutive points of a thread that share a bin are summed first; without
// it every point is one atomic (tiles whose periods are short against the
// cadence, where neighbours almost never share a bin).
// AHEAD: the next period's frequency is read before this one's atomics (LDS
// operations end in order, and a read after them waits for them all); for
// kernels that have the registers.
template <bool WEIGHTED, bool MERGE, bool AHEAD>
__device__ inline void fold_points(const FoldRegs &p, int nbins, int shift, int np,
                                   const double *s_f, unsigned long long *s_hist, int HS) {
  const double nbd = (double)nbins;
  const unsigned long long one = 1ull << shift;
  unsigned long long va[kPPT];
  unsigned long long vb[kPPT];
#pragma unroll
  for (int r = 0; r < kPPT; ++r) {
    const long long qi = p.q[r];
    if (WEIGHTED) {
      va[r] = p.qw[r] >= 0 ? one + (unsigned long long)(long long)p.qw[r] : 0ull;
      vb[r] = (unsigned long long)qi;
    } else {
      va[r] = one + (unsigned long long)qi;
      vb[r] = 0;
    }
  }
  constexpr int wpb = WEIGHTED ? 2 : 1;
  double fnext = AHEAD ? s_f[0] : 0.0;
  for (int t = 0; t < np; ++t) {
    const double f = AHEAD ? fnext : s_f[t];
    if (AHEAD) fnext = s_f[min(t + 1, np - 1)];
    unsigned long long *h = s_hist + (size_t)t * HS * wpb;
    // A thread's consecutive points that share a bin (common at long
    // periods) are summed in registers and sent as one atomic.
    int bin[kPPT];
#pragma unroll
    for (int r = 0; r < kPPT; ++r) bin[r] = raw_bin(p.d[r], f, nbd);
    if (!MERGE) {
#pragma unroll
      for (int r = 0; r < kPPT; ++r) {
        __hip_atomic_fetch_add(h + bin[r], va[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (WEIGHTED)
          __hip_atomic_fetch_add(h + HS + bin[r], vb[r], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      continue;
    }
    unsigned long long accA = 0, accB = 0;
#pragma unroll
    for (int r = 0; r < kPPT; ++r) {
      accA += va[r];
      if (WEIGHTED) accB += vb[r];
      if (r == kPPT - 1 || bin[r + 1 < kPPT ? r + 1 : r] != bin[r]) {  // the run ends
        __hip_atomic_fetch_add(h + bin[r], accA, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (WEIGHTED)
          __hip_atomic_fetch_add(h + HS + bin[r], accB, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        accA = 0;
        accB = 0;
      }
    }
  }
}

// Load and bin one chunk of kBlock kPPT points (or, gap 1, the calling wave's
// 64 kPPT of them).
template <bool WEIGHTED, bool MERGE>
__device__ inline void fold_chunk(const SearchArgs &a, const CurveDesc &cd, int64_t base,
                                  int np, const double *s_f, unsigned long long *s_hist,
                                  int HS, int gap) {
  // The gap passes through an opaque copy so that the compiler recomputes
  // the offset per chunk instead of holding it in VGPRs through the item.
  asm volatile("" : "+s"(gap));
  FoldRegs p;
  fold_load<WEIGHTED>(a, uniform_i64(cd.n_off + base), fold_offset(gap), p);
  fold_points<WEIGHTED, MERGE, false>(p, cd.nbins, cd.shift, np, s_f, s_hist, HS);
}

// The curve's last points, fewer than kBlock kPPT of them (`left` from point
// `base` on), kPPT to a thread as in a whole chunk, merged or not likewise.
template <bool WEIGHTED, bool MERGE>
__device__ inline void fold_rest(const SearchArgs &a, const CurveDesc &cd, int64_t base, int left,
                                 int np, const double *s_f, unsigned long long *s_hist, int HS) {
  const int64_t off = uniform_i64(cd.n_off + base);
  const int k0 = fold_offset(1);
  const double nbd = (double)cd.nbins;
  const unsigned long long one = 1ull << cd.shift;
  double d[kPPT];
  unsigned long long va[kPPT], vb[kPPT];
#pragma unroll
  for (int r = 0; r < kPPT; ++r) {
    const bool ok = k0 + r < left;
    const int64_t i = off + (ok ? k0 + r : 0);
    d[r] = a.dt[i];
    const long long qi = a.q[i];
    const int qwi = WEIGHTED ? a.qw[i] : 0;
    va[r] = !WEIGHTED ? one + (unsigned long long)qi
            : qwi >= 0 ? one + (unsigned long long)(long long)qwi : 0ull;
    vb[r] = (unsigned long long)qi;
  }
  constexpr int wpb = WEIGHTED ? 2 : 1;
  if (k0 >= left) return;
  for (int t = 0; t < np; ++t) {
    unsigned long long *h = s_hist + (size_t)t * HS * wpb;
    const double f = s_f[t];
    int bin[kPPT];
    if (MERGE) {
#pragma unroll
      for (int r = 0; r < kPPT; ++r) bin[r] = raw_bin(d[r], f, nbd);
    }
    unsigned long long accA = 0, accB = 0;
#pragma unroll
    for (int r = 0; r < kPPT; ++r) {
      if (k0 + r < left) {
        accA = MERGE ? accA + va[r] : va[r];
        if (WEIGHTED) accB = MERGE ? accB + vb[r] : vb[r];
        const int rn = r + 1 < kPPT ? r + 1 : r;
        if (!MERGE || r == kPPT - 1 || k0 + rn >= left || bin[rn] != bin[r]) {  // the run ends
          unsigned long long *w = h + (MERGE ? bin[r] : raw_bin(d[r], f, nbd));
          __hip_atomic_fetch_add(w, accA, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (WEIGHTED)
            __hip_atomic_fetch_add(w + HS, accB, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          accA = accB = 0;
        }
      }
    }
  }
}

// The whole chunks of a curve, each one's points loaded while the one before
// is binned.
template <bool WEIGHTED, bool MERGE>
__device__ inline void fold_chunks(const SearchArgs &a, const CurveDesc &cd, int64_t nchunks,
                                   int np, const double *s_f, unsigned long long *s_hist, int HS,
                                   int gap) {
  int64_t off = cd.n_off;
  const int k0 = fold_offset(gap);
  FoldRegs next;
  fold_load<WEIGHTED>(a, off, k0, next);
  for (int64_t i = 0; i < nchunks; ++i) {
    const FoldRegs p = next;
    off += kBlock * kPPT;
    if (i + 1 < nchunks) fold_load<WEIGHTED>(a, off, k0, next);
    fold_points<WEIGHTED, MERGE, true>(p, cd.nbins, cd.shift, np, s_f, s_hist, HS);
  }
}

// The curve's last points, one wave's share of fewer than 64 kPPT of them
// (`left` from point `first` on): a point per lane and step, as many steps as
// there are points for, instead of kPPT per lane with most lanes idle.
template <bool WEIGHTED>
__device__ inline void fold_tail(const SearchArgs &a, const CurveDesc &cd, int64_t first, int left,
                                 int np, const double *s_f, unsigned long long *s_hist, int HS) {
  const int64_t off = uniform_i64(cd.n_off + first);
  const int lane = threadIdx.x & 63;
  const double nbd = (double)cd.nbins;
  const unsigned long long one = 1ull << cd.shift;
  constexpr int wpb = WEIGHTED ? 2 : 1;
  for (int k = lane; k < left; k += 64) {
    const double d = a.dt[off + k];
    const long long qi = a.q[off + k];
    unsigned long long va = one + (unsigned long long)qi, vb = 0ull;
    if (WEIGHTED) {
      const int qwi = a.qw[off + k];
      va = qwi >= 0 ? one + (unsigned long long)(long long)qwi : 0ull;
      vb = (unsigned long long)qi;
    }
    for (int t = 0; t < np; ++t) {
      unsigned long long *h = s_hist + (size_t)t * HS * wpb + raw_bin(d, s_f[t], nbd);
      __hip_atomic_fetch_add(h, va, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (WEIGHTED)
        __hip_atomic_fetch_add(h + HS, vb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
}

}  // namespace
}  // namespace bls
