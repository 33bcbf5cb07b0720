// gfx950 search kernel for boxes of at most half the bins: phase and bin as
// in bls_kernels.hip, then find each period's best box by bounds over blocks
// of start and end bins instead of scoring every box.
//
// What bounds it.  Scoring every box costs 4.5 VALU instructions per box and
// was most of the former kernel's time (a period of the 300-bin uniform batch
// has 8400 boxes, one of the 1000-bin long baseline 46000).  Here a wave owns
// a period: the bins become prefix sums in place, about 60 to 120 blocks of
// consecutive prefix sums keep their extremes, and one test per pair of
// blocks (25 to 80 boxes) rejects all but about a twentieth of the pairs; the
// boxes of the rest are scored from prefix differences.  What is left is the
// fold, its FP64 operations and LDS atomics; below about 500 bins the search
// itself is still the larger part (a period of 2000 points and 300 bins takes
// 1270 VALU instructions, 1480 in search_kernel).
//
// Measured, search_kernel against this one (weights within a factor of four,
// boxes of 0.01 to 0.1 cycle where not stated): 169 weighted curves x 859
// points x 6456 periods x 525 bins 8.8 / 5.9 ms; 6 x 24601 x 26314 x 897 (0.005
// to 0.08) 3.1 / 2.2; weighted 3 x 36710 x 42741 x 864 (0.005 to 0.08) 4.2 /
// 3.6; 24 x 50000 x 100000 x 1000 (0.005 to 0.05) 51.5 / 44.2.
//
// VALU instructions per CU and clock (1.15 is what search_kernel reaches at
// 300 bins), and the share of the clocks in which the LDS is active: 300 bins
// 0.92 and 0.62, weighted 0.75 and 0.61; 525 bins 0.87 and 0.43, weighted 0.71
// and 0.43; 1000 bins and 20000 points 0.74 and 0.71, weighted 0.63 and 0.60.
// So neither is full: the registers and the LDS leave six to three waves per
// SIMD, whose latencies (LDS, cross-lane sums) show.
//
// The answer is exactly the one that scoring every box in FP32 gives: bounds
// and scores carry an error term that covers every rounding on both sides,
// and unless one box is above all others by more than that, the boxes in
// question are scored by the FP32 running sums of the definition.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include "bls_block.h"
#include "bls_device.h"
#include "bls_fold.h"
#include "bls_items.h"
#include "../../include/bls.h"

namespace bls {
namespace {

typedef unsigned long long u64;

// Prunings of the candidate list after which a sweep is left (on noise it is
// pruned once at its end), at least; one per 2^13 boxes where there are more,
// as scoring every start bin then costs 35 instructions per 64 boxes against
// 500 a pruning (periods longer than the data, 46 curves x 8267 points x 68
// periods to 20 d in 10 d x 2271 bins, 0.041 to 0.397: 5.3 ms with eight, 1.3
// so, 1.2 with every box).  And the error of a difference of two prefix words'
// weights, in quanta.
constexpr int kMaxPrunes = 8;
constexpr float kWordError = 3.0f;
// Theta where no box is known to be valid: below the value of any that holds a
// signal (its bound is at least 2^-20, R (W - R) below 2^62).  With 0 there
// the boxes that cannot be dips (a bound of 0) would pass the screens.
constexpr float kThetaMin = 0x1p-110f;
constexpr int kMarked = -2;  // PeriodScan::best: left to marked_starts

// LDS operations of one wave complete in order; this keeps the compiler from
// moving them across.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// v_max_f32 and v_min_f32 as they are: fmaxf would first quiet both operands,
// and nothing here is a signalling NaN.
__device__ __forceinline__ float max_raw(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float min_raw(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Inclusive prefix sum of 64-bit integers across the wave: row shifts by 1,
// 2, 4 and 8, then the rows' totals broadcast into the rows after them.
template <int CTRL>
__device__ __forceinline__ u64 scan_step(u64 v) {
  const unsigned lo = (unsigned)dpp_zero<CTRL>((int)(unsigned)v);
  const unsigned hi = (unsigned)dpp_zero<CTRL>((int)(unsigned)(v >> 32));
  return v + (((u64)hi << 32) | lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ u64 scan_rows(u64 v) {
  const unsigned lo = (unsigned)dpp_i32<CTRL, ROWS>((int)(unsigned)v);
  const unsigned hi = (unsigned)dpp_i32<CTRL, ROWS>((int)(unsigned)(v >> 32));
  return v + (((u64)hi << 32) | lo);
}

__device__ __forceinline__ u64 wave_scan(u64 v) {
  v = scan_step<0x111>(v);
  v = scan_step<0x112>(v);
  v = scan_step<0x114>(v);
  v = scan_step<0x118>(v);
  v = scan_rows<0x142, 0xa>(v);
  return scan_rows<0x143, 0xc>(v);
}

__device__ __forceinline__ u64 lane_u64(u64 v, int lane) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
  return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ float lane_f32(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// A value every lane holds alike, moved to a scalar register (the curve record
// is read through vector loads: the kernel writes global memory).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ int lanes_below(u64 mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// One period's search by one wave.  U: the period's plane of bin words (and
// for weighted curves V, the plane of signal words), nb bins and the clamp
// word, zeros up to the plane's end.  scr: the wave's scratch.
//
// Words to numbers: a signed number of quanta 2^x (x = count bits + qbits -
// 31) is the 32 bits of a signal (or weight) sum from bit x on.  The count
// field lies above the signal; a box's signal is less than half the field
// (the values are centred), so the count between two prefixes is the rounded
// difference of their high words, also across the end of the cycle, where
// the field has wrapped.
template <bool WEIGHTED, bool DIP>
struct PeriodScan {
  u64 *U, *V;
  float4 *tab;           // block: largest, smallest and first prefix sum, first count (weight)
  float2 *tab2;          // block: last count (weight), least count (weight) of kmin bins
  int *cand;             // candidate boxes: j | k << 16
  unsigned short *queue; // passing block pairs: start block | offset << 8
  unsigned *marks;       // start bins with a box in question
  const int lane, nb, kmin, kmax, s, NB, omin, omax, pad;
  const int x, sh;
  const unsigned magic, half;
  const float nf, mipf, Wf, qscale;
  const int qwmin;
  const bool mip1;
  float Wt;      // total count (weight) in the units of the prefix counts
  float E;       // error of a signal difference, all roundings (quanta)
  float c0, eR;  // weighted: absolute and relative error of a weight difference
  float Ws, es;  // screens: R (Ws - R) (1 - es) is at most what a box may give
                 // whose weight is at least R
  float wlo;     // least weight of a valid box (positive)
  float theta, thr;  // largest lower value of a valid box; the same, relaxed
  float thrs, tW;    // the screens' threshold, and times Ws
  int qn;            // queued block pairs
  int ncand;         // candidates
  int prunes;        // times the list was pruned in this sweep; kMaxPrunes: the
                     // sweep is left, for more candidates than that resolves

  __device__ __forceinline__ PeriodScan(const CurveDesc &d, int mip, u64 *u, u64 *v,
                                        unsigned char *scr)
      : U(u), V(v), lane(threadIdx.x & 63), nb(uniform(d.nbins)), kmin(uniform(d.kmin)),
        kmax(uniform(d.kmax)), s(uniform(d.bsize)), NB(uniform(d.nblocks)),
        omin(uniform(d.omin)), omax(uniform(d.omax)), pad(NB * s - nb),
        x(uniform(33 - d.shift + d.qbits)), sh(uniform(d.shift - 32)),
        magic((unsigned)uniform(d.bmagic)), half(1u << (sh - 1)), nf(uniform((float)d.n_eff)),
        mipf((float)mip), Wf(uniform(d.Wf)), qscale(uniform(ldexpf(1.0f, -d.qbits))),
        qwmin(uniform(d.qwmin)), mip1(mip <= 1) {
    tab = reinterpret_cast<float4 *>(scr);
    tab2 = reinterpret_cast<float2 *>(tab + NB + omax + 3);
    cand = reinterpret_cast<int *>(tab2 + NB);
    queue = reinterpret_cast<unsigned short *>(cand + kBlockCand);
    marks = reinterpret_cast<unsigned *>(queue + kBlockQueue);
  }

  __device__ __forceinline__ int low(u64 w) const {
    return (int)__builtin_amdgcn_alignbit((unsigned)(w >> 32), (unsigned)w, (unsigned)x);
  }
  __device__ __forceinline__ static unsigned high(u64 w) { return (unsigned)(w >> 32); }
  // Points between two prefixes: from the high word h1 of the later one and
  // the earlier one's less half a count.
  __device__ __forceinline__ int points(unsigned h1, unsigned h0_half) const {
    return (int)((h1 - h0_half) >> sh);
  }
  // Weight (count, or quanta of weight) between two prefixes.
  __device__ __forceinline__ int weight(u64 w1, u64 w0) const {
    return WEIGHTED ? low(w1) - low(w0) : points(high(w1), high(w0) - half);
  }
  __device__ __forceinline__ int first_of(int b) const { return b * s - (b < NB ? 0 : pad); }

  // A lane's block of K bins (u, v: its words): the bins and their sums.
  template <int K>
  __device__ __forceinline__ void totals(const u64 *u, const u64 *v, u64 *w, u64 *wv, u64 &su,
                                         u64 &sv) const {
#pragma unroll
    for (int i = 0; i < K; ++i) {
      w[i] = u[i];
      if (WEIGHTED) wv[i] = v[i];
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
      su += w[i];
      if (WEIGHTED) sv += wv[i];
    }
  }
  // Their prefixes in place (run: before the first, after the last), the
  // extremes, and the prefix before the last bin.
  template <int K>
  __device__ __forceinline__ void prefixes(u64 *u, u64 *v, const u64 *w, const u64 *wv, u64 &run,
                                           u64 &runv, u64 &last, int &hi, int &lo) const {
#pragma unroll
    for (int i = 0; i < K; ++i) {
      u[i] = run;
      if (WEIGHTED) v[i] = runv;
      const int p = low(WEIGHTED ? runv : run);
      hi = max(hi, p);
      lo = min(lo, p);
      last = run;
      run += w[i];
      if (WEIGHTED) runv += wv[i];
    }
  }
  // One wave-full of blocks (a: the lane's block): scan of the blocks' sums,
  // prefixes, table entries.  K > 0: all K = s bins of a block in registers;
  // K = 0: any s, four bins at a time, read twice.
  template <int K>
  __device__ __forceinline__ void prefix_round(int a, u64 &carry, u64 &carryv, float &rhi,
                                               float &rlo) {
    constexpr int KR = K > 0 ? K : 4;
    const bool live = a < NB;
    u64 *u = U + (live ? a * s : 0), *v = V + (live ? a * s : 0);
    u64 su = 0ull, sv = 0ull, w[KR], wv[KR];
    if (live) {
      if (K > 0) {
        totals<KR>(u, v, w, wv, su, sv);
      } else {
        int m = 0;
        for (; m + 4 <= s; m += 4) totals<4>(u + m, v + m, w, wv, su, sv);
        for (; m < s; ++m) totals<1>(u + m, v + m, w, wv, su, sv);
      }
    }
    const u64 iu = wave_scan(su);
    u64 run = carry + (iu - su);
    carry += lane_u64(iu, 63);
    u64 runv = 0ull;
    if (WEIGHTED) {
      const u64 iv = wave_scan(sv);
      runv = carryv + (iv - sv);
      carryv += lane_u64(iv, 63);
    }
    if (live) {
      const int p0 = low(WEIGHTED ? runv : run);
      const float cf = (float)weight(run, 0ull);
      int hi = p0, lo = p0;
      u64 last = run;  // prefix before the block's last bin
      if (K > 0) {
        prefixes<KR>(u, v, w, wv, run, runv, last, hi, lo);
      } else {
        int m = 0;
        u64 t0 = 0ull, t1 = 0ull;
        for (; m + 4 <= s; m += 4) {
          totals<4>(u + m, v + m, w, wv, t0, t1);
          prefixes<4>(u + m, v + m, w, wv, run, runv, last, hi, lo);
        }
        for (; m < s; ++m) {
          totals<1>(u + m, v + m, w, wv, t0, t1);
          prefixes<1>(u + m, v + m, w, wv, run, runv, last, hi, lo);
        }
      }
      const float fh = (float)hi, fl = (float)lo;
      rhi = max_raw(rhi, fh);
      rlo = max_raw(rlo, -fl);
      tab[a] = make_float4(fh, fl, (float)p0, cf);
      tab2[a].x = (float)weight(last, 0ull);
    }
  }
  // Least weight of kmin consecutive bins from K start bins.  (Past nb - 1 the
  // last block's words belong to the next cycle or to nothing: they can only
  // lower the bound.)
  template <int K>
  __device__ __forceinline__ void narrowest(const u64 *u, int &least) const {
    u64 w0[K], w1[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      w0[i] = u[i];
      w1[i] = u[i + kmin];
    }
#pragma unroll
    for (int i = 0; i < K; ++i) least = min(least, weight(w1[i], w0[i]));
  }

  // Bins to prefix sums (U[i]: before bin i), the wrapped copy up to nb +
  // kmax, and the blocks' extremes.  A lane takes block a's s bins; s is odd
  // so that the lanes' strides spread over the LDS banks.
  __device__ __forceinline__ void prefix() {
    if (lane == 0) {  // the clamp word joins the last bin
      const u64 cw = U[nb];
      U[nb] = 0ull;
      U[nb - 1] += cw;
      if (WEIGHTED) {
        const u64 cv = V[nb];
        V[nb] = 0ull;
        V[nb - 1] += cv;
      }
    }
    wave_sync();
    u64 carry = 0ull, carryv = 0ull;
    float rhi = 0.0f, rlo = 0.0f;  // largest prefix sum, smallest (negated); U[0] = 0
    for (int r = 0; r < NB; r += 64) {
      if (s == 5)
        prefix_round<5>(r + lane, carry, carryv, rhi, rlo);
      else if (s == 7)
        prefix_round<7>(r + lane, carry, carryv, rhi, rlo);
      else if (s == 3)
        prefix_round<3>(r + lane, carry, carryv, rhi, rlo);
      else
        prefix_round<0>(r + lane, carry, carryv, rhi, rlo);
    }
    // one cycle's totals
    const u64 tot = carry, totv = carryv;
    const float Pt = (float)low(WEIGHTED ? totv : tot);
    Wt = WEIGHTED ? (float)low(tot) : nf;
    wave_sync();
    for (int i = lane; i <= kmax; i += 64) {
      U[nb + i] = U[i] + tot;
      if (WEIGHTED) V[nb + i] = V[i] + totv;
    }
    for (int i = lane; i <= omax + 1; i += 64) {
      float4 t = tab[i];
      t.x += Pt;
      t.y += Pt;
      t.z += Pt;
      t.w += Wt;
      tab[NB + i] = t;
    }
    wave_sync();
    // Every signal difference used below is within E of the FP32 running sum
    // of the same bins.  With D the range of the prefix sums: the quanta (8:
    // the floors of both prefixes and of the total), the conversions to float
    // and their sums (2^-24 D each, at most 16 of them), and the running sum
    // itself, whose kmax additions each round a sum of at most D (and a term
    // of at most D) by 2^-24 of it.
    E = uniform(8.0f + (wave_fmax(rhi) + wave_fmax(rlo)) * ((float)(2 * kmax + 16) * 0x1.01p-24f));
    c0 = WEIGHTED ? uniform(3.0f + Wt * 0x1p-22f) : 0.0f;
    eR = uniform((float)(kmax + 8) * 0x1p-24f);
    wlo = WEIGHTED ? uniform(max_raw(mipf * (float)qwmin, 1.0f) * ldexpf(1.0f, -x)) : mipf;
    // Least weight of kmin consecutive bins from each block's starts (weights:
    // two quanta less, the floors of both prefixes).
    for (int a = lane; a < NB; a += 64) {
      int least = 0x7fffffff, m = 0;
      const u64 *u = U + a * s;
      for (; m + 4 <= s; m += 4) narrowest<4>(u + m, least);
      if (m + 3 == s)
        narrowest<3>(u + m, least);
      else
        narrowest<1>(u + m, least);
      tab2[a].y = (float)(WEIGHTED ? least - 2 : least);
    }
    // The screens take R and W - R at their least: R less its absolute error
    // where it comes from prefix weights (c0 from the blocks' table, two quanta
    // from the words), W - R with Ws for W; then the rounding of the running
    // weight, which is relative.
    Ws = Wt;
    if (WEIGHTED) {
      Ws = uniform(Wt - 2.0f * (Wt * eR + c0));
      es = uniform(2.0f * eR);
    }
    wave_sync();
  }
  // Whether no bin holds a signal (a constant curve): no box has a value then.
  __device__ __forceinline__ bool flat() const {
    bool any = false;
    for (int i = lane; i < nb; i += 64)
      any |= WEIGHTED ? V[i + 1] != V[i] : ((U[i + 1] - U[i]) << (32 - sh)) != 0ull;
    return __builtin_amdgcn_ballot_w64(any) == 0ull;
  }
  // Least and largest R (W - R) that the FP32 sums of a valid box may give (c:
  // the absolute error of R; that of W - R is c0, by the rounding of W).
  __device__ __forceinline__ void denominators(float R, float c, float &den_lo,
                                               float &den_hi) const {
    const float d = Wt - R;
    if (WEIGHTED) {
      const float er = fmaf(R, eR, c), ed = fmaf(R, eR, c0);
      // (points of encoded weight 0 do not make a box valid)
      const float least = qwmin > 0 ? wlo * (1.0f - 0x1p-12f) : 0.0f;
      den_lo = max_raw(R - er, least) * max_raw(d - ed, 0.0f);
      den_hi = (R + er) * (d + ed);
    } else {
      den_lo = den_hi = R * d;
    }
  }

  // Lower value of a box that is certainly valid, 0 otherwise (weighted
  // curves with a minimum count: cnt is its count).
  __device__ __forceinline__ float lower(float S, float R, int cnt) const {
    float lo, hi;
    denominators(R, kWordError, lo, hi);
    const float sl = (DIP ? -S : fabsf(S)) - E;
    bool ok = sl > 0.0f;
    if (WEIGHTED)
      ok = ok & (lo > 0.0f) & (mip1 | ((float)cnt >= mipf));
    else
      ok = ok & (R >= mipf) & (R < Wt);
    return ok ? sl * sl * __builtin_amdgcn_rcpf(hi) * (1.0f - 0x1p-18f) : 0.0f;
  }
  // The same for box (j, e) from its prefixes.
  __device__ __forceinline__ float lower_at(int j, int e) const {
    const u64 u0 = U[j], u1 = U[e];
    const int cnt = points(high(u1), high(u0) - half);
    const float R = (float)(WEIGHTED ? low(u1) - low(u0) : cnt);
    return lower((float)(WEIGHTED ? low(V[e]) - low(V[j]) : low(u1) - low(u0)), R, cnt);
  }

  __device__ __forceinline__ void raise(float t) {
    theta = uniform(t);
    thr = uniform(t * (1.0f - 0x1p-17f));
    thrs = WEIGHTED ? uniform(thr * (1.0f - es)) : thr;
    // (Points are counted exactly, but the product is rounded: an error of
    // W - R that is all of it where a box leaves few.)
    tW = uniform(thrs * (WEIGHTED ? Ws : Ws * (1.0f - 0x1p-22f)));
  }

  // A first theta: boxes between the blocks' first bins, then the boxes
  // around the best of them.
  __device__ __forceinline__ void seed() {
    // offsets whose boxes are within the width range, wrapped or not
    const int o0 = max(1, (kmin + pad + s - 1) / s), o1 = min(omax, kmax / s);
    float bv = 0.0f;
    int bp = 0;
    for (int r = 0; r < NB; r += 64) {
      const int a = min(r + lane, NB - 1);
      const float4 *tp = tab + a;
      const float4 t0 = *tp;
      // Every other offset: all of them raise the first theta by a twentieth
      // of the best value and save two of thirty passing pairs.
      float4 tn = tp[o0];
      for (int o = o0; o <= o1; o += 2) {
        // Lower value as in lower(); where R (W - R) is not positive the box
        // holds no signal either, and the quotient is NaN or not above 0, or
        // it holds every point and the remainder of an inexact mean: infinite.
        const float4 t = tn;
        tn = tp[min(o + 2, o1)];
        const float R = t.w - t0.w;
        const float S = t.z - t0.z;
        const float sl = max_raw((DIP ? -S : fabsf(S)) - E, 0.0f);
        float lo, hi;
        denominators(R, c0, lo, hi);
        const float v = sl * sl * __builtin_amdgcn_rcpf(hi);
        bool ok = v > bv;
        if (WEIGHTED) {
          ok = ok & (lo > 0.0f);
          if (!mip1)
            ok = ok & ((float)points(high(U[first_of(a + o)]), high(U[a * s]) - half) >= mipf);
        } else if (!mip1) {
          ok = ok & (R >= mipf);
        }
        bv = ok ? v : bv;
        bp = ok ? (r | (o << 8)) : bp;
      }
    }
    bv *= 1.0f - 0x1p-18f;
    float t = wave_fmax(bv);
    if (!WEIGHTED && t == __builtin_inff()) t = 0.0f;  // (none is valid: the sweep finds one)
    if (t > 0.0f) {
      const u64 m = __builtin_amdgcn_ballot_w64(bv == t);
      const int l = (int)__builtin_ctzll(m);
      const int p = __builtin_amdgcn_readlane(bp, l);
      const int a = min((p & 255) + l, NB - 1), b = a + (p >> 8);
      const int j = a * s - 4 + (lane & 7), k = first_of(b) - a * s + (lane >> 3) - (lane & 7);
      float v = 0.0f;
      if (j >= 0 && j < nb && k >= kmin && k <= kmax) v = lower_at(j, j + k);
      t = max_raw(t, wave_fmax(v));
    }
    raise(max_raw(t, kThetaMin));
  }

  // K boxes from start j (ends e0 + i on; len boxes in all), scored against
  // thr.  The words past a lane's last box are read but not scored: planes
  // have room for them.  Boxes not below theta become candidates (MARK: their
  // start bins are marked).
  template <int K, bool MARK>
  __device__ __forceinline__ void boxes(int i, int e0, int j, int len, unsigned h0, int l0,
                                        int s0) {
    u64 w[K], any = 0ull, hit[K];
    int sv[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
      w[q] = U[e0 + i + q];
      sv[q] = WEIGHTED ? low(V[e0 + i + q]) : 0;
    }
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const float S = (float)((WEIGHTED ? sv[q] : low(w[q])) - s0);
      const float R =
          max_raw((float)(WEIGHTED ? low(w[q]) - l0 : points(high(w[q]), h0)), wlo);
      const float su = DIP ? max_raw(E - S, 0.0f) : E + fabsf(S);
      hit[q] = __builtin_amdgcn_ballot_w64(su * su >= R * fmaf(R, -thrs, tW)) &
               __builtin_amdgcn_ballot_w64(i + q < len);
      any |= hit[q];
    }
    if (any == 0ull) return;
#pragma unroll
    for (int q = 0; q < K; ++q) {
      if (hit[q] == 0ull) continue;
      const bool mine = __builtin_amdgcn_inverse_ballot_w64(hit[q]);
      if (MARK) {
        if (mine)
          __hip_atomic_fetch_or(&marks[j >> 5], 1u << (j & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
      } else {
        // (at most half of the list is in use here)
        if (mine) cand[ncand + lanes_below(hit[q])] = j | ((e0 + i + q - j) << 16);
        ncand += (int)__popcll(hit[q]);
        if (ncand > kBlockCand / 2) {
          wave_sync();
          prune();
          prunes = ncand > kBlockCand / 2 ? kMaxPrunes : prunes + 1;
          ncand = min(ncand, kBlockCand / 2);
          qn = prunes >= kMaxPrunes ? 0 : qn;  // (ends the loop over the queue)
        }
      }
    }
  }

  // The boxes of the queued block pairs, a lane per (pair, start bin).
  template <bool MARK>
  __device__ __forceinline__ void drain() {
    wave_sync();
    // lane -> (pair, start bin) of a batch of 64 / s pairs
    const int pl = (int)(((unsigned)lane * magic) >> 20), js = lane - pl * s;
    const int per = 64 / s;
    for (int base = 0; base < qn; base += per) {
      const bool in = (pl < per) & (base + pl < qn);
      const int ent = queue[in ? base + pl : 0];
      const int as = (ent & 255) * s, fbw = as + (ent >> 8) * s;
      const int fb = fbw - (fbw < NB * s ? 0 : pad);
      const int j = min(as + js, nb - 1);
      const int e1 = max(fb, j + kmin);
      int e2 = min(fb + s - 1, j + kmax);
      // (the last block's ends stop at nb - 1, its start bins likewise)
      if (pad != 0) e2 = as + js >= nb ? 0 : fb < nb ? min(e2, nb - 1) : e2;
      const u64 u0 = U[j], u1 = U[j + 1];
      const unsigned h0 = high(u0) - half;
      // A box whose first bin is empty ties with the one from the next bin
      // on, which is narrower and so preferred, unless it is of least width.
      if (!MARK && points(high(u1), h0) == 0) e2 = min(e2, j + kmin);
      const int len = in ? e2 - e1 + 1 : 0;
      const int l0 = low(u0) + 2, s0 = WEIGHTED ? low(V[j]) : low(u0);
      const int e0 = len > 0 ? e1 : j;  // (lanes without boxes read in range)
      int i = 0;
      for (; i + 4 <= s; i += 4) boxes<4, MARK>(i, e0, j, len, h0, l0, s0);
      if (i + 3 == s)
        boxes<3, MARK>(i, e0, j, len, h0, l0, s0);
      else
        boxes<1, MARK>(i, e0, j, len, h0, l0, s0);
    }
    qn = 0;
    wave_sync();
  }

  // Every pair (start block a, end block a + o) that can hold a box of value
  // theta is queued, and the queue is worked off as it fills.  S over the
  // pair is at most the difference of the blocks' extremes, and R (W - R) is
  // concave in R, so its least value is at the least or the largest R.
  template <bool MARK>
  __device__ __forceinline__ void sweep() {
    qn = 0;
    for (int r = 0; r < NB; r += 64) {
      const u64 live = NB - r >= 64 ? ~0ull : (1ull << (NB - r)) - 1ull;
      const int a = min(r + lane, NB - 1);
      float4 t0 = tab[a];
      float2 u0 = tab2[a];
      if (WEIGHTED) {
        t0.w -= c0;
        u0.x += c0;
      }
      const float4 *tp = tab + a + omin;
      float4 t = tp[0], tn = tp[1];
      for (int o = omin; o <= omax; ++o) {
        const float4 t2 = tp[2];  // (one entry past the table's last is read, not used)
        ++tp;
        const float dn = t0.x - t.y;
        const float sm = DIP ? max_raw(dn + E, 0.0f) : max_raw(t.x - t0.y, dn) + E;
        float R1 = max_raw(t.w - u0.x, u0.y), R2 = tn.w - t0.w;
        R1 = max_raw(R1, wlo);
        if (!WEIGHTED) R2 = min_raw(R2, Wt - 1.0f);
        const float g = min_raw(R1 * fmaf(R1, -thrs, tW), R2 * fmaf(R2, -thrs, tW));
        t = tn;
        tn = t2;
        // (g is negative where a box could hold every point: that passes)
        const u64 m = __builtin_amdgcn_ballot_w64(sm * sm >= g) & live;
        if (m != 0ull) {
          if (__builtin_amdgcn_inverse_ballot_w64(m))
            queue[qn + lanes_below(m)] = (unsigned short)(a | (o << 8));
          qn += (int)__popcll(m);
          if (qn >= 64) {
            drain<MARK>();
            if (!MARK) {  // (a return here would cost 25 to 40 spilled SGPRs)
              o = prunes >= kMaxPrunes ? omax : o;
              r = prunes >= kMaxPrunes ? NB : r;
            }
          }
        }
      }
    }
    if (qn > 0) drain<MARK>();
  }

  // Bin i as the running sums of the definition take it.
  __device__ __forceinline__ float2 bin(int i, float qscale, int &cnt) const {
    const BinWord w = decode_word(U[i + 1] - U[i], sh + 32);
    cnt = (int)w.count;
    if (WEIGHTED)
      return make_float2(int47_to_float(w.sum) * qscale,
                         int47_to_float((long long)(V[i + 1] - V[i])) * qscale);
    return make_float2((float)w.count, int47_to_float(w.sum) * qscale);
  }

  // Every width from start bin j by FP32 running sums, in bin order: the
  // chain runs along the lanes (lane l's sum is its neighbour's plus bin l),
  // one addition per bin.  Returns the key of the start's best box, taken in
  // the order of the widths by the divide-free comparison; 0 if none.  At the
  // start bins that search_kernel seeds its scan with, the box of least width
  // also counts by itself, as it does there.
  __device__ __forceinline__ u64 exact_start(int j) {
    float cS = 0.0f, cR = 0.0f, bn = 0.0f, bd = 1.0f;
    int bm = -1;
    u64 key = 0ull;
    const int sq = (j * 32 + nb - 1) / nb;
    const bool seeded = sq < 32 && sq * nb / 32 == j;
    for (int base = 0; base < kmax; base += 64) {
      const int m = base + lane;
      const bool in = m < kmax;
      int c = 0;
      float2 e = make_float2(0.0f, 0.0f);
      if (in) e = bin(j + m, qscale, c);
      const int C = points(high(U[min(j + m + 1, nb + kmax)]), high(U[j]) - half);
      float S = 0.0f, R = 0.0f;
      const int steps = min(64, kmax - base);
      for (int i = 0; i < steps; ++i) {
        const float ps = __int_as_float(__builtin_amdgcn_update_dpp(
            __float_as_int(cS), __float_as_int(S), 0x138, 0xf, 0xf, false));
        S = ps + e.y;
        if (WEIGHTED) {
          const float pr = __int_as_float(__builtin_amdgcn_update_dpp(
              __float_as_int(cR), __float_as_int(R), 0x138, 0xf, 0xf, false));
          R = pr + e.x;
        }
      }
      cS = lane_f32(S, 63);
      cR = lane_f32(R, 63);
      float d;
      if (WEIGHTED) {
        d = Wf - R;
      } else {
        R = (float)C;  // exact, as W - (W - R) in the running form
        d = Wf - R;
      }
      const float num = S * S, den = R * d;
      bool ok = in & (m + 1 >= kmin) & (num > 0.0f) & (den > 0.0f);
      if (WEIGHTED)
        ok = ok & ((float)C <= nf - 1.0f) & ((float)C >= mipf);
      else
        ok = ok & (d >= 1.0f) & (mip1 | (R >= mipf));
      if (DIP) ok = ok & (S < 0.0f);
      if (seeded && kmin - 1 >= base && kmin - 1 < base + 64) {
        const int l = kmin - 1 - base;
        if ((__builtin_amdgcn_ballot_w64(ok) >> l) & 1ull)
          key = key_of(lane_f32(num, l), lane_f32(den, l), kmin, j);
      }
      const float top = wave_fmax(ok ? num * __builtin_amdgcn_rcpf(den) : 0.0f);
      u64 mask = __ballot(ok && num >= top * (1.0f - 0x1p-14f) * den);
      while (mask != 0ull) {
        const int l = (int)__builtin_ctzll(mask);
        mask &= mask - 1;
        const float ln = lane_f32(num, l), ld = lane_f32(den, l);
        if (ln * bd > bn * ld) {
          bn = ln;
          bd = ld;
          bm = base + l;
        }
      }
    }
    return max(key, bm < 0 ? 0ull : key_of(bn, bd, bm + 1, j));
  }
  // Every width from the marked start bins, a lane each, by the same sums, tests
  // and order as exact_start: where there are too many to take one by one.
  __device__ __forceinline__ int marked_starts() const {
    u64 key = 0ull;
    int n = 0;  // marked starts in hand (cand)
    for (int base = 0; base < nb || n > 0; base += 64) {
      if (base < nb) {
        const bool in = base + lane < nb && ((marks[(base + lane) >> 5] >> (lane & 31)) & 1u) != 0u;
        const u64 m = __builtin_amdgcn_ballot_w64(in);
        if (in) cand[n + lanes_below(m)] = base + lane;
        n += (int)__popcll(m);
        wave_sync();
        if (n < 64 && base + 64 < nb) continue;
        if (n == 0) break;
      }
      const int j = cand[min(lane, n - 1)];  // (the last one again where there are fewer)
      const int left = cand[min(64 + lane, kBlockCand - 1)];
      n = max(n - 64, 0);
      wave_sync();
      cand[lane] = left;
      wave_sync();
      const int sq = (j * 32 + nb - 1) / nb;
      const bool seeded = sq < 32 && sq * nb / 32 == j;
      float S = 0.0f, R = 0.0f, bn = 0.0f, bd = 1.0f;
      int bm = -1, C = 0;
#pragma unroll 1
      for (int m = 0; m < kmax; ++m) {
        int c;
        const float2 e = bin(j + m, qscale, c);
        S += e.y;
        C += c;
        if (WEIGHTED)
          R += e.x;
        else
          R = (float)C;
        if (m + 1 < kmin) continue;
        const float d = Wf - R;
        const float num = S * S, den = R * d;
        bool ok = num * bd > bn * den;
        if (WEIGHTED)
          ok = ok & (den > 0.0f) & ((float)C <= nf - 1.0f) & ((float)C >= mipf);
        else
          ok = ok & (d >= 1.0f) & (mip1 | (R >= mipf));
        if (DIP) ok = ok & (S < 0.0f);
        if (ok) {
          bn = num;
          bd = den;
          bm = m;
          if (m + 1 == kmin && seeded) key = max(key, key_of(num, den, kmin, j));
        }
      }
      if (bm >= 0) key = max(key, key_of(bn, bd, bm + 1, j));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) key = max(key, (u64)__shfl_xor(key, o, 64));
    return box_of(lane_u64(key, 0));
  }
  // The box of a key: j | k << 16, or -1.
  __device__ __forceinline__ int box_of(u64 key) const {
    if (key == 0ull) return -1;
    const unsigned idx = 0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull);
    const int k = (int)(idx / (unsigned)nb);
    const int j = (int)(idx - (unsigned)k * (unsigned)nb);
    return j | (k << 16);
  }
  // Key of a box: its value, then the smaller width and start.
  __device__ __forceinline__ u64 key_of(float bn, float bd, int k, int j) const {
    const float v = bn * __builtin_amdgcn_rcpf(bd);
    const unsigned idx = (unsigned)k * (unsigned)nb + (unsigned)j;
    return ((u64)__float_as_uint(v) << 32) | (u64)(0xFFFFFFFFu - idx);
  }

  // The kept candidates' lower values raise theta; those then below it leave,
  // and boxes that are not valid or tie with one that is preferred: with an
  // empty last bin (the narrower box without it), or, of least width, with
  // the same points as the box one bin earlier.  Returns the last one kept.
  __device__ __forceinline__ int prune() {
    int kept = 0, jkept = -1;
    const int n = min(ncand, kBlockCand);
    float top = 0.0f;
    for (int pass = 0; pass < 2; ++pass) {
      for (int base = 0; base < n; base += 64) {
        const bool in = base + lane < n;
        const int jk = cand[in ? base + lane : 0];
        const int j = jk & 0xFFFF, k = jk >> 16, e = j + k;
        const u64 u0 = U[j], u1 = U[e], ul = U[e - 1];
        const unsigned h0 = high(u0) - half;
        const int cnt = points(high(u1), h0);
        const float R = (float)(WEIGHTED ? low(u1) - low(u0) : cnt);
        const float S = (float)(WEIGHTED ? low(V[e]) - low(V[j]) : low(u1) - low(u0));
        if (pass == 0) {
          top = max_raw(top, lower(S, R, cnt));
        }
        if (n > 64 && pass == 0) continue;
        if (pass == 0) raise(max_raw(theta, wave_fmax(top)));
        float lo, hi;
        denominators(max_raw(R, wlo), kWordError, lo, hi);
        const float su = DIP ? max_raw(E - S, 0.0f) : E + fabsf(S);
        const bool last_empty = points(high(u1), high(ul) - half) == 0;
        const bool same_before = (j > 0) & (points(high(u0), high(U[max(j - 1, 0)]) - half) == 0);
        const u64 m = __builtin_amdgcn_ballot_w64(
            in & (su * su >= thr * lo) & ((float)cnt >= mipf) & ((float)cnt <= nf - 1.0f) &
            (su > 0.0f) & !(last_empty & (k > kmin || same_before)));
        if (__builtin_amdgcn_inverse_ballot_w64(m)) cand[kept + lanes_below(m)] = jk;
        if (m != 0ull) jkept = __builtin_amdgcn_readlane(jk, 63 - (int)__builtin_clzll(m));
        kept += (int)__popcll(m);
      }
      if (n <= 64) break;
      if (pass == 0) raise(max_raw(theta, wave_fmax(top)));
    }
    ncand = kept;
    wave_sync();
    return jkept;
  }

  // Of a pruned list, without the boxes of least width that run past the end of
  // the cycle and hold the same points as the one from bin 0 (the first point
  // is always there): how many are left, and the last of them.
  __device__ __forceinline__ int distinct(int &jk) const {
    const bool in = lane < ncand;
    const int c = cand[in ? lane : 0];
    const int j = c & 0xFFFF, k = c >> 16, e = j + k;
    const int other = points(high(U[nb]), high(U[j]) - half) +
                      points(high(U[kmin]), high(U[min(max(e - nb, 0), kmin)]) - half);
    const u64 m =
        __builtin_amdgcn_ballot_w64(in & !((e > nb) & (k == kmin) & (other == 0)));
    if (m != 0ull) jk = __builtin_amdgcn_readlane(c, 63 - (int)__builtin_clzll(m));
    return (int)__popcll(m);
  }

  // Best box of the period: j | k << 16, -1 if there is none, kMarked where
  // marked_starts has to find it.
  __device__ __forceinline__ int best() {
    prefix();
    seed();
    if (!(theta > kThetaMin) && flat()) return -1;
    // A sweep that is left for its many candidates is taken once more if theta
    // has risen since its start (a seed of little value); where it has not,
    // boxes in question are the rule.
    float before;
    int tries = 0;
    do {
      before = theta;
      ncand = 0;
      prunes = min(0, kMaxPrunes - (nb * kmax >> 13));
      sweep<false>();
    } while (prunes >= kMaxPrunes && ++tries < 2 && theta > 1.1f * before);
    if (prunes >= kMaxPrunes) {
      for (int i = lane; i < (nb + 31) / 32; i += 64) marks[i] = ~0u;
      return kMarked;
    }
    // With every candidate at hand, a single box not below theta is the best.
    if (ncand == 0) return -1;
    int jk = cand[0];
    if (ncand > 1 || !(theta > kThetaMin)) jk = prune();
    if (ncand == 0) return -1;
    if (theta > kThetaMin && (ncand == 1 || distinct(jk) == 1)) return jk;
    // Boxes within the error of each other: all of them once more, their
    // start bins marked, and those starts by the definition's running sums
    // (about 3 kmax + 100 instructions a start, 35 kmax for 64 at a time).
    for (int i = lane; i < (nb + 31) / 32; i += 64) marks[i] = 0u;
    wave_sync();
    sweep<true>();
    int starts = 0;
    for (int i = lane; i < (nb + 31) / 32; i += 64) starts += (int)__popc(marks[i]);
    starts = wave_isum(starts);
    if (starts * (3 * kmax + 100) > (starts + 63) / 64 * 35 * kmax) return kMarked;
    u64 key = 0ull;
    for (int i = 0; i < (nb + 31) / 32; ++i) {
      unsigned word = (unsigned)__builtin_amdgcn_readfirstlane((int)marks[i]);
      while (word != 0u) {
        const int j = i * 32 + (int)__builtin_ctz(word);
        word &= word - 1u;
        const u64 k = exact_start(j);
        key = k > key ? k : key;
      }
    }
    return box_of(key);
  }

  // The box's sums in FP64 from its FP32 bins (every lane's result).
  __device__ __forceinline__ void sums(int jk, double &Rs, double &Ss) const {
    const int j = jk & 0xFFFF, k = jk >> 16;
    double r = 0.0, sg = 0.0;
    for (int m = lane; m < k; m += 64) {
      int c;
      const float2 e = bin(j + m, qscale, c);
      r = r + (double)e.x;
      sg = sg + (double)e.y;
    }
    Ss = wave_sum(sg);
    Rs = WEIGHTED ? wave_sum(r) : (double)points(high(U[j + k]), high(U[j]) - half);
  }
};

// WIDE: the copy for launches of at most four workgroups per CU, which have
// the registers of four waves per SIMD to themselves.  In the others' 80 (96
// weighted) VGPRs a period's set-up spills 31 (35), 21 GB of writes for 256
// x 50000 points x 100000 periods x 1000 bins; in 122 (128) none does.
// Narrow / wide: 24 x 50000 x 100000 x 1000 (0.005 to 0.05) 47.9 / 46.5 ms;
// weighted 24 x 20000 x 20000 x 700 8.5 / 8.3; but where the LDS leaves room
// for five or six, weighted 23 x 805 x 9306 x 585 1.53 / 1.74 and 158 x 1346 x
// 5016 x 218 1.98 / 2.52.
template <bool WEIGHTED, bool DIP, bool WIDE>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(WIDE ? 4 : WEIGHTED ? 5 : 6))) void block_search_kernel(
    SearchArgs a) {
  extern __shared__ __align__(16) u64 s_hist[];
  __shared__ double s_f[kTileMax];
  __shared__ CurveDesc s_cd;
  // the item's periods: the winning boxes' sums, the boxes
  __shared__ double s_S[kGroupMax];
  __shared__ double s_R[kGroupMax];
  __shared__ int s_jk[kGroupMax];
  __shared__ Claims s_claims;
  __shared__ long long s_item;
  __shared__ int s_curve;
  __shared__ int s_p0, s_gp0, s_gp1, s_t, s_edge;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int wpb = WEIGHTED ? 2 : 1;
  // Items and groups as in search_kernel: thread 0 claims one group ahead and
  // steps through the group's tiles.
  ItemRef nx = {-1, 0, 0};
  if (tid == 0) {
    claims_start(s_claims);
    nx = claim_item(a, s_claims);
    s_p0 = 0;
    s_t = 0;
    s_gp1 = 0;
  }

  for (;;) {
    if (tid == 0) {
      int p0 = s_p0 + s_t;
      int edge = 0;
      if (p0 >= s_gp1) {  // next group (groups are never empty)
        edge = 1;
        s_item = nx.item;
        s_curve = nx.curve;
        if (nx.item >= 0) {
          const CurveDesc *d = a.curves + nx.curve;
          const int G = d->group > 0 ? d->group : d->tile;
          const int gp0 = max(0, nx.tile * G - d->galign);
          s_t = d->tile;
          s_gp0 = gp0;
          s_gp1 = min(d->nperiods, (nx.tile + 1) * G - d->galign);
          p0 = gp0;
        }
      }
      if (p0 + s_t >= s_gp1) edge |= 2;  // last tile of the group
      s_p0 = p0;
      s_edge = edge;
    }
    __syncthreads();
    if (s_item < 0) break;
    const int c = __builtin_amdgcn_readfirstlane(s_curve);
    const int p0 = __builtin_amdgcn_readfirstlane(s_p0);
    const int edge = __builtin_amdgcn_readfirstlane(s_edge);
    const int gp0 = __builtin_amdgcn_readfirstlane(s_gp0);
    const int gp1 = __builtin_amdgcn_readfirstlane(s_gp1);
    if (tid == 0 && (edge & 1)) nx = claim_item(a, s_claims);
    // The curve's record, in LDS for the group: read where it is needed, its
    // fields do not occupy registers through the tile.
    if (edge & 1) {
      if (tid < (int)(sizeof(CurveDesc) / 4))
        reinterpret_cast<int *>(&s_cd)[tid] = reinterpret_cast<const int *>(a.curves + c)[tid];
      __syncthreads();
    }
    const CurveDesc &cd = s_cd;
    const int np = min(uniform(cd.tile), gp1 - p0);
    // Every item reaches the barrier at the end of the loop body (no
    // `continue`, see search_kernel).
    if (np <= 0) {
    } else if (uniform(cd.status) != kCurveOk) {
      for (int t = tid; t < np; t += kBlock) {
        const int64_t r = cd.r_off + p0 + t;
        a.sr[r] = NAN;
        a.depth[r] = NAN;
        a.jstart[r] = -1;
        a.kwidth[r] = -1;
      }
    } else {
      const int HS = uniform(cd.hstride);
      for (int i = tid; i < np * HS * wpb; i += kBlock) s_hist[i] = 0ull;
      if (tid < np) s_f[tid] = 1.0 / a.periods[cd.p_off + p0 + tid];
      __syncthreads();
      CurveDesc fd;  // what the fold reads of it
      fd.n_off = uniform_i64(cd.n_off);
      fd.n = uniform_i64(cd.n);
      fd.nbins = uniform(cd.nbins);
      fd.shift = uniform(cd.shift);
      const int64_t n = fd.n;
      const double ftile = fmin(s_f[0], s_f[np - 1]);
      const int gap = uniform(fold_lane_gap(ftile, fd.nbins, cd.cadence));
      const bool merge =
          uniform((int)fold_merges(ftile, fd.nbins, cd.cadence, a.fold_policy, WEIGHTED, 0.15)) !=
          0;
      const int64_t nchunks = n / (kBlock * kPPT), base = nchunks * (kBlock * kPPT);
      if (nchunks > 0) {
        if (merge)
          fold_chunks<WEIGHTED, true>(a, fd, nchunks, np, s_f, s_hist, HS, gap);
        else
          fold_chunks<WEIGHTED, false>(a, fd, nchunks, np, s_f, s_hist, HS, gap);
      }
      // The rest: merged, or 64 kPPT points a wave as long as they last.
      const int64_t first = base + wave * 64 * kPPT;
      if (merge) {
        if (base < n)
          fold_rest<WEIGHTED, true>(a, fd, base, (int)(n - base), np, s_f, s_hist, HS);
      } else if (first + 64 * kPPT <= n)
        fold_chunk<WEIGHTED, false>(a, fd, base, np, s_f, s_hist, HS, 1);
      else if (first < n)
        fold_tail<WEIGHTED>(a, fd, first, (int)(n - first), np, s_f, s_hist, HS);
      __syncthreads();
      // One wave per period.
      unsigned char *scr = reinterpret_cast<unsigned char *>(s_hist) + uniform(cd.scr_offset) +
                           wave * uniform(cd.scr_bytes);
      for (int t = wave; t < np; t += kBlock / 64) {
        u64 *u = s_hist + (size_t)t * HS * wpb;
        PeriodScan<WEIGHTED, DIP> ps(cd, a.min_in_points, u, u + HS, scr);
        int jk = __builtin_amdgcn_readfirstlane(ps.best());
        if (jk == kMarked) {
          // (the curve's record is read again: what only this needs of it
          // occupies no registers through the search)
          wave_sync();
          const PeriodScan<WEIGHTED, DIP> es(cd, a.min_in_points, u, u + HS, scr);
          jk = __builtin_amdgcn_readfirstlane(es.marked_starts());
        }
        double Rs = 0.0, Ss = 0.0;
        if (jk >= 0) ps.sums(jk, Rs, Ss);
        if ((tid & 63) == 0) {
          const int g = p0 + t - gp0;
          s_S[g] = Ss;
          s_R[g] = Rs;
          s_jk[g] = jk;
        }
      }
      // After the group's last tile: statistic and depth of its periods, the
      // results written out together, and one update of the curve's best key.
      if (edge & 2) {
        __syncthreads();
        const int ng = gp1 - gp0;
        u64 key = 0ull;
        if (tid < ng) {
          const int jk = s_jk[tid];
          const int p = gp0 + tid;
          float srf = 0.0f, dpf = NAN;
          int j = -1, k = -1;
          if (jk >= 0) {
            const double W = cd.Wtot;
            const double R = s_R[tid];
            const double S = s_S[tid];
            const double den = R * (W - R);
            srf = (float)(sqrt(S * S / den) * cd.out_scale);
            dpf = (float)(-S * W / den * cd.out_scale);
            j = jk & 0xFFFF;
            k = jk >> 16;
          }
          const int64_t r = cd.r_off + p;
          a.sr[r] = srf;
          a.depth[r] = dpf;
          a.jstart[r] = j;
          a.kwidth[r] = k;
          key = ((u64)__float_as_uint(srf) << 32) | (u64)(0xFFFFFFFFu - (unsigned)p);
        }
        if (tid < 64) {  // groups hold at most 32 periods
#pragma unroll
          for (int o = 16; o > 0; o >>= 1) {
            const u64 y = __shfl_xor(key, o, 64);
            key = y > key ? y : key;
          }
          if (tid == 0)
            __hip_atomic_fetch_max(a.best_key + c, key, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    __syncthreads();
  }
}

template <bool WEIGHTED, bool DIP, bool WIDE>
const void *block_fn() {
  return reinterpret_cast<const void *>(&block_search_kernel<WEIGHTED, DIP, WIDE>);
}

}  // namespace

const void *block_search_fn(bool weighted, bool dip, bool wide) {
  if (weighted) {
    if (wide) return dip ? block_fn<true, true, true>() : block_fn<true, false, true>();
    return dip ? block_fn<true, true, false>() : block_fn<true, false, false>();
  }
  if (wide) return dip ? block_fn<false, true, true>() : block_fn<false, false, true>();
  return dip ? block_fn<false, true, false>() : block_fn<false, false, false>();
}

}  // namespace bls
