// gfx950 kernel of the unbinned box search (box edges between data points,
// a range of durations and phases taken to the data, section 2.2.2).
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "bls_block.h"
#include "bls_device.h"
#include "bls_items.h"
#include "../../include/bls.h"

namespace bls {
namespace {

// ------------------------------------------------------ unbinned search
// Box edges between data points: per period the kept points are put in
// phase order (ties by index) and every cyclic run that some box with duty
// cycle in [qlo, qhi] holds exactly is scored.  The order is found without a
// comparison sort: a counting sort on a fine phase grid (about one point per
// cell) groups the points, and each point's rank is its cell's start plus
// the number of cell mates that precede it.  Sums over a run are exact:
// differences of FP64 prefix sums of the integer fixed-point values of the
// prep pass, all below 2^53.  The runs are screened by pairs of blocks of
// 8 or 16 starts and ends, then of kUnbSub starts and ends: one bound from
// the blocks' extreme prefix sums rejects most pairs, and only the runs of
// the pairs left are scored.
//
// What bounds it, and what it measured against the walk over every start's
// ends, eight at a time, that the screens replace.  8 curves of 1000 points x
// 5000 periods: 1.79 / 1.03 ms, instruction issue (10000 wave instructions a
// period, of which the walk alone took that many; two thirds now the screens,
// one third the sort).  2 curves of 20000 points x 1500 periods: 31.0 / 2.67
// ms, latency of the workspace: the sort with its cell counts in device
// memory took two thirds of the time, and now, the counts in LDS and four
// points of a thread in flight, about half.

__host__ __device__ inline int pow2_at_least(int n) {
  int m = 1;
  while (m < n) m <<= 1;
  return m;
}

// Array stride of the per-point arrays for curves of up to n points: a
// multiple of four, so that four values are 16-byte aligned in every array,
// and at least 112, so that the blocks' table (60 bytes per block of 8 ranks)
// fits the arrays it takes over.
__host__ __device__ inline int unbinned_stride(int n) { return n < 112 ? 112 : (n + 3) & ~3; }

// Ints after the weights, for the last block's part of the table.
constexpr int kUnbPad = 16;

// Ranks per small block of run starts or ends.
constexpr int kUnbSub = 4;

// Where the screens' threshold starts: below the value of any run that holds a
// signal (|S| >= 1 and R (W - R) < 2^102 in the integers' units), so that runs
// without one never pass, and its product with any R (W - R) is a normal float.
// From 0 all of them would: 20000 points of one flux took 124 ms for 64 periods
// (0.4 ms so; curves with a signal the same).
constexpr float kUnbThetaMin = 0x1p-110f;

// Bounds as floats, wide enough for the float arithmetic on them: sums and
// differences of a few such values and of cycle totals up to t.
__device__ inline float at_least(double v, float t) {
  const float f = (float)v;
  return fmaf(fabsf(f) + t, 0x1p-22f, f);
}
__device__ inline float at_most(double v, float t) {
  const float f = (float)v;
  return fmaf(fabsf(f) + t, -0x1p-22f, f);
}

// Forward phase distance from sorted position i (phase pi) to j (phase pj),
// one cycle added when the step passes the end of the order.
__device__ inline double fwd_phase(double pi, double pj, int i, int j) {
  return j > i ? pj - pi : (pj + 1.0) - pi;
}

// Inclusive sum over the wave's lanes.
__device__ inline double wave_scan(double v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}

// MODE (unbinned_mode): where the per-point arrays are.
template <bool WEIGHTED, bool DIP, int MODE>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(4))) void unbinned_kernel(SearchArgs a) {
  extern __shared__ __align__(16) unsigned char s_lds[];
  __shared__ Claims s_claims;
  __shared__ long long s_item;
  __shared__ int s_curve;
  __shared__ int s_per;
  __shared__ unsigned long long s_vbits;
  __shared__ unsigned int s_theta;
  __shared__ unsigned int s_tie;
  __shared__ long long s_wsum[kBlock / 64];
  __shared__ double s_wtot[2 * (kBlock / 64)];
  __shared__ int s_part[kBlock / 64];
  // per wave: the block pairs that pass the first screen and the second, by
  // their first start and end
  __shared__ int2 s_pairs[(kBlock / 64) * (64 + 16)];
  __shared__ int2 s_subs[(kBlock / 64) * (64 + 4)];

  // Ranks per large block.  With 16, a quarter of the pairs pass the first
  // screen on curves of 1000 points (8: a fourteenth) and the second costs
  // more than it saves; long curves have more pairs, and few pass.
  constexpr int kBlk = MODE == kUnbLds ? 8 : 16;
  constexpr bool kPacked = MODE == kUnbLds;  // block offsets: 16 bits each
  constexpr int kK = kBlk / kUnbSub, kPer = 64 / (kK * kK);  // pairs at a time

  const int tid = threadIdx.x;
  const int N = unbinned_stride(a.ucap);
  unsigned char *s_raw = MODE != kUnbLds ? a.uws + (int64_t)blockIdx.x * a.uws_stride : s_lds;
  double *sph = reinterpret_cast<double *>(s_raw);  // phases in order
  double *cph = sph + N;                            // phases grouped by cell
  int *sidx = reinterpret_cast<int *>(cph + N);
  int *sq = sidx + N;
  int *sw = sq + N;  // weighted only
  int *grp = sw + (WEIGHTED ? N + kUnbPad : 0);
  int *cnt = MODE == kUnbCells ? reinterpret_cast<int *>(s_lds) : grp + N;
  // After the ranking: the prefix sums of the values over the grouped phases,
  // those of the weights over grp and the cell counts (weighted; unit weights
  // keep the cell counts, which place the longest runs), and the blocks'
  // table over the values and the next array (the weights or grp), 8 bytes
  // per point; where the cell counts are in LDS by themselves, the large
  // blocks' extremes take their place.
  double *Pq = cph;
  double *Pw = reinterpret_cast<double *>(grp);
  float2 *tab = reinterpret_cast<float2 *>(sq);

  ItemRef nx = {-1, 0, 0};
  if (tid == 0) {
    claims_start(s_claims);
    nx = claim_item(a, s_claims);  // one item ahead
  }
  for (;;) {
    if (tid == 0) {
      s_item = nx.item;
      s_curve = nx.curve;
      s_per = nx.tile;
    }
    __syncthreads();
    if (s_item < 0) break;
    const int c = __builtin_amdgcn_readfirstlane(s_curve);
    const int p = __builtin_amdgcn_readfirstlane(s_per);
    __syncthreads();
    if (tid == 0) nx = claim_item(a, s_claims);

    const CurveDesc cd = a.curves[c];
    const int64_t r_out = cd.r_off + p;
    // Every item, valid or not, reaches the one barrier at the end of the
    // loop body: a `continue` here would give the loop header a second way
    // in that skips thread 0's fetch, and the compiler may then keep the
    // other lanes circling the header barrier without thread 0.
    if (cd.status != kCurveOk) {
      if (tid == 0) {
        a.sr[r_out] = NAN;
        a.depth[r_out] = NAN;
        a.jstart[r_out] = -1;
        a.kwidth[r_out] = -1;
      }
    } else {
    const int n = (int)cd.n;
    const int M = MODE == kUnbCells ? min(pow2_at_least(n), kUnbMaxCells) : pow2_at_least(n);
    const double Md = (double)M;
    const double f = 1.0 / a.periods[cd.p_off + p];
    const double *dt = a.dt + cd.n_off;
    const int32_t *q = a.q + cd.n_off;
    const int32_t *qw = WEIGHTED ? a.qw + cd.n_off : nullptr;
    const int lane = tid & 63, wave = tid >> 6;
    auto cell_of = [&](double ph) { return (int)min((unsigned)(int)(ph * Md), (unsigned)(M - 1)); };

    // Phases and fine-grid cells; dropped points go to the extra cell M.
    // (Four points a thread at a time: their loads go out together.)
    constexpr int kU = 4;
    for (int i = tid; i <= M; i += kBlock) cnt[i] = 0;
    if (tid == 0) {
      s_vbits = 0ull;
      s_theta = __float_as_uint(kUnbThetaMin);
      s_tie = 0xFFFFFFFFu;
    }
    __syncthreads();
    long long wsum = 0;
    for (int i0 = tid; i0 < n; i0 += kU * kBlock) {
      double d[kU];
      int w[kU];
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        const int i = min(i0 + k * kBlock, n - 1);
        d[k] = dt[i];
        w[k] = WEIGHTED ? qw[i] : 0;
      }
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        if (i0 + k * kBlock >= n) break;
        atomicAdd(&cnt[w[k] >= 0 ? cell_of(__builtin_amdgcn_fract(d[k] * f)) : M], 1);
        if (WEIGHTED && w[k] >= 0) wsum += w[k];
      }
    }
    __syncthreads();
    // Exclusive scan of the M + 1 cell counts: a run of cells per thread,
    // a scan of the run totals across each wave, then across the waves.
    {
      const int per = (M + 1 + kBlock - 1) / kBlock;
      const int b0 = min(M + 1, tid * per), b1 = min(M + 1, b0 + per);
      int run = 0;
      for (int b = b0; b < b1; ++b) run += cnt[b];
      int x = run;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (lane == 63) s_part[wave] = x;
      __syncthreads();
      int acc = x - run;
      for (int w = 0; w < wave; ++w) acc += s_part[w];
      for (int b = b0; b < b1; ++b) {
        const int v = cnt[b];
        cnt[b] = acc;
        acc += v;
      }
    }
    __syncthreads();
    // Scatter into cells (any order inside a cell); cnt becomes cell ends.
    for (int i0 = tid; i0 < n; i0 += kU * kBlock) {
      double d[kU];
      int w[kU];
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        const int i = min(i0 + k * kBlock, n - 1);
        d[k] = dt[i];
        w[k] = WEIGHTED ? qw[i] : 0;
      }
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        const int i = i0 + k * kBlock;
        if (i >= n) break;
        const double ph = __builtin_amdgcn_fract(d[k] * f);
        const int at = atomicAdd(&cnt[w[k] >= 0 ? cell_of(ph) : M], 1);
        cph[at] = ph;
        grp[at] = i;
      }
    }
    long long W = 0;
    if (WEIGHTED) {
      for (int o = 32; o > 0; o >>= 1) wsum += __shfl_xor(wsum, o, 64);
      if (lane == 0) s_wsum[wave] = wsum;
    }
    __syncthreads();
    const int nk = cnt[M - 1];  // kept points come first
    if (WEIGHTED) {
      for (int k = 0; k < kBlock / 64; ++k) W += s_wsum[k];
    } else {
      W = nk;
    }
    const double Wd = (double)W;
    const double qlo = cd.qlo, qhi = cd.qhi;
    // Rank = cell start + cell mates before this point in (phase, index).
    // A thread per place in the grouped order (four at a time): a cell's
    // mates are its neighbours.  The indices are compared only where phases
    // are equal.
    for (int at0 = tid; at0 < nk; at0 += kU * kBlock) {
      double ph[kU];
      int id[kU], v[kU], w[kU], b[kU], e[kU], rank[kU], most = 0;
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        const int at = min(at0 + k * kBlock, nk - 1);
        ph[k] = cph[at];
        id[k] = grp[at];
      }
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        const int cell = cell_of(ph[k]);
        v[k] = q[id[k]];
        w[k] = WEIGHTED ? qw[id[k]] : 0;
        b[k] = cell == 0 ? 0 : cnt[cell - 1];
        e[k] = cnt[cell];
        rank[k] = b[k];
        most = max(most, e[k] - b[k]);
      }
      for (int m = 0; m < most; ++m) {
        double pj[kU];
#pragma unroll
        for (int k = 0; k < kU; ++k) pj[k] = cph[min(b[k] + m, e[k] - 1)];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
          const int j = b[k] + m;
          bool before = pj[k] < ph[k];
          if (pj[k] == ph[k] && j != at0 + k * kBlock && j < e[k]) before = grp[j] < id[k];
          rank[k] += (int)(before & (j < e[k]));
        }
      }
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        if (at0 + k * kBlock >= nk) break;
        sph[rank[k]] = ph[k];
        sq[rank[k]] = v[k];
        sidx[rank[k]] = id[k];
        if (WEIGHTED) sw[rank[k]] = w[k];
      }
    }
    __syncthreads();

    // Prefix sums in phase order, Pq[i] = q summed over ranks 0..i (and Pw
    // for the weights), in FP64: every partial sum is an integer below 2^53
    // (|q|, w < 2^31 and at most 2^20 points), so each is exact and a run's
    // sum is a difference of two of them, exact as well.  A wave takes a
    // quarter of the ranks, four to a lane at a time: its total, then, the
    // totals before it known, the running sums.
    {
      const int len = (nk + 4 * kBlock - 1) / (4 * kBlock) * kBlock;
      const int cb = min(nk, wave * len), ce = min(nk, cb + len);
      auto four = [&](const int *v, int i, double *d) {  // d: running sums of v[i..i+3]
        int4 x = make_int4(0, 0, 0, 0);
        if (i < ce) x = *reinterpret_cast<const int4 *>(v + i);
        d[0] = (double)x.x;
        d[1] = d[0] + (i + 1 < ce ? (double)x.y : 0.0);
        d[2] = d[1] + (i + 2 < ce ? (double)x.z : 0.0);
        d[3] = d[2] + (i + 3 < ce ? (double)x.w : 0.0);
      };
      double tq = 0.0, tw = 0.0, d[4];
      for (int i = cb + lane * 4; i < ce; i += 256) {
        four(sq, i, d);
        tq += d[3];
        if (WEIGHTED) {
          four(sw, i, d);
          tw += d[3];
        }
      }
      tq = wave_scan(tq, lane);
      if (WEIGHTED) tw = wave_scan(tw, lane);
      if (lane == 63) {
        s_wtot[wave] = tq;
        if (WEIGHTED) s_wtot[kBlock / 64 + wave] = tw;
      }
      __syncthreads();
      double rq = 0.0, rw = 0.0;
      for (int w = 0; w < wave; ++w) {
        rq += s_wtot[w];
        if (WEIGHTED) rw += s_wtot[kBlock / 64 + w];
      }
      auto put = [&](double *P, const int *v, int i, double &run) {
        four(v, i, d);
        const double x = wave_scan(d[3], lane);
        const double before = run + (x - d[3]);
        if (i < ce) {  // (ranks past the last hold the total)
          *reinterpret_cast<double2 *>(P + i) = make_double2(before + d[0], before + d[1]);
          *reinterpret_cast<double2 *>(P + i + 2) = make_double2(before + d[2], before + d[3]);
        }
        run += __shfl(x, 63, 64);
      };
      for (int i0 = cb; i0 < ce; i0 += 256) {
        put(Pq, sq, i0 + lane * 4, rq);
        if (WEIGHTED) put(Pw, sw, i0 + lane * 4, rw);
      }
    }
    __syncthreads();
    const double Tq = nk > 0 ? Pq[nk - 1] : 0.0;
    const double Tw = WEIGHTED ? (nk > 0 ? Pw[nk - 1] : 0.0) : Wd;
    const float Tqf = (float)Tq, Tabs = fabsf(Tqf) * 2.0f;

    auto spans_less = [&](int r, double ph_r, int u) {  // end u unwrapped
      const int e = u >= nk ? u - nk : u;
      return fwd_phase(ph_r, sph[e], r, e) < qhi;
    };
    // Phase of an unwrapped rank, a cycle added past the end of the order.
    auto phase_at = [&](int x) { return x >= nk ? sph[x - nk] + 1.0 : sph[x]; };
    // The ends that runs from ranks a0..a1 can have lie between these two:
    // the first such that the points around the run are more than qlo apart,
    // and the last such that the run spans less than qhi (with a margin for
    // the rounding of the phase differences; a run of one point spans
    // nothing, and runs hold at most nk - 1 points).  With unit weights the
    // cells of the sort give them, to a cell; weighted curves have no room
    // left for the cell counts and bisect.
    auto first_end = [&](int a0) {
      const double t = (a0 == 0 ? sph[nk - 1] - 1.0 : sph[a0 - 1]) + (qlo - 0x1p-48);
      int u = a0;
      if (WEIGHTED) {
        int hi = a0 + nk - 1;  // least u with the phase after it above t
        while (u < hi) {
          const int mid = (u + hi) >> 1;
          if (phase_at(mid + 1) > t)
            hi = mid;
          else
            u = mid + 1;
        }
      } else if (t >= 0.0) {
        const bool wr = t >= 1.0;
        const int cell = cell_of(wr ? t - 1.0 : t);
        u = (cell == 0 ? 0 : cnt[cell - 1]) + (wr ? nk : 0) - 1;
      }
      return max(u, a0);
    };
    auto last_end = [&](int a1) {
      const double t = sph[a1] + (qhi + 0x1p-48);
      int u = a1, hi = a1 + nk - 2;
      if (WEIGHTED) {
        while (u < hi) {
          const int mid = (u + hi + 1) >> 1;
          if (phase_at(mid) < t)
            u = mid;
          else
            hi = mid - 1;
        }
      } else {
        const bool wr = t >= 1.0;
        u = min(cnt[cell_of(wr ? t - 1.0 : t)] - 1 + (wr ? nk : 0), hi);
      }
      return max(u, a1);
    };

    // Blocks of kBlk consecutive ranks (the last one shorter) and of
    // kUnbSub.  Table: the largest and smallest prefix sum over the ranks as
    // run ends (e; for the large blocks also a cycle on), and as run starts
    // (b: the prefix before the rank), the least weight, and the offsets to
    // the first and the last block with ends of the block's runs.
    const int NB = (nk + kBlk - 1) / kBlk, NS = NB * (kBlk / kUnbSub);
    float2 *eS = tab, *gS = eS + NS, *gB = gS + NS;
    float2 *eB = MODE == kUnbCells ? reinterpret_cast<float2 *>(cnt) : gB + NB;
    int *ends = reinterpret_cast<int *>(MODE == kUnbCells ? gB + NB : eB + 2 * NB);
    int *wB = ends + (kPacked ? NB : 2 * NB);  // weighted only
    for (int A = tid; A < NB; A += kBlock) {
      const int a0 = A * kBlk, u0 = first_end(a0), u1 = last_end(min(a0 + kBlk, nk) - 1);
      const int o0 = (u0 < nk ? u0 / kBlk : NB + (u0 - nk) / kBlk) - A;
      const int o1 = (u1 < nk ? u1 / kBlk : NB + (u1 - nk) / kBlk) - A;
      if (kPacked) {
        ends[A] = o0 | o1 << 16;
      } else {
        ends[2 * A] = o0;
        ends[2 * A + 1] = o1;
      }
    }
    if (MODE == kUnbCells) __syncthreads();
    // (a thread per small block, joined across its large block's; a run does not
    // split equal phases, so ranks after an equal phase are not starts and
    // ranks before one no ends: a block without any has NaN extremes, which no
    // pair passes)
    for (int i0 = 0; i0 < NS; i0 += kBlock) {
      const int i = i0 + tid, r0 = i * kUnbSub;
      double hi = -INFINITY, lo = INFINITY, bhi = -INFINITY, blo = INFINITY;
      int wm = 0x7fffffff;
      // (the block's four ranks and their neighbours, loaded together)
      const int rc = min(r0, (nk - 1) & ~(kUnbSub - 1)), rb = max(rc - 1, 0);
      const double2 p0 = *reinterpret_cast<const double2 *>(sph + rc),
                    p1 = *reinterpret_cast<const double2 *>(sph + rc + 2),
                    v0 = *reinterpret_cast<const double2 *>(Pq + rc),
                    v1 = *reinterpret_cast<const double2 *>(Pq + rc + 2);
      const double ph[kUnbSub + 1] = {p0.x, p0.y, p1.x, p1.y, sph[min(rc + kUnbSub, nk - 1)]};
      const double v[kUnbSub] = {v0.x, v0.y, v1.x, v1.y};
      double before = rc > 0 ? Pq[rb] : 0.0;
      double wbefore = WEIGHTED && rc > 0 ? Pw[rb] : 0.0;
      bool start = rc == 0 || sph[rb] < ph[0];
#pragma unroll
      for (int k = 0; k < kUnbSub; ++k) {
        const int r = r0 + k;
        if (r < nk) {
          const bool end = r == nk - 1 || ph[k] < ph[k + 1];
          if (end) {
            hi = fmax(hi, v[k]);
            lo = fmin(lo, v[k]);
          }
          if (start) {
            bhi = fmax(bhi, before);
            blo = fmin(blo, before);
          }
          start = end;
          before = v[k];
          if (WEIGHTED) {
            const double w = Pw[r];
            wm = min(wm, (int)(w - wbefore));
            wbefore = w;
          }
        }
      }
      float2 e = make_float2(at_least(hi, Tabs), at_most(lo, Tabs));
      float2 g = make_float2(at_least(bhi, Tabs), at_most(blo, Tabs));
      if (i < NS) {
        eS[i] = e;
        gS[i] = g;
      }
#pragma unroll
      for (int o = 1; o < kK; o <<= 1) {
        e.x = fmaxf(e.x, __shfl_xor(e.x, o, 64));
        e.y = fminf(e.y, __shfl_xor(e.y, o, 64));
        g.x = fmaxf(g.x, __shfl_xor(g.x, o, 64));
        g.y = fminf(g.y, __shfl_xor(g.y, o, 64));
        if (WEIGHTED) wm = min(wm, __shfl_xor(wm, o, 64));
      }
      if (i < NS && i % kK == 0) {
        eB[i / kK] = e;
        eB[NB + i / kK] = make_float2(e.x + Tqf, e.y + Tqf);
        gB[i / kK] = g;
        if (WEIGHTED) wB[i / kK] = wm;
      }
    }
    __syncthreads();

    // A run of L points from start r has S = P(r + L - 1) - P(r - 1) and
    // R = L (or the same difference of the weight sums), exact, as above.
    // Runs are screened against theta, the best value any lane of the
    // workgroup has found so far in this period (s_theta holds it relaxed, as
    // a float of at most theta (1 - 2^-20), raised as lanes improve; the
    // lanes' final bests go to s_vbits): a run with S^2 < theta (1 - 2^-20)
    // R (W - R) can be neither the best nor a tie of it.
    double bnum = 0.0, bden = 1.0;
    unsigned int btie = 0xFFFFFFFFu;
    float thr = kUnbThetaMin;
    bool raised = false;  // thr since the last publish()
    auto reload_theta = [&]() {  // (any value read is one some run reached)
      const unsigned tb =
          __hip_atomic_load(&s_theta, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      thr = fmaxf(thr, __uint_as_float(tb));
    };
    // Run from r to the unwrapped end e >= r: the exact comparison, without a
    // division (S^2 / den against the lane's best as cross products), and the
    // admissibility of the edges.
    auto score = [&](int r, int e, double S, double R) {
      const int L = e - r + 1;
      if (DIP && !(S < 0.0)) return;
      const double den = R * (Wd - R);
      const double num = S * S;
      if (num < (double)thr * den) return;
      // Rare: the run passed the screen; its edges must be admissible.
      const int prev = r == 0 ? nk - 1 : r - 1;
      const double ph_r = sph[r], ph_prev = sph[prev];
      if (!(fwd_phase(ph_prev, ph_r, prev, r) > 0.0)) return;
      if (L >= nk || !(L == 1 || spans_less(r, ph_r, e))) return;
      const int x = e >= nk ? e - nk : e;
      const int next = x + 1 == nk ? 0 : x + 1;
      const double pe = sph[x], pn = sph[next];
      if (!(fwd_phase(pe, pn, x, next) > 0.0)) return;
      const double gap = prev == next ? 1.0 : fwd_phase(ph_prev, pn, prev, next);
      if (!(gap > qlo)) return;
      if (L < a.min_in_points) return;
      if (!(den > 0.0) || S == 0.0) return;
      const double lhs = num * bden, rhs = bnum * den;
      const unsigned int tie = (unsigned)L * (unsigned)nk + (unsigned)r;
      if (lhs > rhs || (lhs == rhs && tie < btie)) {
        bnum = num;
        bden = den;
        btie = tie;
        thr = fmaxf(thr, (float)(num / den) * (1.0f - 0x1p-19f));  // relaxed
        raised = true;
      }
    };
    // The wave's largest theta, to its lanes and the workgroup (by one lane:
    // an atomic of many lanes becomes a loop over them).
    auto publish = [&]() {
      if (__builtin_amdgcn_ballot_w64(raised) != 0ull) {
        const unsigned top = wave_umax(__float_as_uint(thr));
        if (lane == 0)
          __hip_atomic_fetch_max(&s_theta, top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        thr = __uint_as_float(top);
        raised = false;
      }
      reload_theta();
    };
    const float Wf = (float)Wd;
    // Whether some run from starts r0..r1 to ends f..l may beat theta: |S| is
    // at most the largest difference of their prefix sums (only negative S
    // for dips), and R (W - R) is concave in R, so its least value is at the
    // least or the largest R.  cq: one cycle's total past the end of the
    // order; R1, R2: least and largest R.  In FP32: the extremes are wide
    // enough, and the roundings of the rest are within theta's 2^-20.
    auto may_beat = [&](float2 e, float2 g, float cq, auto R1, auto R2) {
      const float dn = g.x - (e.y + cq);
      const float sm = DIP ? fmaxf(dn, 0.0f) : fmaxf((e.x + cq) - g.y, dn);
      float den;
      if (WEIGHTED)
        den = (float)fmin(R1 * (Wd - R1), R2 * (Wd - R2));
      else
        den = fminf((float)R1 * (Wf - (float)R1), (float)R2 * (Wf - (float)R2));
      return sm * sm >= thr * den;
    };
    // Weight before rank r, and up to rank x; unit weights: their number.
    using Sum = std::conditional_t<WEIGHTED, double, int>;
    auto before_rank = [&](int r) -> Sum {
      if constexpr (WEIGHTED) return r == 0 ? 0.0 : Pw[r - 1];
      else return r;
    };
    auto up_to = [&](int x) -> Sum {
      if constexpr (WEIGHTED) return Pw[x];
      else return x + 1;
    };
    const Sum cycle = WEIGHTED ? (Sum)Tw : (Sum)nk;
    auto base_at = [&](int r) { return r == 0 ? 0.0 : Pq[r - 1]; };
    auto run_at = [&](int r, int e) {  // scores a run, if there is such a run
      if (r < 0 || r >= nk || e < r || e >= r + nk - 1) return;
      const bool wr = e >= nk;
      const int x = wr ? e - nk : e;
      score(r, e, Pq[x] + (wr ? Tq : 0.0) - base_at(r),
            (double)(up_to(x) + (wr ? cycle : (Sum)0) - before_rank(r)));
    };
    int2 *pairs = s_pairs + wave * (64 + 16);
    int2 *subs = s_subs + wave * (64 + 4);
    int npairs = 0, nsubs = 0;
    const unsigned long long below = (1ull << lane) - 1ull;
    auto push = [&](int2 *list, int &n, unsigned long long m, bool mine, int r, int e) {
      if (mine) list[n + (int)__popcll(m & below)] = make_int2(r, e);
      n = __builtin_amdgcn_readfirstlane(n + (int)__popcll(m));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    // The runs of four queued small pairs (or what is left), a lane each.
    auto score_subs = [&]() {
      const int cnt = min(nsubs, 4), q = lane >> 4;
      nsubs = __builtin_amdgcn_readfirstlane(nsubs - cnt);
      if (q < cnt) {
        const int2 s = subs[nsubs + q];
        const int r = s.x + (lane & 3), e = s.y + ((lane >> 2) & 3);
        if (s.y >= nk || e < nk) run_at(r, e);
      }
      __builtin_amdgcn_wave_barrier();
      publish();
    };
    // The second screen of kPer queued pairs, a lane per pair of small blocks.
    auto screen_pairs = [&]() {
      const int cnt = min(npairs, kPer), q = lane / (kK * kK);
      npairs = __builtin_amdgcn_readfirstlane(npairs - cnt);
      const int2 pr = pairs[npairs + min(q, cnt - 1)];
      const int r0 = pr.x + (lane % kK) * kUnbSub;
      const int e0 = pr.y + (lane / kK % kK) * kUnbSub;
      const bool wr = pr.y >= nk;
      const int x0 = wr ? e0 - nk : e0;
      const bool in = (q < cnt) & (r0 < nk) & (x0 < nk);
      const int rc = min(r0, nk - 1), xc = min(x0, nk - 1);
      const int r1 = min(rc + kUnbSub, nk) - 1, x1 = min(xc + kUnbSub, nk) - 1;
      const Sum cs = wr ? cycle : (Sum)0;
      const Sum R1 =
          max(up_to(xc) + cs - before_rank(r1), WEIGHTED ? (Sum)wB[rc / kBlk] : (Sum)1);
      const Sum R2 = up_to(x1) + cs - before_rank(rc);
      bool ok = in & (e0 + kUnbSub > r0) &
                may_beat(eS[xc / kUnbSub], gS[rc / kUnbSub], wr ? Tqf : 0.0f, R1, R2);
      if (__builtin_amdgcn_ballot_w64(ok) == 0ull) return;
      // Too wide: the narrowest run spans qhi; too narrow: the points around
      // the widest are within qlo (both with a margin for the rounding of the
      // phase differences).
      const double c = wr ? 1.0 : 0.0;
      const double after = x1 + 1 == nk ? sph[0] + 1.0 : sph[x1 + 1];
      const double before = rc == 0 ? sph[nk - 1] - 1.0 : sph[rc - 1];
      ok = ok & ((e0 <= r1) | (sph[xc] + c - sph[r1] < qhi + 0x1p-48)) &
           (after + c - before > qlo - 0x1p-48);
      const unsigned long long m = __builtin_amdgcn_ballot_w64(ok);
      if (m != 0ull) push(subs, nsubs, m, ok, r0, e0);
    };
    // The two screens' queues worked off: all of it, or what fills a step.
    auto drain = [&](bool all) {
      for (;;) {
        if (nsubs >= 4 || (all && npairs == 0 && nsubs > 0))
          score_subs();
        else if (npairs >= kPer || (all && npairs > 0))
          screen_pairs();
        else
          break;
      }
    };
    // Two passes over the pairs (start block A, a lane each; end block A + o,
    // the waves taking the offsets in turn).  The first looks at every other
    // offset (every fourth of many) for the pair with the largest bound, R
    // taken between the blocks' middles: the runs of each wave's best pair
    // give a good theta.  The second bounds every pair, and those that pass
    // once more by small blocks, kPer pairs at a time.
    for (int pass = 0; pass < 2; ++pass) {
      float top = 0.0f;
      int top_r = 0, top_o = 0;
      for (int A0 = 0; A0 < NB; A0 += 64) {
        const bool live = A0 + lane < NB;
        const int A = live ? A0 + lane : NB - 1;
        const int a0 = A * kBlk, a1 = min(a0 + kBlk, nk) - 1;
        const int oA = kPacked ? ends[A] & 0xFFFF : ends[2 * A];
        const int oZ = kPacked ? ends[A] >> 16 : ends[2 * A + 1];
        const int omin = 0xFFFFFF - (int)wave_umax(0xFFFFFF - oA);
        const int omax = (int)wave_umax(oZ);
        const unsigned span = live && oZ >= oA ? oZ - oA + 1 : 0;
        const Sum w0 = before_rank(a0), w1 = before_rank(a1);
        const Sum wl = WEIGHTED ? (Sum)wB[A] : (Sum)1;
        const float2 g = gB[A];
        const int step = (pass != 0 ? 1 : omax - omin >= 32 ? 4 : 2) * (kBlock / 64);
        for (int o = omin + wave; o <= omax; o += step) {
          const int B = min(A + o, 2 * NB - 1);
          const bool wr = B >= NB;
          const float2 e = eB[B];
          const float dn = g.x - e.y;
          const float sm = DIP ? fmaxf(dn, 0.0f) : fmaxf(e.x - g.y, dn);
          const bool in = (unsigned)(o - oA) < span;
          float den;
          if (WEIGHTED) {
            const int f = (wr ? B - NB : B) * kBlk, l = min(f + kBlk, nk) - 1;
            const Sum cw = wr ? cycle : (Sum)0;
            const Sum R1 = max(up_to(f) + cw - w1, wl), R2 = up_to(l) + cw - w0;
            den = pass == 0 ? 0.25f * (float)(R1 + R2) * (float)(2.0 * Wd - (R1 + R2))
                            : (float)fmin(R1 * (Wd - R1), R2 * (Wd - R2));
          } else {
            // (of full blocks, less the ranks that the last one lacks where
            // the run passes it: uniform but for that)
            const int R = o * kBlk - (wr ? NB * kBlk - nk : 0);
            const float R1 = (float)max(R - kBlk + 2, 1), R2 = (float)(R + kBlk);
            den = pass == 0 ? (float)(R + 1) * (Wf - (float)(R + 1))
                            : fminf(R1 * (Wf - R1), R2 * (Wf - R2));
          }
          if (pass == 0) {
            const float v = sm * sm * __builtin_amdgcn_rcpf(den);
            if (in & (den > 0.0f) & (v > top)) {
              top = v;
              top_r = a0;
              top_o = o;
            }
            continue;
          }
          reload_theta();
          const bool hit = in & (sm * sm >= thr * den);
          const unsigned long long m = __builtin_amdgcn_ballot_w64(hit);
          if (m == 0ull) continue;
          push(pairs, npairs, m, hit, a0, B * kBlk - (wr ? NB * kBlk - nk : 0));
          drain(false);
        }
      }
      if (pass == 0) {
        const float t = __uint_as_float(wave_umax(__float_as_uint(top)));
        if (t > 0.0f) {  // this wave's best pair
          const int l = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(top == t));
          const int r = __builtin_amdgcn_readlane(top_r, l);
          const int B = r / kBlk + __builtin_amdgcn_readlane(top_o, l);
          push(pairs, npairs, 1ull, lane == 0, r, B < NB ? B * kBlk : nk + (B - NB) * kBlk);
        }
      }
      drain(true);
      __syncthreads();
    }
    const double bv = bnum > 0.0 ? bnum / bden : 0.0;
    const unsigned long long vb = (unsigned long long)__double_as_longlong(bv);
    if (bv > 0.0) atomicMax(&s_vbits, vb);
    __syncthreads();
    if (bv > 0.0 && vb == s_vbits) atomicMin(&s_tie, btie);
    __syncthreads();
    if (tid == 0) {
      float srf = 0.0f;
      if (s_vbits == 0ull) {
        a.sr[r_out] = 0.0f;
        a.depth[r_out] = NAN;
        a.jstart[r_out] = -1;
        a.kwidth[r_out] = -1;
      } else {
        const int len = (int)(s_tie / (unsigned)nk);
        const int r = (int)(s_tie - (unsigned)len * (unsigned)nk);
        const double scale = WEIGHTED ? ldexp(1.0, cd.ew - cd.es) : ldexp(1.0, -cd.es);
        const double v = __longlong_as_double((long long)s_vbits);
        const int x = r + len - 1 >= nk ? r + len - 1 - nk : r + len - 1;
        const bool wr = r + len - 1 >= nk;
        // (exact integers)
        const double Sd = Pq[x] + (wr ? Tq : 0.0) - base_at(r);
        const double Rd = (double)(up_to(x) + (wr ? cycle : (Sum)0) - before_rank(r));
        const double den = Rd * (Wd - Rd);
        srf = (float)(sqrt(v) * scale);
        a.sr[r_out] = srf;
        a.depth[r_out] = (float)(-Sd * Wd / den * scale);
        a.jstart[r_out] = sidx[r];
        a.kwidth[r_out] = sidx[x];
      }
      const unsigned long long ckey = ((unsigned long long)__float_as_uint(srf) << 32) |
                                      (unsigned long long)(0xFFFFFFFFu - (unsigned)p);
      __hip_atomic_fetch_max(a.best_key + c, ckey, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    }  // valid curve
    __syncthreads();
  }
}

template <bool W, bool D, int MODE>
const void *unbinned_fn() {
  return reinterpret_cast<const void *>(&unbinned_kernel<W, D, MODE>);
}

template <int MODE>
const void *pick_mode(bool weighted, bool dip) {
  if (weighted) return dip ? unbinned_fn<true, true, MODE>() : unbinned_fn<true, false, MODE>();
  return dip ? unbinned_fn<false, true, MODE>() : unbinned_fn<false, false, MODE>();
}

const void *pick_unbinned(bool weighted, bool dip, int mode) {
  return mode == kUnbLds     ? pick_mode<kUnbLds>(weighted, dip)
         : mode == kUnbCells ? pick_mode<kUnbCells>(weighted, dip)
                             : pick_mode<kUnbGlobal>(weighted, dip);
}

}  // namespace

int64_t unbinned_array_bytes(int n, bool weighted) {
  const int64_t N = unbinned_stride(n);
  const int64_t M = pow2_at_least((int)N);
  return 8 * N + 8 * N + 4 * N + 4 * N + 4 * N + 4 * (M + 1) + (weighted ? 4 * (N + kUnbPad) : 0);
}

int unbinned_lds_bytes(int n, bool weighted) {
  const int mode = unbinned_mode(n);
  return mode == kUnbLds     ? (int)unbinned_array_bytes(n, weighted)
         : mode == kUnbCells ? 4 * (kUnbMaxCells + 4)
                             : 0;
}

int launch_unbinned(const SearchArgs &a, bool weighted, bool dip_only, int grid, void *stream) {
  if (a.nitems <= 0) return 0;
  const void *fn = pick_unbinned(weighted, dip_only, unbinned_mode(a.ucap));
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, a.hist_bytes);
  if (e != hipSuccess) return (int)e;
  void *args[] = {const_cast<SearchArgs *>(&a)};
  e = hipLaunchKernel(fn, dim3(grid), dim3(kBlock), args, (size_t)a.hist_bytes,
                      (hipStream_t)stream);
  if (e != hipSuccess) return (int)e;
  return (int)hipGetLastError();
}

int unbinned_blocks_per_cu(bool weighted, bool dip_only, int ucap, int *blocks) {
  const void *fn = pick_unbinned(weighted, dip_only, unbinned_mode(ucap));
  const int lds_bytes = unbinned_lds_bytes(ucap, weighted);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (e != hipSuccess) return (int)e;
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, fn, kBlock, (size_t)lds_bytes);
}

}  // namespace bls
