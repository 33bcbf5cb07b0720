// Work items of the persistent kernels: claiming the next item from the
// XCD-partitioned counters and placing it in its segment (curve, tile).
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "bls_device.h"

namespace bls {
namespace {

// What a persistent workgroup holds of the work, in LDS (thread 0 only, and
// seldom: it would occupy registers of every thread): items claimed and not
// yet taken, the last item claimed, the partitions found empty, and the
// segment of the last item: items of a partition are claimed in increasing
// order, so the next one usually falls in the same segment and is placed
// without a memory access.
struct Claims {
  long long cur, end, last;
  long long seg_lo, seg_hi;  // items [lo, hi) of the segment
  int seg_curve, seg_tile0;
  unsigned done_mask;
  int started;
};
__device__ inline void claims_start(Claims &q) {  // thread 0
  q.cur = q.end = q.last = q.seg_lo = q.seg_hi = 0;
  q.done_mask = 0u;
  q.started = 0;
}

// Next work item of a persistent workgroup (thread 0 only): items of its
// own partition first, then of the others in turn; -1 once all are taken.
//
// Claims of all the XCDs on one counter are served one after the other, 14 ns
// each: 20000 one-period items of one curve took 280 us for that alone.  So a
// workgroup's first item is its own by its number, without a claim (a call of
// no more items than workgroups makes none), and where all share one counter a
// claim takes up to kClaimMax items, a quarter of what is left per workgroup,
// fewer and at last one towards the end.  (With a counter per XCD claims of
// one are fast enough, and 2% faster than larger ones on the uniform batch.)
constexpr int kClaimMax = 8;
__device__ inline long long next_item(const SearchArgs &a, Claims &q) {
  if (q.cur < q.end) return q.cur++;
  const int np = a.nparts;
  const int home = (int)(blockIdx.x % (unsigned)np);
  if (!q.started) {
    q.started = 1;
    const long long item = a.part_begin[home] + (long long)(blockIdx.x / (unsigned)np);
    if (item < a.part_begin[home + 1]) return item;
  }
  for (int k = 0; k < np; ++k) {
    const int x = home + k < np ? home + k : home + k - np;
    if (q.done_mask & (1u << x)) continue;
    // workgroups whose own the partition is, and the items beyond their first
    const int own = ((int)gridDim.x - x + np - 1) / np;
    const long long first = a.part_begin[x] + own, end = a.part_begin[x + 1];
    if (first < end) {
      int want = 1;
      if (np == 1) {
        const long long left = end - (q.last > first ? q.last : first);
        const long long share = left / (4 * (long long)own);
        want = share < 1 ? 1 : share > kClaimMax ? kClaimMax : (int)share;
      }
      const long long item =
          first + (long long)__hip_atomic_fetch_add(a.counter + x, (unsigned long long)want,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (item < end) {
        q.cur = item + 1;
        q.end = item + want < end ? item + want : end;
        q.last = item;
        return item;
      }
    }
    q.done_mask |= 1u << x;
  }
  return -1;
}

// A claimed work item and its place: curve and tile (period, for the
// unbinned search) within the curve.
struct ItemRef {
  long long item;
  int curve;
  int tile;
};

// Claim the next item and place it (thread 0 only).
__device__ inline ItemRef claim_item(const SearchArgs &a, Claims &q) {
  ItemRef r;
  r.item = next_item(a, q);
  r.curve = 0;
  r.tile = 0;
  if (r.item < 0) return r;
  if (!(r.item >= q.seg_lo && r.item < q.seg_hi)) {
    int lo = 0, hi = a.nseg - 1;  // last s with seg_start[s] <= item
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.seg_start[mid] <= r.item)
        lo = mid;
      else
        hi = mid - 1;
    }
    q.seg_lo = a.seg_start[lo];
    q.seg_hi = a.seg_start[lo + 1];
    q.seg_curve = a.seg_curve[lo];
    q.seg_tile0 = a.seg_tile0[lo];
  }
  r.curve = q.seg_curve;
  r.tile = q.seg_tile0 + (int)(r.item - q.seg_lo);
  return r;
}

}  // namespace
}  // namespace bls
