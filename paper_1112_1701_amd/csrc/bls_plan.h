// Plan object and host-side planning shared by the C ABI, the autotuner and
// the serving scheduler.
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/bls.h"
#include "bls_device.h"

namespace bls {

// Launch shape chosen per batch (by the tuner or the built-in table).
struct TileChoice {
  int lds_budget = 32768;   // dynamic LDS bytes per workgroup to aim for
  int tile_cap = kTileMax;  // upper bound on periods per work item
  int occupancy = 0;        // workgroups per CU to launch (0 = max resident)
  bool block = false;       // the block search (every curve qualifies)
};

// A fully planned call: descriptors in pinned host memory, ready to upload.
struct PlannedBatch {
  int32_t ncurves = 0;
  bool weighted = false;
  int64_t total_points = 0;
  int64_t total_results = 0;
  int64_t nitems = 0;
  int32_t nseg = 0;
  int32_t hist_bytes = 0;  // dynamic LDS of a workgroup
  bool block = false;      // block_search_kernel
  int32_t grid = 0;
  double trial_points = 0.0;
  double box_evals = 0.0;
  int32_t ucap = 0;         // unbinned search: largest curve (points)
  unsigned char *uws = nullptr;  // unbinned search: workspace of long curves
  int64_t uws_stride = 0;        // its bytes per workgroup
  int32_t nparts = 1;       // work partitions (XCDs)
  int64_t part_begin[bls::kMaxParts + 1] = {};
};

// Per-curve shape after validation (host only).
struct CurveShape {
  int64_t n_off, n, p_off, r_off;
  int32_t nperiods, nbins, kmin, kmax;
};

}  // namespace bls

struct bls_plan {
  bls_plan_config cfg{};
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int num_cus = 0;
  int max_lds = 0;

  // device working set
  bls::CurveDesc *d_curves = nullptr;
  int64_t *d_seg_start = nullptr;
  int32_t *d_seg_curve = nullptr;
  int32_t *d_seg_tile0 = nullptr;
  double *d_dt = nullptr;
  int32_t *d_q = nullptr;
  int32_t *d_qw = nullptr;
  unsigned long long *d_counter = nullptr;

  // staging of the host-array and recovery calls (allocated on first use):
  // inputs and best keys; results where the host call has no pinned memory
  // for them, and of the recovery
  double *d_t = nullptr, *d_x = nullptr, *d_w = nullptr, *d_periods = nullptr;
  int64_t *d_best = nullptr;
  float *d_sr = nullptr, *d_depth = nullptr;
  int32_t *d_j = nullptr, *d_k = nullptr;
  // pinned host staging of the host API (allocated on first use): a call's
  // inputs on the way in, its results on the way out
  char *h_stage = nullptr;
  size_t h_stage_bytes = 0;

  // detection buffers (allocated on first use)
  bls::DetectDesc *d_detect_desc = nullptr;
  void *d_detect_out = nullptr;

  // injection-recovery buffers (allocated on first use): per-injection
  // parameters [max_curves] and the cadence's t0
  void *d_inj = nullptr;
  double *d_inj_t0 = nullptr;

  // unbinned search of long curves: per-workgroup workspace (grown as needed)
  unsigned char *d_uws = nullptr;
  int64_t uws_bytes = 0;

  // eclipse-window buffers (allocated on first use)
  bls::WindowDesc *d_window_desc = nullptr;
  unsigned int *d_window_flag = nullptr;

  // variability pre-search scratch (allocated on first use, grown as needed)
  int64_t *d_var_noff = nullptr;      // [max_curves + 1]
  uint8_t *d_var_alive = nullptr;     // [max_curves]
  int64_t *d_var_chip = nullptr;      // [var_chip_cap + 1]
  int64_t var_chip_cap = 0;

  // pinned host descriptors, one block (place_desc)
  bls::CurveDesc *h_curves = nullptr;
  int64_t *h_seg_start = nullptr;
  int32_t *h_seg_curve = nullptr;
  int32_t *h_seg_tile0 = nullptr;

  // The curves' status, in pinned memory that the prep kernel writes itself: a
  // call's wait is then for the stream alone, without a copy of its own (one
  // curve of 1000 points x 5000 periods 73 us a call, 63 so).
  int32_t *h_status = nullptr;
  int32_t *status_dev = nullptr;  // the device's address of it

  // bls_search_device: while nothing has rewritten the descriptors, a call
  // like the last one launches its plan (last) again, without validation,
  // planning and upload.  (As three captured graphs with the timing events
  // between them the same sequence took 121 us instead of 105 for 1000 points
  // and 5000 periods: graphs of one kernel launch slower than the kernel.)
  uint64_t replay_sig = 0;
  bool replay_valid = false;

  hipEvent_t ev_begin = nullptr, ev_search0 = nullptr, ev_search1 = nullptr,
             ev_end = nullptr;

  // The pinned descriptors above are read by queued copies until ev_desc,
  // recorded after them, completes; a call that rewrites them first waits for
  // it.
  hipEvent_t ev_desc = nullptr;
  bool desc_pending = false;

  // Search-kernel durations of the last kTimeRing calls: events recorded
  // just before and after each search (or unbinned) kernel launch.
  static constexpr int kTimeRing = 64;
  hipEvent_t ev_k0[kTimeRing] = {};
  hipEvent_t ev_k1[kTimeRing] = {};
  int64_t k_recorded = 0;   // kernel launches bracketed so far
  int64_t k_base = 0;       // value of k_recorded at the last reset

  bls::PlannedBatch last;
  bls_call_stats stats{};
  std::string last_error;
  std::vector<bls::CurveShape> shapes;   // scratch for planning
  std::vector<int> order;                // scratch for planning
  bool tuned_valid = false;
  uint64_t tuned_key = 0;
  bls::TileChoice tuned;
};

namespace bls {

// Validation of a batch description and its parameters (host only; no
// device access).  With check_data, also the host data arrays.  Without
// binned, nbins is ignored and each curve's duty-cycle range is checked as
// phase limits (0 < qmin <= qmax < 1) with at most kUnbinnedMaxPoints points.
int validate_batch(const bls_plan_config &cfg, const bls_batch &b, bool check_data,
                   std::vector<CurveShape> &shapes, std::string &err, bool binned = true);
// The same into caller-owned storage (no heap use): shapes has room for
// shapes_cap curves; a failure's message goes to err (NUL-terminated).
int validate_batch_into(const bls_plan_config &cfg, const bls_batch &b, bool check_data,
                        CurveShape *shapes, int shapes_cap, char *err, size_t err_len,
                        bool binned = true);
// Host fields of one curve's descriptor (prep fields zero): fixed-point
// layout, and the period tile and plane stride that fit tc's LDS budget.
// block: the layout of the block search (bls_blocks.hip).
void fill_curve_desc(const CurveShape &s, bool weighted, const TileChoice &tc,
                     bool check_periods, bool block, CurveDesc &d);

// Whether the block search can run every curve of a launch (boxes of at most
// half the bins) and is the faster kernel for it.  tuned: the tiles of the
// other kernel would be tuned.
bool block_batch(const CurveShape *shapes, int n, bool weighted, int min_in_points, bool tuned,
                 int num_cus, int max_lds);
// LDS budget per workgroup of the block search (`rep`: the batch's typical
// curve).
int block_lds_budget(const CurveShape &rep, bool weighted, int max_lds);
constexpr int kBlockStaticLds = 1536;  // static LDS of block_search_kernel, rounded up
// Periods per work item of the block search within an LDS budget (at least
// one), its plane stride and geometry.
void fit_block_tile(int nbins, int kmin, int kmax, int64_t nperiods, int lds_budget, int tile_cap,
                    bool weighted, int *tile, int *stride, BlockGeom *g);
// Block search: a curve's geometry and the place of the waves' scratch into
// its descriptor (tile, stride, bins and weighted are set).
void set_block_layout(CurveDesc &d, const BlockGeom &g);
// Dynamic LDS of a launch, extended by one curve at a time: the most that any
// of its curves needs.
struct LdsLayout {
  int bytes = 0;
  void add(const CurveDesc &d, bool block);
  int total() const { return bytes; }
};
// LDS of a block-search tile of T periods: its planes, and scratch for the
// waves that have a period.
inline int block_tile_bytes(int T, int nbins, int kmax, bool weighted, const BlockGeom &g) {
  return T * block_plane_words(nbins, kmax, g) * 8 * (weighted ? 2 : 1) +
         (T < 4 ? T : 4) * block_scratch_bytes(nbins, g);
}

// Segments grouped into work partitions (one per XCD), curves assigned
// round-robin in descending cost; items_of[c] = work items of curve c.
void layout_partitions(bls_plan *p, const std::vector<double> &cost,
                       const std::vector<int64_t> &items_of, PlannedBatch &out);

// Periods per work item of a batch: kGroupMax when the batch has at least
// four such groups per workgroup of a full grid (the kernel then writes each
// item's results as whole lines), else 0 (one period tile per item).  The
// environment variable BLS_ITEM_GROUP (0 or kGroupMax) overrides the choice.
int item_group(const bls_plan *p, const std::vector<CurveShape> &shapes);

// Fill the pinned descriptors for a validated batch and size the launch.
int plan_batch(bls_plan *p, const std::vector<CurveShape> &shapes, bool weighted,
               const TileChoice &tc, PlannedBatch &out);

// The launch sequence of a search, in three parts: (1) upload descriptors,
// clear counters and keys, prep; (2) the search kernel (with unbinned, the
// unbinned kernel: js and ks then receive the first and last point of each
// best box); (3) per-curve best index from the best keys, in their place or
// elsewhere.  upload: the descriptors are new.
int enqueue_pre(bls_plan *p, const PlannedBatch &pb, const double *t, const double *x,
                const double *w, const double *periods, int64_t *best, bool upload);
int enqueue_kernel(bls_plan *p, const PlannedBatch &pb, const double *periods, float *sr,
                   float *depth, int32_t *js, int32_t *ks, int64_t *best, bool unbinned);
int enqueue_post(bls_plan *p, const PlannedBatch &pb, const int64_t *keys, int64_t *best);
// All three, with ev_desc after the uploads and the kernel bracketed by the
// timing ring's events (streams that are not capturing).
int enqueue_search(bls_plan *p, const PlannedBatch &pb, const double *t, const double *x,
                   const double *w, const double *periods, float *sr, float *depth,
                   int32_t *js, int32_t *ks, int64_t *best, bool unbinned = false,
                   bool upload = true, int64_t *keys = nullptr);
// Bytes of the descriptors of nc curves, and their places in the pinned and
// the device block.
size_t desc_bytes(int nc);
void place_desc(bls_plan *p, int nc);
// Wait until no queued copy still reads the pinned descriptors.
int desc_wait(bls_plan *p);
// Mark the pinned descriptors as read by work queued so far on the stream.
int desc_mark(bls_plan *p);
// Events of the timing ring around the next kernel launch.
int ring_begin(bls_plan *p);
int ring_end(bls_plan *p);

int set_error(bls_plan *p, int status, const std::string &msg);
// The calling thread's error without a plan (what bls_last_error(NULL)
// returns), recorded without heap use.
int set_error_noplan(int status, const char *msg);
int hip_error(bls_plan *p, hipError_t e, const char *what);
int width_range(int32_t nbins, double qmin, double qmax, int32_t *kmin, int32_t *kmax);

// Search-kernel duration of the last bracketed launch (ms; 0 if none).
double last_kernel_ms(bls_plan *p);
// Call statistics of a planned batch.
void fill_stats(bls_plan *p, const PlannedBatch &pb, bool replayed);
// Device inputs and best keys of the host-array and recovery calls
// (max_points, max_periods, max_curves sized), allocated on first use.
int ensure_staging(bls_plan *p);
// The same for their results, for calls whose kernels write them to device
// memory.
int ensure_result_staging(bls_plan *p);
// INVALID_ARG naming the first curve whose prep found invalid data.
int check_device_status(bls_plan *p, int ncurves);
// Per-curve flags (1: invalid data or trial periods) of the last prep.
int device_status_flags(bls_plan *p, int ncurves, int32_t *bad);
// Detection buffers (max_curves descriptors and results), on first use.
int ensure_detect_buffers(bls_plan *p);
// Queue the detection kernel over ncurves periodograms of one shared grid,
// curve c's SR at sr[c * nperiods]; results in p->d_detect_out.
int enqueue_detect_shared(bls_plan *p, int ncurves, const double *periods, int64_t nperiods,
                          const float *sr, int max_peaks, double window, double threshold);
// Injection-recovery buffers, on first use.
int ensure_recovery_buffers(bls_plan *p);

// Device allocation with the optional failure-injection hook.
hipError_t device_alloc(void **ptr, size_t bytes);

// LDS words (64-bit) one period's histogram plane needs: the bins, then the
// clamp word / wrap-around copy of the first min(kmax, nbins / 2) - 1 bins.
int hist_words(int nbins, int kmax);
// Words between consecutive periods' planes for a tile of `tile` periods:
// at least hist_words, padded so that the scan's 64-bit reads, served 16
// lanes at a time across 32 four-byte banks, meet as few bank conflicts as
// the layout allows (lane task (start bin, period) = divmod(lane, tile)).
int hist_stride(int nbins, int kmax, int tile, bool weighted);
// Periods per work item that fit an LDS budget (at least one, at most
// tile_cap and nperiods) and the padded stride that goes with it.
void fit_tile(int nbins, int kmax, int64_t nperiods, int lds_budget, int tile_cap,
              bool weighted, int *tile, int *stride);

// Tile choice for a batch: autotuned (cached) unless disabled.
TileChoice choose_tiles(bls_plan *p, const std::vector<CurveShape> &shapes, bool weighted);
// The built-in table the tuner starts from.
TileChoice default_tiles(bool weighted);
// The built-in table's LDS budget for a call of `periods` trial periods whose
// typical curve is `rep`.
int untuned_lds_budget(const CurveShape &rep, int64_t periods, bool weighted, int num_cus);

}  // namespace bls
