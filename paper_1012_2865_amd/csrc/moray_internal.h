// Host-side internals shared by the one-shot runtime (moray_runtime.cpp) and
// the serving engine (moray_serve.cpp). Not part of the public ABI.
#pragma once
#include "moray.h"
#include "moray_device.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <vector>

namespace moray {

// ---- kernel launchers (moray_kernels.hip) ----
hipError_t launch_reset(hipStream_t, Counters*, SgStats*, int);
hipError_t launch_reset_levels(hipStream_t, Counters*);
hipError_t launch_reset_generation(hipStream_t, Counters*, int cin, int cout);
hipError_t launch_reset_stats(hipStream_t, SgStats*, int first, int count);
// mark: the n_mark optically-thin marks the prep pass clears (NULL: none);
// kappa64: where it also writes the columns in float64 (NULL: nowhere)
template <typename R>
hipError_t launch_prep(hipStream_t, int, const GridDev*, int, int, const ProblemDev*, long long, long long, R*, double*,
                       Counters*, uint8_t* mark = nullptr, long long n_mark = 0, double* kappa64 = nullptr);
template <typename R>
hipError_t launch_trace_level(hipStream_t, int num_cu, int blocks, const TraceArgs<R>&, bool cache, int width, bool cover,
                              bool radp, bool thin = false);
template <typename R>
hipError_t launch_trace_level_halt(hipStream_t, int num_cu, int blocks, const TraceArgs<R>&, bool cache, int width);
// Serving: empty the queued rays (counter row `row`, nseg segments) whose
// tree index lies in one of the n ranges [lo[i], hi[i]) (n <= kDropRanges).
hipError_t launch_drop_trees(hipStream_t, uint32_t* tree, const Counters* ctr, int row, unsigned long long seg_cap,
                             int nseg, const int* lo, const int* hi, int n);
// moray_td_kernels.hip: the halt list sorted by (level, tree, pixel); levels are at most top_level but for
// empty records
int td_level_bits(int top_level);
hipError_t td_sort_temp_bytes(unsigned long long cap, size_t* bytes);
hipError_t launch_td_sort(hipStream_t, int num_cu, const RayQueue& pool, const int* lev, unsigned long long n,
                          int top_level, int tree_bits, int pix_bits, int pix_drop, void* keys_in, void* keys_out,
                          uint32_t* idx_in, uint32_t* idx_out, void* temp, size_t temp_bytes);
// trees, mark: the tree table and the optically-thin marks (NULL when no problem uses them)
hipError_t launch_finalize(hipStream_t, int, const GridDev*, const ProblemDev*, const FinalBlock*, const double*,
                           const double*, double*, const Counters*, const TreeDev* trees = nullptr,
                           const uint8_t* mark = nullptr);
hipError_t trace_occupancy(int precision, bool cache, int* blocks_per_cu);
// photo-ionisation equilibrium (moray_equilibrium.hip)
// dx: 1 + kEqMaxBlocks doubles; dx[0] receives the largest change of the pass
constexpr int kEqMaxBlocks = 2048;
hipError_t launch_equilibrium_update(hipStream_t, const double* kph, const float* n_h, double* x64, float* x32,
                                     long long n, double alpha_b, double w, const unsigned char* skip, double* dx);
hipError_t launch_widen(hipStream_t, int num_cu, const float* x32, double* x64, long long n);
// moray_evolve: lim receives the per-cell limits, dmin (1 + kEqMaxBlocks doubles) their smoothed minimum in dmin[0]
hipError_t launch_step_limit(hipStream_t, int num_cu, const double* kph, const float* n_h, const double* x64, int nx,
                             int ny, int nz, double alpha_b, double sigma_bar, double dx_cm, double eps,
                             double tau_front, double dt_max, const unsigned char* skip, double* lim, double* dmin);
hipError_t launch_evolve_update(hipStream_t, int num_cu, const double* kph, const float* n_h, double* x64, float* x32,
                                long long n, double alpha_b, double dt, const unsigned char* skip);

struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
};

// moray_noalloc.hip: the fixed scratch array of moray_trace_noalloc and its
// address on a device (looked up once per device, with that device current)
size_t scratch_bytes();
hipError_t scratch_address(int device, void** ptr);

struct Engine;     // serving engine of a context (moray_serve.cpp)
struct PlanHost;   // last one-shot solve and its captured launch sequence (moray_runtime.cpp)

}  // namespace moray

struct moray_ctx {
  int device = 0;
  int precision = MORAY_FP32_ACC64;
  hipStream_t stream = nullptr;
  size_t budget = 0;
  size_t queue_cap_user = 0;
  int waves_per_cu = 0, chunk = 0, profile = 0;
  int refill = 0;                // moray_init_params.refill_lanes, reported back and kept in tuning files; no launch reads it
  int reserve_user = 0;          // next-level rays a wave reserves room for at once; 0 = from the queue size
  bool cache = true;
  int num_cu = 0;
  int blocks_per_cu = 1;
  std::string err = "no error";
  // moray_trace_noalloc: the device address of the library's fixed scratch
  // array on this context's device (null if its lookup failed: scratch_err),
  // and while such a call runs, the part of it the call has carved so far
  char* scratch = nullptr;
  std::string scratch_err;
  bool arena = false;
  size_t arena_used = 0;
  bool fail_capture_once = false;  // test hook (MORAY_INJECT_CAPTURE_FAILURE=1 at moray_init): the next capture
                                   // of a launch sequence fails as if HIP had refused it
  bool overflow_serve_once = false;  // test hook (MORAY_INJECT_SERVE_OVERFLOW=1 at moray_init): the serving
                                     // engine's first launch with two or more problems reports a queue overflow
  bool stale_serve_rates = false;    // test hook (MORAY_INJECT_SERVE_STALE_RATES=1 at moray_init): the serving
                                     // engine's queue memory starts with NaN in every photon rate
  size_t allocated = 0;
  moray::DevBuf grids, probs, trees, stats, ctr, kappa, kappa64, acc, mark, eexc, fblocks, partial, fields, outs;
  moray::DevBuf q_pix[2], q_tree[2], q_r[2], q_P[2];
  size_t q_cap = 0;
  void* h_stage = nullptr;
  size_t h_stage_bytes = 0;
  std::vector<hipEvent_t> evs;
  moray::Engine* engine = nullptr;
  moray::PlanHost* plan = nullptr;
  hipStream_t gstream = nullptr;   // stream of captured launch sequences
  hipEvent_t gev = nullptr;
  moray::DevBuf eq_x, eq_kph, eq_heat, eq_dx;   // moray_equilibrate / moray_evolve: float64 iterate, rates,
                                                 // reduction partials
  moray::DevBuf ev_lim;                          // moray_evolve: per-cell step limits
  moray::DevBuf eq_skip;                         // both: root cells under a child grid (1) or not (0)
};

namespace moray {

moray_status fail(moray_ctx* c, moray_status s, const std::string& msg);
bool hip_ok(moray_ctx* c, hipError_t e, const char* what);
void release(moray_ctx* c, DevBuf& b);
moray_status ensure(moray_ctx* c, DevBuf& b, size_t bytes, const char* what);
moray_status validate(moray_ctx* c, const moray_problem& P, int pi);
int reach_level(const moray_problem& P);
double level_rays_bound(const moray_problem& P);

// Energy groups a ray of a problem with n groups carries: n split evenly over
// the fewest packs of at most kPack; pack k holds groups [first, first + count).
inline int pack_count(int n) { return (n + kPack - 1) / kPack; }
inline int pack_first(int n, int k) { return (int)((long long)n * k / pack_count(n)); }
inline int pack_width(int n) { return (n + pack_count(n) - 1) / pack_count(n); }

// Planes of photon rates a queue slot holds for rays of up to `width` groups
// (the widths the trace kernel is built for).
inline int rate_planes(int width) { return width <= 1 ? 1 : (width == 2 ? 2 : kPack); }

// Bytes of one queue slot.
constexpr size_t slot_bytes(int planes) { return sizeof(uint64_t) + sizeof(uint32_t) + sizeof(double) * (1 + planes); }

// Bytes a time-dependent state holds per pool record, besides the sort's scratch: the
// record and its level in both pools, its place in the sorted order, and its share
// of two level queues.
constexpr size_t td_record_bytes(int planes) {
  return 2 * (slot_bytes(planes) + sizeof(int)) + sizeof(uint32_t) + 2 * slot_bytes(planes) / 4;
}

// The parts of a tree's record that follow from its problem: the rays of
// source `src` carrying groups [g0, g0 + n) (one group per ray in the modes
// that keep a plane of accumulators per group).
void fill_tree(TreeDev& d, const moray_problem& P, int src, int g0, int n, const ProblemDev& pd, const GridDev& root);

// Level at which the seeds of `trees` trees enter (see the trace kernel): the
// finest, not beyond `top` (the finest any of them reaches), that still has no
// more pixels than half the lanes of the launch and than the level queue has room
// for (`cap`: a queue too small for a level is reported as such). Half, so that the
// repeated part of the work runs beside the rest: one 32^3 source, 20 steps of a 64^3
// front, and the ragged float64 case: 117 us, 3.50 and 1.00 ms at 3 thousand, 108 us,
// 3.19 and 0.97 ms at 13 thousand, 112 us, 3.12 and 0.95 ms at 98 thousand (half of
// 256 CUs with three blocks each), 132 us, 3.35 and 0.94 ms at 200 thousand; larger
// problems differ by less than 2%. Requests admitted to a running queue, whose rays
// hold lanes already, enter alike: in Poisson streams of 20, 50, 100 and 150 requests a
// second (edges 32 to 256) the mean latency was 9.9, 12.1, 117.2 and 62.3 ms, and 10.0,
// 12.3, 116.9 and 60.4 ms with their seeds at their own level.
inline int descend_level(long long trees, int l0, int top, size_t cap, long long lanes) {
  const long long most = cap < (size_t)(lanes / 2) ? (long long)cap : lanes / 2;
  int l = l0;
  while (l < top && trees * (12ll << (2 * (l + 1))) <= most) ++l;
  return l;
}
// the lanes of a context's launches
inline long long launch_lanes(const moray_ctx* c) {
  return (long long)std::max(1, c->num_cu * c->blocks_per_cu) * kTraceBlock;
}

// Segments of a level queue for `cap` rays: a power of two up to kSegMax, so
// the trace kernel splits a launch's seeds among them with shifts.
inline int queue_segments(size_t cap) {
  int n = 1;
  while (n < kSegMax && (size_t)(2 * n) * 65536 <= cap) n *= 2;
  return n;
}

// serving engine (moray_serve.cpp)
bool engine_busy(moray_ctx* c);
void engine_stop(moray_ctx* c);

constexpr double kEvErgConst = 1.602176634e-12;
constexpr double kPiConst = 3.14159265358979323846;

}  // namespace moray
