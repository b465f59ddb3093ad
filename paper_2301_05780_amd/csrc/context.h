// Library context: device, stream, caches and scratch owned by one pdd_ctx.
#pragma once

#include <algorithm>
#include <cmath>

#include <hip/hip_runtime.h>

#include <memory>
#include <string>
#include <vector>

#include "geometry.h"
#include "kernels.h"
#include "pdd.h"
#include "spectral.h"

namespace pdd {

// Owning device allocation that only grows.
struct DeviceBuffer {
  void* ptr = nullptr;
  size_t bytes = 0;
  DeviceBuffer() = default;
  DeviceBuffer(const DeviceBuffer&) = delete;
  DeviceBuffer& operator=(const DeviceBuffer&) = delete;
  ~DeviceBuffer();
  hipError_t reserve(size_t want);
  void release();
  template <typename T> T* as() const { return static_cast<T*>(ptr); }
};

// Polls of a wait between the workgroups of one launch before it is given up (some seconds).
constexpr uint32_t WAIT_POLLS = 1u << 21;

// Device scratch of one kind of call, in use by one such call at a time also
// when the context's stream changes between calls: acquire() makes the stream
// wait for the last use on another one, release() marks the use just enqueued.
struct StreamScratch {
  DeviceBuffer buf;
  hipEvent_t done = nullptr;
  hipStream_t stream = nullptr;
  StreamScratch() = default;
  StreamScratch(const StreamScratch&) = delete;
  StreamScratch& operator=(const StreamScratch&) = delete;
  ~StreamScratch() {
    if (done) (void)hipEventDestroy(done);
  }
  pdd_status acquire(pdd_ctx* ctx, size_t bytes);
  pdd_status release(pdd_ctx* ctx);
};

// Host geometry of one (partition, knots) pair and its device copies.
struct GeoCache {
  pdd_partition part{};
  pdd_knots kn{};
  Geometry g;
  DeviceBuffer desc, knot_ij, row_ptr, col_idx, lattice;
};

// Tickets of one (geometry, path counts, ticket size) combination.
struct TicketCache {
  const GeoCache* geo = nullptr;
  std::vector<int32_t> npk;       // paths per knot
  std::vector<double> hk;         // per-knot time steps (empty: the launch's h)
  DeviceBuffer h_knot;            // device copy of hk
  int32_t per_ticket = 0;
  uint32_t inst = 0;
  bool spatial = false;           // spatial order (tabulated coefficients) instead of longest-first
  int64_t n_tickets = 0;
  DeviceBuffer tickets, ticket_begin, n_paths, order;
  // spatial order: cumulative expected cost along the order, and the XCD
  // split of the order for the grid it was last computed for
  std::vector<double> cum_cost;
  int32_t xcd_grid = -1;
  DeviceBuffer xcd_begin;
};

// Device-side tables of one batch of instances (rebuilt when the batch changes).
struct BatchCache {
  std::vector<pdd_partition> parts;
  std::vector<pdd_knots> knots;
  std::vector<std::vector<int32_t>> npk;
  std::vector<double> h, a;
  std::vector<uint32_t> inst_ids;
  int32_t per_ticket = 0;
  std::vector<std::unique_ptr<GeoCache>> geos;
  std::vector<int64_t> knot_off, ticket_off, n_tickets;
  int64_t total_tickets = 0;
  int slot_len = 0;
  DeviceBuffer desc, insts, tickets, order;
  std::vector<std::unique_ptr<DeviceBuffer>> ticket_begin, n_paths;
};

struct TuneEntry {
  std::string sig;
  int block, grid, per_ticket, schedule, refill, spare;
  double ms;
  std::string report;
};

struct AssembleJob {
  pdd_coeffs coeffs;
  pdd_partition part;
  pdd_knots knots;
  pdd_run run;
  int32_t* row_ptr;
  int32_t* col_idx;
  double* val;
  double* b;
  double* diag;
};

}  // namespace pdd

namespace pdd {
// Collocation tables of one spectral degree p on the device.
struct SpecCache {
  int32_t p = 0;
  DeviceBuffer buf;
  SpecDev dev{};
  double decomp_residual = 0, inverse_residual = 0;
};
// Inverses of the RBF stencil matrices for one (slot length, spacing, c).
struct RbfCache {
  int32_t slot_len = 0;
  double dx = 0, dy = 0, c = 0;
  int64_t half = 0;
  DeviceBuffer tab;
};
}  // namespace pdd

struct pdd_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  int cu_count = 0;
  std::string arch;
  std::string err;
  std::vector<std::unique_ptr<pdd::GeoCache>> geo;
  std::unique_ptr<pdd::TicketCache> tickets;
  std::unique_ptr<pdd::BatchCache> batch;
  std::unique_ptr<pdd::RbfCache> rbf;
  std::unique_ptr<pdd::SpecCache> spec;
  pdd::DeviceBuffer spec_range;      // LUT field ranges of the spectral solve (12 + 1024 * 12 doubles)
  hipGraph_t graph = nullptr;
  hipGraphExec_t graph_exec = nullptr;
  bool capturing = false;
  std::vector<pdd::TuneEntry> tune_cache;
  pdd::DeviceBuffer partial;
  void* host_words = nullptr;        // pinned, 256 bytes: small results read back
  pdd::DeviceBuffer solve_scratch;
  pdd::StreamScratch eval_scratch;   // per-wave sums of the point evaluation
  pdd::DeviceBuffer collect_scratch, mlp_scratch, calib_scratch, calib_alpha;
  pdd::StreamScratch mlp_wide;       // the trainer's exchange between workgroups,
  uint32_t mlp_epoch = 0;            // and no flag in it is above this
  std::vector<std::unique_ptr<pdd::DeviceBuffer>> mlp_slices;   // gradients of captured training (run_mlp_train)
  uint32_t wait_polls = pdd::WAIT_POLLS;   // of a wait between the workgroups of one launch
  // launch overrides (0 = automatic), set by the tuner
  int force_block = 0, force_grid = 0, force_per_ticket = 0;
  int schedule = PDD_SCHEDULE_STATIC;
  int refill_min = 1;                // refill idle lanes once at least this many are idle
  int spare_rows = -1;               // tally rows per workgroup beyond one per wave (-1: one per wave)
  pdd::DeviceBuffer ticket_counter;
  pdd::DeviceBuffer lut_max;         // LUT + GM: table-wide |sigma| maxima
  pdd::DeviceBuffer lut_cells;       // float32 LUT assembly: cell-major copy of the table
  pdd::DeviceBuffer lut_info;        // its varying fields, layout and constant fields (16 words)
  int32_t table_read_all = 0;        // 1: the full cooperative read even for constant fields
  bool lut_lane = false;             // the last eager float32 table assembly found the lane-read layout
  // shape of the last assembly launch (reported by pdd_last_launch)
  int last_grid = 0, last_block = 0;
  int64_t last_tickets = 0;
  // optional event pairs around the assembly kernels
  bool timing = false;
  bool timing_with_finalize = false;  // the autotuner's pairs also cover the row sums
  std::vector<hipEvent_t> ev_pool;   // 2 per timed launch, reused
  int ev_used = 0;                   // pairs recorded since pdd_set_timing
  ~pdd_ctx() {
    for (hipEvent_t e : ev_pool) (void)hipEventDestroy(e);
    if (host_words) (void)hipHostFree(host_words);
    if (graph_exec) (void)hipGraphExecDestroy(graph_exec);
    if (graph) (void)hipGraphDestroy(graph);
  }
};

namespace pdd {

pdd_status check_hip(pdd_ctx* ctx, hipError_t e, const char* what);
pdd_status get_geometry(pdd_ctx* ctx, const pdd_partition& part, const pdd_knots& kn, GeoCache** out);
pdd_status get_lattice(pdd_ctx* ctx, GeoCache* gc);
pdd_status build_geo_cache(pdd_ctx* ctx, const pdd_partition& part, const pdd_knots& kn,
                           std::unique_ptr<GeoCache>& out);
bool same_geometry(const GeoCache& gc, const pdd_partition& part, const pdd_knots& kn);
pdd_status run_assemble_batch(pdd_ctx* ctx, int32_t n_inst, const pdd_instance* inst);
pdd_status validate_run(pdd_ctx* ctx, const pdd_coeffs& c, const pdd_run& r);
void fill_asm_params(const GeoCache& gc, const pdd_coeffs& co, const pdd_run& run, AsmParams& P);
pdd_status run_assemble(pdd_ctx* ctx, const AssembleJob& job);
// LUT family under the GM rule: enqueue the table-bound kernels and point
// P.coef.lut_max at their result (no-op otherwise).
pdd_status prepare_lut_bound(pdd_ctx* ctx, const pdd_coeffs& co, const pdd_run& run, AsmParams& P, bool capturing,
                             bool scanned = false);
// LUT family in float32: enqueue the cell-major copy of the table and point
// P.coef.cells at it (no-op otherwise).
bool uses_lut_cells(const pdd_coeffs& co, const pdd_run& run);
pdd_status prepare_lut_cells(pdd_ctx* ctx, const pdd_coeffs& co, const pdd_run& run, bool capturing, bool* lane_layout);
// RBF interpolation: build (once per geometry and shape parameter) and
// upload the inverses of the stencil matrices; point P.rbf_inv at them.
pdd_status prepare_rbf(pdd_ctx* ctx, const Geometry& g, const pdd_run& run, AsmParams& P, bool capturing);
pdd_status run_eval_subdomain(pdd_ctx* ctx, const pdd_coeffs& co, const pdd_partition& part, const pdd_knots& kn,
                              const double* u_knots, int64_t n_pts, const double* xy, const pdd_run& run, double* u,
                              double* se);
pdd_status run_solve(pdd_ctx* ctx, int64_t n, const int32_t* rp, const int32_t* ci, const double* val,
                     const double* b, double* u, double tol, int32_t max_iter, int32_t* iters, double* relres);
// pdd_solve_noalloc: the same solve on the library's static device scratch
// (SOLVE_NOALLOC_BYTES per GPU); solve_noalloc_setup(device) looks up that
// device's copy once (the device current).
constexpr size_t SOLVE_NOALLOC_BYTES = (size_t)128 << 20;
hipError_t solve_noalloc_setup(int device);
pdd_status run_solve_noalloc(pdd_ctx* ctx, int64_t n, const int32_t* rp, const int32_t* ci, const double* val,
                             const double* b, double* u, double tol, int32_t max_iter, int32_t* iters,
                             double* relres);

// Tally rows in an assembly workgroup's pool: one per wave plus the context's
// spare rows (at most one more per wave).
inline int pool_rows_for(const pdd_ctx* ctx, int block) {
  const int w = block / 64;
  return ctx->spare_rows < 0 ? 2 * w : w + std::min(ctx->spare_rows, w);
}


// Automatic shape of the kernels with a shared row pool (batched launches and
// the table family) for large runs: workgroups of one wave with one tally row,
// claiming their tickets from the device counters.  A wave with a single row
// finishes a ticket before it opens the next one, so a ticket's sums do not
// depend on which wave runs it or when, and the result is bitwise reproducible
// although the waves balance themselves.  The fixed stride does not: a SIMD
// issues its oldest wave first, and the waves end between half and all of the
// launch.  One row per wave also leaves LDS for more waves.  Measured, 256 threads
// with two rows per wave and the fixed stride against this: 64-instance batch
// 157 ms, 75 ms; 4096^2 table with the control variate 43.8 ms, 30.4 ms;
// 2049^2 table of seven varying fields 12.7 ms, 10.8 ms.
inline bool default_shape(const pdd_ctx* ctx) {
  return !ctx->force_block && !ctx->force_grid && !ctx->force_per_ticket && ctx->spare_rows < 0 &&
         ctx->schedule == PDD_SCHEDULE_STATIC;
}
// Paths per ticket: fewer cost more drained lanes (about 60 paths' worth per
// ticket), more a longer wait for the last ticket: 8 sqrt(paths per wave) is
// 2800 for the 4096^2 table (1250 to 2500: 30.3 ms; 5000: 34), 970 for the
// 2049^2 table (500: 11.2, 1000: 10.7, 2000: 12.4 ms) and 4650 for the batch
// (4096: 76.9, 8192: 74.9, whole knots: 78.4 ms).
inline int64_t solo_ticket(int64_t paths, int64_t waves) {
  return std::max<int64_t>(64, (int64_t)(8.0 * std::sqrt((double)paths / (double)std::max<int64_t>(waves, 1))));
}
// From how many paths per wave on: a ticket's last paths run with idle lanes,
// so a small run loses more than the balance gives, unless one row per wave
// lets many more waves reside than two rows do (`waves` against `strided`).
// Measured old / new time: equal residency 0.9 at 6750 paths per wave, 1.0 at
// 8400; 1.25 times the waves 0.97 at 4700; 1.33 times 0.93 at 1480, 1.10 at
// 5900, 1.35 at 74,000; 2.25 times 1.19 at 2430, 2.7 at 24,000.
// No ticket is longer than a knot's paths (`knots` of them), and short ones lose
// their lanes' ends more often: with 1.67 times the waves and 2700 paths per wave
// 0.82 at 213 paths per knot, 1.03 at 349 (a table with 34,753 knots 0.92 at 450), with
// 6000 per wave 1.03 at 214, with 9000 1.17 at 321; with 2.12 times the waves 0.90 at
// 67 (2100 per wave), 0.97 at 112 (3500), 1.15 at 168 (2700).
inline bool solo_pays(int64_t paths, int64_t waves, int64_t strided, int64_t knots) {
  const double r = (double)waves / (double)std::max<int64_t>(strided, 1), r4 = r * r * r * r;
  const double per_wave = (double)paths / (double)std::max<int64_t>(waves, 1);
  const double ticket = std::min((double)solo_ticket(paths, waves), (double)paths / (double)std::max<int64_t>(knots, 1));
  return per_wave >= std::max(2048.0, 16384.0 / r4) && ticket * per_wave >= 1.1e7 / r4;
}

// Paths per ticket under the fixed stride.  `paths` in all on `waves` waves;
// `knots` with `each` paths (each = 0: the counts differ, or several
// instances).  `per_wave`: tickets per wave of a large run.
//   Small runs (fewer than 1.3 tickets of 256 paths per wave): the run lasts as
// long as a wave's paths take one after the other, so at least 64 paths (one per
// lane) and no more than 1.7 tickets per wave.  29 knots of 1000 float64 paths:
// 1.02 ms with 256, 0.64 ms with 64; 369 knots of 1000: 0.92, 0.69 ms; 369 of 4000:
// 1.20, 0.99 ms; 1729 of 1000: 2.01, 1.82 ms.
// 256 over this cut, means of four seeds at 110 random sizes (6 to 100 steps): 0.98 to
// 1.5; 1.14 on average below half a ticket of 256 per wave, 1.06 up to one, 1.03 above.
//   Large runs: per_wave tickets' worth of paths per wave; shorter tickets than 256 cost
// more.  No other number of them is better in general: of 1729 knots of 10,000 paths the
// times for 4.5 to 8.7 tickets per wave lie between 1.03 ms (5.63) and 1.16 (5.91, 8.16),
// 7.04 1.11, and where the short ones lie changes with the paths per knot (2625 knots,
// 5.64 against 7.18: 0.952 and 0.910 ms for 5000 paths, 1.047 and 1.129 for 6000).
inline int64_t strided_ticket(int64_t paths, int64_t waves, int64_t knots, int64_t each, int64_t per_wave) {
  if ((double)paths < 1.3 * 256.0 * (double)waves) {
    const double most = 1.7 * (double)waves;
    const int64_t cuts = each > 0 ? (int64_t)(most / (double)knots) : 0;
    const int64_t p = cuts > 0 ? (each + cuts - 1) / cuts : (int64_t)std::ceil((double)paths / most);
    return std::min<int64_t>(256, std::max<int64_t>(64, p));
  }
  return std::max<int64_t>(256, (paths + per_wave * waves - 1) / (per_wave * waves));
}

}  // namespace pdd
