// Phase II calibration (Sec. 4.1-4.2, eqs. 32-39): mixed Gobet-Menozzi /
// Euler-Maruyama trajectories scored with the warm-up solution.
//
// One lane per path (knot k, path p < N0'), the assembly's random stream,
// step and exit rules; waves are persistent and claim path ids from a
// device counter as their lanes fall idle.  A path runs until it leaves the
// closed patch (the naive exit); on the way, the first step whose iterate
// is not strictly inside the Gobet-Menozzi-shrunk patch is its GM exit.
// Each exit is
// resolved as in the assembly (side choice, projection, hat weights) and
// scored with u0: phi = Z_K + Y_K u0(P_K), u0 interpolated from the warm-up
// knot values on interface sides and the boundary datum g on the domain
// boundary.  xi is the control variate (eq. 37, with the gradient table) at
// the GM exit.  Each path writes (phi_GM, phi_EM, xi, K_GM, K_EM);
// a second kernel sums a knot's paths in a fixed order into
//   sum(phi_EM - phi_GM), sum phi_GM, sum phi_GM^2, sum xi, sum xi^2,
//   sum phi_GM xi, sum K_GM, sum K_EM.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "context.h"
#include "device_common.h"
#include "net_grad.h"

namespace pdd {

namespace {

constexpr int BLK = 256;
constexpr int REC = 5;               // per-path record width

struct CalArgs {
  AsmParams P;                       // geometry, coefficients, step, stream, gradient table
  int64_t n;                         // knots
  int32_t n_paths;                   // N0' paths per knot
  const double* u0;                  // warm-up knot values
  uint32_t inst;                     // fourth Philox counter word
  double* rec;                       // REC doubles per path
  unsigned long long* counter;       // next path id (zeroed before the launch)
  int32_t claim;                     // path ids per claim
  const float4* cells;               // the gradient table by cells (nullable)
  // RBF interpolation of u0 (nullable: hat weights): per knot and side the
  // coefficients alpha = Phi^{-1} v of the interpolant of the stencil values
  // v (knot values, g at boundary lattice points), slot_len per side
  const double* alpha;
  int32_t slot_len;
};

// u0 at the exit point resolved from the flagged sides `fl` (bit o: side o)
template <int KIND, typename R, bool F64>
__device__ R exit_value(const AsmParams& P, const KnotDesc& d, const double* u0, const double* alpha, int SL, R x,
                        R y, uint32_t fl) {
  const bool fE = fl & 1u, fN = (fl >> 1) & 1u, fW = (fl >> 2) & 1u, fS = (fl >> 3) & 1u;
  const int o = choose_side<R>(x, y, fE, fN, fW, fS, d.line);
  const bool vert = (o == 0 || o == 2);
  const R along = vert ? y : x;
  const R lpos = (R)d.line[o];
  if ((d.bmask >> o) & 1) {
    const R a0 = vert ? (R)P.y0 : (R)P.x0, a1 = vert ? (R)P.y1 : (R)P.x1;
    const R pa = fmin(fmax(along, a0), a1);
    return vert ? g_at<KIND>(lpos, pa) : g_at<KIND>(pa, lpos);
  }
  if (alpha) {
    // RBF: u0(z) = sum_i alpha_i phi_c(|z - z_i|) over the side's stencil,
    // z the exit point clamped to the stencil, in float64
    const double da = vert ? P.dy : P.dx;
    const double a0 = vert ? P.y0 : P.x0;
    const int clo = d.clo[o], S = d.chi[o] - clo + 1;
    const double zd = fmin(fmax(((double)along - a0) / da, (double)clo), (double)d.chi[o]) * da;
    const double* a = alpha + ((size_t)d.knot * 4 + o) * SL;
    double acc = 0.0;
    for (int i = 0; i < S; ++i) {
      const double rr = zd - (double)(clo + i) * da;
      acc = fma(a[i], rsqrt_f64(fma(rr, rr, P.rbf_c2)), acc);
    }
    return (R)acc;
  }
  int q0;
  R w;
  hat_weights<R, F64>(along, vert ? (R)P.y0 : (R)P.x0, vert ? P.dy : P.dx, vert ? P.inv_dy : P.inv_dx, d.clo[o],
                      d.chi[o], q0, w);
  R val = 0;
  for (int e = 0; e < 2; ++e) {
    const int q = q0 + e;
    R v;
    if (q == 0 || q == P.L) {
      const R qc = vert ? (R)P.y0 + (R)q * (R)P.dy : (R)P.x0 + (R)q * (R)P.dx;
      v = vert ? g_at<KIND>(lpos, qc) : g_at<KIND>(qc, lpos);
    } else {
      const int lx = vert ? d.at[o] : q, ly = vert ? q : d.at[o];
      v = (R)u0[P.lattice[(size_t)ly * (P.L + 1) + lx]];
    }
    {
#pragma clang fp contract(off)
      val = val + (e == 0 ? (R)1 - w : w) * v;
    }
  }
  return val;
}

// Persistent: each wave claims up to 64 path ids at a time from a device counter
// and starts them in its idle lanes (once at least REFILL are idle, or all of
// them).  Both kinds of exit are queued in LDS, the path going on or its lane
// taking the next one, and their values are computed for 64 exits together: u0
// at an exit is a loop over the stencil with RBF weights, and a lane that waited
// for it would step no further.  A path's arithmetic is independent of which
// lane runs it, so the records do not depend on the schedule.
// What bounds it with a gradient table: the L1's requests to L2, two per step and
// lane (1.2 TB in 46 ms for EQ43, 1025 nodes; 207 G/s of some
// 300 G/s, VALU busy 62 %), hence the cells below; without one, VALU issue and the
// longest paths.  11,241 knots x 1000 paths of 421 steps (EQ43, table, RBF weights):
// 51.9 ms with every exit kept in its lane until 16 waited, 45.8 with the queue,
// 38.2 with the cells, with half the requests to L2 and VALU busy 85 %: VALU issue
// bounds that form.  POISSON, 2000 paths of hat weights a knot: 2.54 and 1.29.
// REFILL 4, 8, 16: 46.3, 45.4, 45.8 there, and 1.00, 0.98, 0.93 ms for 209 paths a
// knot, where starting a path (its thresholds in float64) counts.
constexpr int REFILL = 16;
constexpr int64_t CLAIMS = 8;
// the gradient table by cells (calibrate_cell_bytes)
constexpr int64_t CELLS_MAX = 11584;  // per direction: byte offsets in 32 bits
constexpr double CELLS_PATCH = 2e6, CELLS_STEPS = 300.0;
constexpr int64_t CELLS_PATHS = 4000000;
constexpr int QCAP = 64 + 128;       // fewer than 64 waiting, and two exits per lane

// The gradient table cell by cell, its four nodes in 32 aligned bytes: one L1
// access and one L2 request where the table's two rows take two.  Cell (i, j)
// holds the nodes (i, j), (i + 1, j), (i, j + 1), (i + 1, j + 1).
__global__ __launch_bounds__(BLK) void k_calib_cells(const float* __restrict__ table, int32_t n,
                                                     float4* __restrict__ cells) {
  const int64_t m = n - 1;
  for (int64_t q = (int64_t)blockIdx.x * BLK + threadIdx.x; q < m * m; q += (int64_t)gridDim.x * BLK) {
    const int64_t j = q / m, i = q - j * m;
    const float2* lo = reinterpret_cast<const float2*>(table) + j * n + i;
    const float2* hi = lo + n;
    cells[2 * q] = make_float4(lo[0].x, lo[0].y, lo[1].x, lo[1].y);
    cells[2 * q + 1] = make_float4(hi[0].x, hi[0].y, hi[1].x, hi[1].y);
  }
}

// grad_lut over the cells: the same bits
__device__ __forceinline__ void grad_cell(const AsmParams& P, const float4* cells, float x, float y, float& gx,
                                          float& gy) {
  const int n = P.cv_lut_n;
  const float fx = clamp_node((x - P.coef.x0f) * P.cv_lut_sx, (float)(n - 1));
  const float fy = clamp_node((y - P.coef.y0f) * P.cv_lut_sy, (float)(n - 1));
  const int i = min((int)fx, n - 2), j = min((int)fy, n - 2);
  const float tx = fx - (float)i, ty = fy - (float)j;
  const uint32_t at = (__umul24((uint32_t)j, (uint32_t)(n - 1)) + (uint32_t)i) * 32u;   // (below 4 GiB)
  const char* base = reinterpret_cast<const char*>(cells);
  const float4 a = *reinterpret_cast<const float4*>(base + at);
  const float4 b = *reinterpret_cast<const float4*>(base + at + 16);
  const float lx = a.x + tx * (a.z - a.x), hx = b.x + tx * (b.z - b.x);
  const float ly = a.y + tx * (a.w - a.y), hy = b.y + tx * (b.w - b.y);
  gx = lx + ty * (hx - lx);
  gy = ly + ty * (hy - ly);
}

template <typename R>
struct CalExit {
  R x, y, Y, Z;
};

// CV: 0 none, 1 the gradient table, 2 its cells
template <int KIND, bool F64, int CV>
__device__ __forceinline__ void calibrate_body(const CalArgs& C) {
  using R = typename std::conditional<F64, double, float>::type;
  using Desc = typename std::conditional<CV == 2, const KnotDesc&, const KnotDesc>::type;
  __shared__ CalExit<R> queue[BLK / 64][QCAP];
  __shared__ int64_t queue_id[BLK / 64][QCAP];
  __shared__ uint32_t queue_kf[BLK / 64][QCAP];
  const AsmParams& P = C.P;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t total = C.n * C.n_paths;
  const R h = (R)P.h, sq = (R)P.sqrt_h;
  CalExit<R>* Q = queue[wid];
  int64_t* Qi = queue_id[wid];
  uint32_t* Qk = queue_kf[wid];
  int qn = 0;
  // the values of the last `count` queued exits; K << 5 | naive << 4 | flags
  auto resolve = [&](int count) __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    qn -= count;
    if (lane < count) {
      const CalExit<R> r = Q[qn + lane];
      const int64_t id = Qi[qn + lane];
      const uint32_t kf = Qk[qn + lane];
      Desc d = P.desc[id / C.n_paths];
      const R phi = r.Z + r.Y * exit_value<KIND, R, F64>(P, d, C.u0, C.alpha, C.slot_len, r.x, r.y, kf & 15u);
      double* out = C.rec + id * REC + (kf >> 4 & 1u);
      out[0] = (double)phi;
      out[3] = (double)(kf >> 5);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  int64_t next = 0, stop = 0;        // claimed ids
  bool active = false, gm_done = false;
  int64_t gid = 0;
  uint32_t k = 0, p = 0, j = 0;
  R egm[4], env[4];
  const double* line = nullptr;      // the knot's side lines (global; read by the table family's GM test)
  R x = 0, y = 0, Y = 0, Z = 0, Xi = 0;
  while (true) {
    // ---- refill idle lanes with the next path ids -----------------------
    const uint64_t idle = __ballot(!active);
    const int n_idle = __popcll(idle);
    if (n_idle >= REFILL) {
      if (next == stop && stop < total) {
        const int claim = max(C.claim, n_idle);
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(C.counter, (unsigned long long)claim);
        base = ((unsigned long long)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32) |
               (unsigned)__builtin_amdgcn_readfirstlane((int)(base & 0xffffffffull));
        next = min((int64_t)base, total);
        stop = min((int64_t)base + claim, total);
      }
      if (next < stop) {
        const int take = (int)min((int64_t)n_idle, stop - next);
        const int rank = __popcll(idle & below);
        if (!active && rank < take) {
          gid = next + rank;
          k = (uint32_t)(gid / C.n_paths);
          p = (uint32_t)(gid - (int64_t)k * C.n_paths);
          Desc d = P.desc[k];
          for (int o = 0; o < 4; ++o) {
            egm[o] = exit_threshold<KIND, R>(P.coef, PDD_EXIT_GM, P.sqrt_h, d, o);
            env[o] = exit_threshold<KIND, R>(P.coef, PDD_EXIT_NAIVE, P.sqrt_h, d, o);
          }
          line = P.desc[k].line;
          x = (R)d.sx; y = (R)d.sy; Y = 1; Z = 0; Xi = 0;
          j = 0;
          gm_done = false;
          active = true;
        }
        next += take;
      } else if (idle == ~0ull) {
        break;                       // every id is claimed, every path has ended
      }
    }
    // ---- one draw, up to two steps ------------------------------------------
    U4 r{};
    if (active) r = philox10(j, p, k, C.inst, P.key0, P.key1);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint32_t fl_gm = 0, fl_em = 0;
      const uint32_t K = 2 * j + half + 1;
      if (active) {
        R z0, z1;
        if constexpr (F64) box_muller(uniform64(half ? r.c : r.a), uniform64(half ? r.d : r.b), z0, z1);
        else box_muller(uniform32(half ? r.c : r.a), uniform32(half ? r.d : r.b), z0, z1);
        R gx = 0, gy = 0;
        if constexpr (CV == 2) grad_cell(P, C.cells, x, y, gx, gy);
        else if constexpr (CV == 1) grad_lut(P, x, y, gx, gy);
        em_step<KIND, R, CV != 0>(P.coef, h, sq, z0, z1, x, y, Y, Z, gx, gy, &Xi);
        if (!gm_done) fl_gm = exit_sides<KIND, R>(P.coef, PDD_EXIT_GM, sq, line, egm, x, y);
        fl_em = exit_sides<KIND, R>(P.coef, PDD_EXIT_NAIVE, sq, line, env, x, y);
        if (K >= (1u << 24) - 2 && fl_em == 0) {         // step cap: every side flagged
          if (!gm_done && fl_gm == 0) fl_gm = 15u;
          fl_em = 15u;
        }
      }
      const uint64_t mg = __ballot(fl_gm != 0), me = __ballot(fl_em != 0);
      if ((mg | me) != 0) {
        const int ng = __popcll(mg);
        if (fl_gm != 0) {
          const int q = qn + __popcll(mg & below);
          Q[q] = CalExit<R>{x, y, Y, Z};
          Qi[q] = gid;
          Qk[q] = K << 5 | fl_gm;
          C.rec[gid * REC + 2] = (double)Xi;
          gm_done = true;
        }
        if (fl_em != 0) {
          const int q = qn + ng + __popcll(me & below);
          Q[q] = CalExit<R>{x, y, Y, Z};
          Qi[q] = gid;
          Qk[q] = K << 5 | 16u | fl_em;
          if (!gm_done) {            // no GM exit at all (a NaN sigma at the side): counted as zeros
            double* out = C.rec + gid * REC;
            out[0] = out[2] = out[3] = 0.0;
          }
          active = false;
        }
        qn += ng + __popcll(me);
      }
    }
    ++j;
    while (qn >= 64) resolve(64);
  }
  if (qn > 0) resolve(qn);
}

template <int KIND, bool F64, bool CVON>
__global__ __launch_bounds__(BLK) void k_calibrate(CalArgs C) {
  calibrate_body<KIND, F64, CVON ? 1 : 0>(C);
}
template <int KIND>
__global__ __launch_bounds__(BLK) void k_calibrate_cells(CalArgs C) {
  calibrate_body<KIND, false, 2>(C);
}

// The RBF coefficients of u0 on every interface side: one wave per (knot,
// side); the stencil values in LDS, then alpha_i = sum_j (Phi^{-1})_ji v_j
// (Phi^{-1} symmetric: lane i reads column i).
template <int KIND>
__global__ __launch_bounds__(256) void k_calib_alpha(AsmParams P, int64_t n, int32_t SL, const double* u0,
                                                     double* alpha) {
  extern __shared__ double vs[];
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (w >= 4 * n) return;
  const int64_t k = w >> 2;
  const int o = (int)(w & 3);
  const KnotDesc& d = P.desc[k];
  if ((d.bmask >> o) & 1) return;
  double* v = vs + (size_t)(threadIdx.x >> 6) * SL;
  const bool vert = (o == 0 || o == 2);
  const int clo = d.clo[o], S = d.chi[o] - clo + 1;
  for (int i = lane; i < S; i += 64) {
    const int q = clo + i;
    if (q == 0 || q == P.L) {
      const double qc = vert ? P.y0 + (double)q * P.dy : P.x0 + (double)q * P.dx;
      v[i] = vert ? g_at<KIND>(d.line[o], qc) : g_at<KIND>(qc, d.line[o]);
    } else {
      const int lx = vert ? d.at[o] : q, ly = vert ? q : d.at[o];
      v[i] = u0[P.lattice[(size_t)ly * (P.L + 1) + lx]];
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const double* Mi = P.rbf_inv + (vert ? P.rbf_half : 0) + rbf_block_offset(S);
  for (int i = lane; i < S; i += 64) {
    double acc = 0.0;
    for (int j = 0; j < S; ++j) acc = fma(Mi[(size_t)j * S + i], v[j], acc);
    alpha[(size_t)w * SL + i] = acc;
  }
}

template <int KIND>
hipError_t launch_alpha_kind(const AsmParams& P, int64_t n, int32_t SL, const double* u0, double* alpha,
                             hipStream_t stream) {
  const int64_t waves = 4 * n;
  const unsigned grid = (unsigned)((waves + 3) / 4);
  const size_t lds = (size_t)4 * SL * sizeof(double);
  hipLaunchKernelGGL((k_calib_alpha<KIND>), dim3(grid), dim3(256), lds, stream, P, n, SL, u0, alpha);
  return hipGetLastError();
}

hipError_t launch_alpha(const AsmParams& P, int64_t n, int32_t SL, const double* u0, double* alpha,
                        hipStream_t stream) {
  switch (P.coef.kind) {
    case PDD_COEF_POISSON: return launch_alpha_kind<PDD_COEF_POISSON>(P, n, SL, u0, alpha, stream);
    case PDD_COEF_VARCOEF: return launch_alpha_kind<PDD_COEF_VARCOEF>(P, n, SL, u0, alpha, stream);
    case PDD_COEF_AMPLITUDE: return launch_alpha_kind<PDD_COEF_AMPLITUDE>(P, n, SL, u0, alpha, stream);
    case PDD_COEF_LUT: return launch_alpha_kind<PDD_COEF_LUT>(P, n, SL, u0, alpha, stream);
    case PDD_COEF_CONSTSOL: return launch_alpha_kind<PDD_COEF_CONSTSOL>(P, n, SL, u0, alpha, stream);
    case PDD_COEF_EQ43: return launch_alpha_kind<PDD_COEF_EQ43>(P, n, SL, u0, alpha, stream);
    default: return launch_alpha_kind<PDD_COEF_EXITTIME>(P, n, SL, u0, alpha, stream);
  }
}

__global__ void k_zero_counter(unsigned long long* c) {
  if (threadIdx.x == 0) *c = 0ull;
}

// Per-knot sums of the path records: one wave per knot, lane l takes paths
// l, l + 64, ... in order, then a fixed butterfly across the lanes.
__global__ __launch_bounds__(BLK) void k_calibrate_sum(const double* __restrict__ rec, int64_t n, int32_t n_paths,
                                                       double* __restrict__ stats) {
  const int lane = threadIdx.x & 63;
  const int64_t k = (int64_t)blockIdx.x * (BLK / 64) + (threadIdx.x >> 6);
  if (k >= n) return;
  double s[PDD_CAL_WIDTH] = {};
  for (int32_t p = lane; p < n_paths; p += 64) {
    const double* r = rec + ((size_t)k * n_paths + p) * REC;
    s[0] += r[1] - r[0];
    s[1] += r[0];
    s[2] += r[0] * r[0];
    s[3] += r[2];
    s[4] += r[2] * r[2];
    s[5] += r[0] * r[2];
    s[6] += r[3];
    s[7] += r[4];
  }
#pragma unroll
  for (int i = 0; i < PDD_CAL_WIDTH; ++i) {
    for (int off = 32; off > 0; off >>= 1) s[i] += __shfl_xor(s[i], off, 64);
  }
  if (lane < PDD_CAL_WIDTH) {
    double v = s[0];
#pragma unroll
    for (int i = 1; i < PDD_CAL_WIDTH; ++i) if (lane == i) v = s[i];
    stats[k * PDD_CAL_WIDTH + lane] = v;
  }
}

template <int KIND, bool F64>
hipError_t launch_kind(CalArgs C, bool cv, hipStream_t stream) {
  // persistent grid: enough workgroups to fill the device, fewer for small runs
  const int64_t threads = C.n * C.n_paths;
  const unsigned grid = (unsigned)std::min<int64_t>((threads + BLK - 1) / BLK, 2048);
  // several claims per wave, of a wave's lanes at most
  C.claim = (int32_t)std::min<int64_t>(64, std::max<int64_t>(1, threads / ((int64_t)grid * (BLK / 64) * CLAIMS)));
  if constexpr (!F64) {
    if (C.cells) {
      hipLaunchKernelGGL((k_calibrate_cells<KIND>), dim3(grid), dim3(BLK), 0, stream, C);
      return hipGetLastError();
    }
  }
  if (cv) hipLaunchKernelGGL((k_calibrate<KIND, F64, true>), dim3(grid), dim3(BLK), 0, stream, C);
  else hipLaunchKernelGGL((k_calibrate<KIND, F64, false>), dim3(grid), dim3(BLK), 0, stream, C);
  return hipGetLastError();
}

template <bool F64>
hipError_t launch_prec(const CalArgs& C, bool cv, hipStream_t stream) {
  switch (C.P.coef.kind) {
    case PDD_COEF_POISSON: return launch_kind<PDD_COEF_POISSON, F64>(C, cv, stream);
    case PDD_COEF_VARCOEF: return launch_kind<PDD_COEF_VARCOEF, F64>(C, cv, stream);
    case PDD_COEF_AMPLITUDE: return launch_kind<PDD_COEF_AMPLITUDE, F64>(C, cv, stream);
    case PDD_COEF_LUT: return launch_kind<PDD_COEF_LUT, F64>(C, cv, stream);
    case PDD_COEF_CONSTSOL: return launch_kind<PDD_COEF_CONSTSOL, F64>(C, cv, stream);
    case PDD_COEF_EQ43: return launch_kind<PDD_COEF_EQ43, F64>(C, cv, stream);
    default: return launch_kind<PDD_COEF_EXITTIME, F64>(C, cv, stream);
  }
}

}  // namespace

// The cells pay for many long paths whose patch, about two cells of the partition
// wide, still fits half an XCD's L2 in their four times larger form (table as it is
// against cells, ms): EQ43, 1025 nodes over 10 cells, 11.2 M paths of 421 steps
// 46.8, 38.2; AMPLITUDE, 513 over 6, 62 steps, 5.7 M paths 3.57, 2.97, 1.5 M 1.57,
// 1.59, 0.4 M 0.94, 0.99; VARCOEF, 1025 over 6 (3.7 MB a patch), 5.7 M of 64 steps
// 4.33, 4.57; 1025 over 10, 10.7 M of 24 steps 3.17, 3.25.
size_t calibrate_cell_bytes(const AsmParams& P, int precision, int64_t paths, double cell_steps, int32_t H) {
  if (P.cv_mode != PDD_CV_GRAD_LUT || precision == PDD_FP64_SAME_STREAM) return 0;
  const int64_t m = P.cv_lut_n - 1;
  const double patch = 2.0 * (double)m / H;
  if (m > CELLS_MAX || patch * patch * 2 * sizeof(float4) > CELLS_PATCH || cell_steps < CELLS_STEPS ||
      paths < CELLS_PATHS)
    return 0;
  return (size_t)(m * m) * 2 * sizeof(float4);
}

// the path records, then the path counter (256-byte aligned), then the cells
size_t calibrate_scratch_bytes(int64_t n, int32_t n_paths) {
  return ((size_t)n * n_paths * REC * sizeof(double) + 255) / 256 * 256 + 256;
}

hipError_t launch_calibrate(const AsmParams& P, int precision, int64_t n, int32_t n_paths, uint32_t inst,
                            const double* u0, double* rec, double* stats, hipStream_t stream, bool cells,
                            double* alpha, int32_t slot_len) {
  CalArgs C;
  C.alpha = alpha;
  C.slot_len = slot_len;
  if (alpha) {
    const hipError_t e = launch_alpha(P, n, slot_len, u0, alpha, stream);
    if (e != hipSuccess) return e;
  }
  C.P = P;
  C.n = n;
  C.n_paths = n_paths;
  C.u0 = u0;
  C.inst = inst;
  C.rec = rec;
  C.counter = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(rec) +
                                                    ((size_t)n * n_paths * REC * sizeof(double) + 255) / 256 * 256);
  C.cells = nullptr;
  if (cells) {
    const int64_t m = P.cv_lut_n - 1;
    float4* to = reinterpret_cast<float4*>(reinterpret_cast<char*>(rec) + calibrate_scratch_bytes(n, n_paths));
    hipLaunchKernelGGL(k_calib_cells, dim3((unsigned)std::min<int64_t>(4096, (m * m + BLK - 1) / BLK)), dim3(BLK), 0, stream,
                       P.cv_lut, P.cv_lut_n, to);
    C.cells = to;
  }
  hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(64), 0, stream, C.counter);
  const bool cv = P.cv_mode == PDD_CV_GRAD_LUT;
  hipError_t e = precision == PDD_FP64_SAME_STREAM ? launch_prec<true>(C, cv, stream) : launch_prec<false>(C, cv, stream);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)((n + BLK / 64 - 1) / (BLK / 64));
  hipLaunchKernelGGL(k_calibrate_sum, dim3(grid), dim3(BLK), 0, stream, rec, n, n_paths, stats);
  return hipGetLastError();
}

}  // namespace pdd
