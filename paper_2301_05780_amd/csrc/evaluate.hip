// Point values inside the subdomains once the knot values are known.
//
// Each subdomain square is an independent Dirichlet problem for (6) whose
// sides carry u: the solved knot values interpolated along the grid lines on
// interfaces, g on the domain boundary (Sec. 3.3).  The value at a point is
// the Feynman-Kac expectation of eq. (8) over paths started there and
// absorbed at the square's boundary, with the assembly's Euler-Maruyama step,
// exit rules and side choice; the exit value is g at the projection on a
// boundary side, else the hat interpolation of the side line's lattice values
// with the along-side coordinate clamped to the side.
//
// Work split.  A point's paths are cut into `waves_per_pt` contiguous ranges,
// one wave each (see eval_split), and a lane whose path has exited starts the
// range's next path at once, as in the assembly: exits are queued in LDS and
// resolved (side choice, side value) 64 at a time with every lane busy.  The
// lanes keep float64 sums of the score and its square; a fixed butterfly
// combines the lanes and, with several waves per point, a second kernel the
// waves in order (deterministic).  Bound by VALU issue, as the assembly:
// 20,000 points of 500 paths run at 2.9e11 path-steps/s.  1000 points of 4000
// VARCOEF paths of about a dozen steps: 0.22 ms (one wave per point, each
// lane's paths in step with the wave's longest: 1.45 ms).
// Stream: counter (draw, path, point, instance + 2^31).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "context.h"
#include "device_common.h"

namespace pdd {

namespace {

constexpr int BLK = 256;
constexpr uint32_t MAX_STEPS = (1u << 24) - 2;
constexpr uint32_t POINT_STREAM = 1u << 31;
constexpr int QCAP = 128;        // queued exits per wave (resolved at >= 64)
// Idle lanes that start new paths (or all of them); measured on paths of 12
// and 44 steps: 1 within 1 %, 8 1 %, 16 4 % slower.
constexpr int REFILL = 4;

struct EvalArgs {
  AsmParams P;                 // geometry, coefficients, step and stream parameters
  int32_t H, m;                // subdomains per direction, lattice intervals per side
  int64_t n_pts;
  int64_t n_paths;
  uint32_t inst;               // fourth counter word (POINT_STREAM already added)
  const double* xy;
  const double* u_knots;
  double* u;
  double* se;
  int32_t waves_per_pt;
  double* part;                // waves_per_pt > 1: per wave, sums of s and s^2
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// u on the grid line of side o of the square: g on a boundary line, else hat
// interpolation of the lattice values (points of the domain boundary take g).
template <int KIND, typename R, bool F64>
__device__ __forceinline__ R line_value(const EvalArgs& A, const KnotDesc& d, int o, R along) {
  const AsmParams& P = A.P;
  const bool vert = (o == 0 || o == 2);
  const R lpos = (R)d.line[o];
  const int lo = d.clo[o], hi = d.chi[o];
  if ((d.bmask >> o) & 1) {
    const R a_lo = vert ? (R)(P.y0 + (double)lo * P.dy) : (R)(P.x0 + (double)lo * P.dx);
    const R a_hi = vert ? (R)(P.y0 + (double)hi * P.dy) : (R)(P.x0 + (double)hi * P.dx);
    const R pa = fmin(fmax(along, a_lo), a_hi);
    return vert ? g_at<KIND>(lpos, pa) : g_at<KIND>(pa, lpos);
  }
  int q0;
  R w;
  hat_weights<R, F64>(along, vert ? (R)P.y0 : (R)P.x0, vert ? P.dy : P.dx, vert ? P.inv_dy : P.inv_dx, lo, hi, q0, w);
  R v[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int q = q0 + e;
    if (q == 0 || q == P.L) {
      const R qc = vert ? (R)P.y0 + (R)q * (R)P.dy : (R)P.x0 + (R)q * (R)P.dx;
      v[e] = vert ? g_at<KIND>(lpos, qc) : g_at<KIND>(qc, lpos);
    } else {
      const int at = d.at[o];
      const int lx = vert ? at : q, ly = vert ? q : at;
      v[e] = (R)A.u_knots[P.lattice[(size_t)ly * (P.L + 1) + lx]];
    }
  }
  R out;
  {
#pragma clang fp contract(off)
    out = ((R)1 - w) * v[0] + w * v[1];
  }
  return out;
}

// u and its standard error from the sums over all paths of the point
__device__ __forceinline__ void write_point(const EvalArgs& A, int64_t pt, double s1, double s2) {
  const double N = (double)A.n_paths;
  const double mean = s1 / N;
  A.u[pt] = mean;
  if (A.se) A.se[pt] = sqrt(fmax(s2 / N - mean * mean, 0.0) / N);
}

// A point whose value needs no paths (outside the domain, or on its square's
// boundary): written as it is, or left for k_eval_sum in the wave's slot, the
// sum of squares marking it (-1: se = 0, -2: se = NaN).
__device__ __forceinline__ void no_paths(const EvalArgs& A, int64_t pt, int64_t wave, double v, double se) {
  if (A.part) {
    A.part[2 * wave] = v;
    A.part[2 * wave + 1] = isnan(se) ? -2.0 : -1.0;
  } else {
    A.u[pt] = v;
    if (A.se) A.se[pt] = se;
  }
}

template <typename R>
struct EvalExit {
  R x, y, Y, Z;
};

template <int KIND, bool F64>
__global__ __launch_bounds__(BLK) void k_eval(EvalArgs A) {
  using R = typename std::conditional<F64, double, float>::type;
  __shared__ EvalExit<R> queue[BLK / 64][QCAP];
  __shared__ uint32_t queue_fl[BLK / 64][QCAP];
  const AsmParams& P = A.P;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t wave = (int64_t)blockIdx.x * (BLK / 64) + wid;
  // (several waves per point: few points, and the wave's number has 32 bits)
  const bool split = A.waves_per_pt > 1;
  const int64_t pt = split ? (int64_t)((uint32_t)wave / (uint32_t)A.waves_per_pt) : wave;
  if (pt >= A.n_pts) return;
  const double px = A.xy[2 * pt], py = A.xy[2 * pt + 1];
  if (!(px >= P.x0 && px <= P.x1 && py >= P.y0 && py <= P.y1)) {
    if (lane == 0) no_paths(A, pt, wave, NAN, NAN);
    return;
  }
  // the square holding the point and its description as a "patch"
  const int m = A.m, H = A.H, L = P.L;
  const int a = max(min((int)floor((px - P.x0) / (P.dx * (double)m)), H - 1), 0);
  const int c = max(min((int)floor((py - P.y0) / (P.dy * (double)m)), H - 1), 0);
  const int xlo = a * m, xhi = xlo + m, ylo = c * m, yhi = ylo + m;
  KnotDesc d;
  d.sx = px;
  d.sy = py;
  d.line[0] = P.x0 + (double)xhi * P.dx;
  d.line[1] = P.y0 + (double)yhi * P.dy;
  d.line[2] = P.x0 + (double)xlo * P.dx;
  d.line[3] = P.y0 + (double)ylo * P.dy;
  d.at[0] = xhi; d.at[1] = yhi; d.at[2] = xlo; d.at[3] = ylo;
  d.clo[0] = d.clo[2] = ylo; d.chi[0] = d.chi[2] = yhi;
  d.clo[1] = d.clo[3] = xlo; d.chi[1] = d.chi[3] = xhi;
  d.bmask = (xhi == L ? 1 : 0) | (yhi == L ? 2 : 0) | (xlo == 0 ? 4 : 0) | (ylo == 0 ? 8 : 0);
  d.knot = (int32_t)pt;

  // a point on the square's boundary takes the line value directly
  const bool on_v = px == d.line[2] || px == d.line[0];
  const bool on_h = py == d.line[3] || py == d.line[1];
  if (on_v || on_h) {
    if (lane == 0) {
      const int o = on_v ? (px == d.line[2] ? 2 : 0) : (py == d.line[3] ? 3 : 1);
      no_paths(A, pt, wave, (double)line_value<KIND, R, F64>(A, d, o, on_v ? (R)py : (R)px), 0.0);
    }
    return;
  }

  R e[4];
#pragma unroll
  for (int o = 0; o < 4; ++o) e[o] = exit_threshold<KIND, R>(P.coef, P.exit_rule, P.sqrt_h, d, o);
  const R h = (R)P.h, sq = (R)P.sqrt_h;
  double s1 = 0.0, s2 = 0.0;
  EvalExit<R>* Q = queue[wid];
  uint32_t* Qf = queue_fl[wid];
  int qn = 0;                            // queued exits
  // this wave's range of the point's paths
  uint32_t next = 0, end = (uint32_t)A.n_paths;
  if (split) {
    const int64_t part = wave - pt * A.waves_per_pt;
    next = (uint32_t)(A.n_paths * part / A.waves_per_pt);
    end = (uint32_t)(A.n_paths * (part + 1) / A.waves_per_pt);
  }
  // the score of a path that ended at (x, y) with the sides `fl` flagged
  auto score = [&](R x, R y, R Y, R Z, uint32_t fl) __attribute__((always_inline)) {
    const int o = choose_side<R>(x, y, fl & 1u, (fl >> 1) & 1u, (fl >> 2) & 1u, (fl >> 3) & 1u, d.line);
    const bool vert = (o == 0 || o == 2);
    R s;
    if (isnan(x) || isnan(y)) {
      s = (R)NAN;
    } else {
      const R val = line_value<KIND, R, F64>(A, d, o, vert ? y : x);
      {
#pragma clang fp contract(off)
        s = Z + Y * val;
      }
    }
    s1 += (double)s;
    s2 += (double)s * (double)s;
  };
  // draw j of path p, up to two steps: the flagged sides (0: goes on)
  auto step_pair = [&](uint32_t p, uint32_t& j, R& x, R& y, R& Y, R& Z) __attribute__((always_inline)) -> uint32_t {
    const U4 r = philox10(j, p, (uint32_t)pt, A.inst, P.key0, P.key1);
    R z0, z1;
    if constexpr (F64) box_muller(uniform64(r.a), uniform64(r.b), z0, z1);
    else box_muller(uniform32(r.a), uniform32(r.b), z0, z1);
    em_step<KIND, R>(P.coef, h, sq, z0, z1, x, y, Y, Z);
    uint32_t fl = exit_sides<KIND, R>(P.coef, P.exit_rule, sq, d.line, e, x, y);
    if (fl == 0) {
      if constexpr (F64) box_muller(uniform64(r.c), uniform64(r.d), z0, z1);
      else box_muller(uniform32(r.c), uniform32(r.d), z0, z1);
      em_step<KIND, R>(P.coef, h, sq, z0, z1, x, y, Y, Z);
      fl = exit_sides<KIND, R>(P.coef, P.exit_rule, sq, d.line, e, x, y);
    }
    ++j;
    if (fl == 0 && 2 * j >= MAX_STEPS) fl = 15u;
    return fl;
  };
  auto resolve = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < qn; i += 64) {
      const EvalExit<R> r = Q[i];
      score(r.x, r.y, r.Y, r.Z, Qf[i]);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    qn = 0;
  };
  bool active = false;
  R x = 0, y = 0, Y = 0, Z = 0;
  uint32_t p = 0, j = 0;
  // A path per lane: nothing to refill or to wait for, and the queue would only cost
  // (1000 points of 64 paths: 43 us, 55 with it)
  if (end - next <= 64u) {
    if (next + lane < end) {
      x = (R)px; y = (R)py; Y = (R)1;
      uint32_t fl = 0;
      while (fl == 0) fl = step_pair(next + lane, j, x, y, Y, Z);
      score(x, y, Y, Z, fl);
    }
    next = end;
  }
  while (true) {
    const uint64_t idle = __ballot(!active);
    const int n_idle = __popcll(idle);
    if (next < end && (n_idle >= REFILL || idle == ~0ull)) {
      const uint32_t take = min((uint32_t)n_idle, end - next);
      const uint32_t rank = (uint32_t)__popcll(idle & ((1ull << lane) - 1ull));
      if (!active && rank < take) {
        p = next + rank;
        x = (R)px; y = (R)py; Y = (R)1; Z = (R)0;
        j = 0;
        active = true;
      }
      next += take;
    } else if (idle == ~0ull) {
      break;                             // every path handed out and ended
    }
    uint32_t fl = 0;
    if (active) fl = step_pair(p, j, x, y, Y, Z);
    const uint64_t em = __ballot(fl != 0);
    if (em != 0) {
      if (fl != 0) {
        const int i = qn + __popcll(em & ((1ull << lane) - 1ull));
        Q[i] = EvalExit<R>{x, y, Y, Z};
        Qf[i] = fl;
        active = false;
      }
      qn += __popcll(em);
      if (qn >= 64) resolve();
    }
  }
  if (qn > 0) resolve();
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  if (lane == 0) {
    if (A.part) {
      A.part[2 * wave] = s1;
      A.part[2 * wave + 1] = s2;
    } else {
      write_point(A, pt, s1, s2);
    }
  }
}

// The waves' sums of a point, in wave order (see no_paths for the marks).
__global__ __launch_bounds__(BLK) void k_eval_sum(EvalArgs A) {
  const int64_t pt = (int64_t)blockIdx.x * BLK + threadIdx.x;
  if (pt >= A.n_pts) return;
  const double* part = A.part + 2 * pt * A.waves_per_pt;
  if (part[1] < 0.0) {
    A.u[pt] = part[0];
    if (A.se) A.se[pt] = part[1] == -1.0 ? 0.0 : NAN;
    return;
  }
  double s1 = 0.0, s2 = 0.0;
  for (int w = 0; w < A.waves_per_pt; ++w) {
    s1 += part[2 * w];
    s2 += part[2 * w + 1];
  }
  write_point(A, pt, s1, s2);
}

// Waves per point: enough waves to fill the device (EVAL_WAVES, six per SIMD),
// each with about 64 paths at least; fewer than 128 stay together, as half-empty
// waves and the second kernel cost more than they give (5000 points of 80 paths, 4
// steps: 44 us in two waves each, 35 in one; 3000 of 65 34, 27).  More, shorter ranges idle more lanes while a
// range's last paths end; fewer leave SIMDs without work: 4096, 6144, 8192 and
// 12288 waves take 0.375, 0.41, 0.42 and 0.51 ms for 50 points of 20,000
// paths, and 0.241, 0.232, 0.229 and 0.229 ms for 1000 points of 4000.
constexpr int64_t EVAL_WAVES = 6144;
int32_t eval_split(int64_t n_pts, int64_t n_paths) {
  const int64_t fill = (EVAL_WAVES + n_pts - 1) / n_pts, most = n_paths < 128 ? 1 : (n_paths + 63) / 64;
  return (int32_t)std::max<int64_t>(1, std::min(fill, most));
}

template <bool F64>
hipError_t launch_kind(const EvalArgs& A, unsigned grid, hipStream_t stream) {
  switch (A.P.coef.kind) {
    case PDD_COEF_POISSON: hipLaunchKernelGGL((k_eval<PDD_COEF_POISSON, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
    case PDD_COEF_VARCOEF: hipLaunchKernelGGL((k_eval<PDD_COEF_VARCOEF, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
    case PDD_COEF_AMPLITUDE: hipLaunchKernelGGL((k_eval<PDD_COEF_AMPLITUDE, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
    case PDD_COEF_LUT: hipLaunchKernelGGL((k_eval<PDD_COEF_LUT, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
    case PDD_COEF_CONSTSOL: hipLaunchKernelGGL((k_eval<PDD_COEF_CONSTSOL, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
    case PDD_COEF_EQ43: hipLaunchKernelGGL((k_eval<PDD_COEF_EQ43, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
    default: hipLaunchKernelGGL((k_eval<PDD_COEF_EXITTIME, F64>), dim3(grid), dim3(BLK), 0, stream, A); break;
  }
  return hipGetLastError();
}

}  // namespace

pdd_status run_eval_subdomain(pdd_ctx* ctx, const pdd_coeffs& co, const pdd_partition& part, const pdd_knots& kn,
                              const double* u_knots, int64_t n_pts, const double* xy, const pdd_run& run, double* u,
                              double* se) {
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return check_hip(ctx, e, "hipSetDevice");
  GeoCache* gc = nullptr;
  pdd_status st = get_geometry(ctx, part, kn, &gc);
  if (st != PDD_OK) return st;
  if ((st = get_lattice(ctx, gc)) != PDD_OK) return st;
  EvalArgs A;
  fill_asm_params(*gc, co, run, A.P);
  if ((st = prepare_lut_bound(ctx, co, run, A.P, false)) != PDD_OK) return st;
  A.H = part.H;
  A.m = kn.m;
  A.n_pts = n_pts;
  A.n_paths = run.n_paths;
  A.inst = run.instance + POINT_STREAM;
  A.xy = xy;
  A.u_knots = u_knots;
  A.u = u;
  A.se = se;
  A.waves_per_pt = eval_split(n_pts, run.n_paths);
  A.part = nullptr;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  // a captured call takes one wave per point, which needs no scratch
  if (hipStreamIsCapturing(ctx->stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusActive) A.waves_per_pt = 1;
  if (A.waves_per_pt > 1) {
    if ((st = ctx->eval_scratch.acquire(ctx, (size_t)n_pts * A.waves_per_pt * 2 * sizeof(double))) != PDD_OK) return st;
    A.part = ctx->eval_scratch.buf.as<double>();
  }
  const int64_t waves = n_pts * A.waves_per_pt;
  const unsigned grid = (unsigned)((waves + BLK / 64 - 1) / (BLK / 64));
  e = run.precision == PDD_FP64_SAME_STREAM ? launch_kind<true>(A, grid, ctx->stream)
                                            : launch_kind<false>(A, grid, ctx->stream);
  if (e == hipSuccess && A.part) {
    hipLaunchKernelGGL(k_eval_sum, dim3((unsigned)((n_pts + BLK - 1) / BLK)), dim3(BLK), 0, ctx->stream, A);
    if ((e = hipGetLastError()) == hipSuccess) return ctx->eval_scratch.release(ctx);
  }
  return check_hip(ctx, e, "launch eval_subdomain");
}

}  // namespace pdd
