// Training pairs for the control-variate network from the method's own paths.
//
// Path (knot k, p < paths_per_knot), float32, the same random stream and step
// as the production assembly, so the recorded points lie on the paths that
// build G and b.  The first `points_per_path` iterates X_n of each path are
// recorded with Y_n and Z_n; when the path exits at step K the value carried
// out of the patch is Z_K + Y_K u(exit), with u at the exit interpolated from
// the solved knot values u0 (hat weights on the exit line) or taken from the
// boundary datum, and each recorded point gets the tail score
// (Z_K + Y_K u(exit) - Z_n) / Y_n, whose conditional mean given X_n is u(X_n).
// Unused record slots get a NaN target.
//
// A point's target needs the end of its path, and a path is a few to a few
// hundred steps of which the first points_per_path are kept.  Holding or
// writing the points until the exit costs more than stepping them twice:
// every path is walked to its exit for its value and K, then its first
// min(K, points_per_path) steps again, the pairs staged in LDS and written out
// as contiguous runs of a path's slots.  Two forms with the same bits:
//   k_collect_whole   one launch, a path per lane from its start to its pairs
//   k_collect_start, _ends, _points
//                     the walk to the exit with lanes refilled and exits queued
//                     as in the assembly, the value and K kept per path; for
//                     many long paths, where a wave of single paths would wait
//                     for its longest one (collect_refills)
// Bound by VALU issue and the 12 B per slot, small calls by their longest path.
// Times in us (VARCOEF, 16 points; before: one thread per path writing every
// point's x, y, Y, Z on its own and reading Y, Z back; cell^2 / h steps):
//   paths, cell^2 / h     before   whole   refilled
//   2177, 31                23.8    21.5       33.7
//   299,250, 40              101      51         72
//   437,280, 20              112      42         70
//   3,997,875, 90           1764     534        616
//   299,250, 400             469     388        458
//   3,997,875, 400          1873    1662       1514
//   1,999,965, 1500         3090    3074       2469
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "context.h"
#include "device_common.h"

namespace pdd {

namespace {

constexpr int BLK = 256;
constexpr int QCAP = 128;            // queued exits per wave (resolved at >= 64)
constexpr int REFILL = 4;            // idle lanes that start new paths (or all of them)
constexpr int64_t COLLECT_WAVES = 6144;   // of k_collect_ends: six per SIMD
// The refilled form: from these numbers on (1.0 M paths of 1500: 1949 us against
// 1815 in one kernel, 2.0 M 2469 against 3074; 4.0 M of 400: 1514 against 1662,
// of 200: 1004 against 935)
constexpr double REFILL_STEPS = 300.0;
constexpr int64_t REFILL_PATHS = 1500000;

// What a path needs of its knot: start, and the strict exit thresholds.
struct CollectStart {
  float x, y;
  float pad0, pad1;
  float e[4];
};
static_assert(sizeof(CollectStart) == COLLECT_START_BYTES, "scratch sizes");

// A path's end: the value carried out of the patch, and K.
struct CollectEnd {
  float v;
  uint32_t K;
};
static_assert(sizeof(CollectEnd) == COLLECT_END_BYTES, "scratch sizes");

struct CollectArgs {
  AsmParams P;               // geometry, coefficients, step and stream parameters
  int64_t n;                 // knots
  int32_t paths_per_knot;
  int32_t points_per_path;
  const double* u0;          // solved knot values
  uint32_t inst;             // fourth Philox counter word
  CollectStart* start;       // scratch, per knot (null: the whole path in one kernel)
  CollectEnd* end;           // scratch, per path
  float* xy;                 // 2 per record slot
  float* target;             // per record slot
};

template <int KIND>
__global__ __launch_bounds__(BLK) void k_collect_start(CollectArgs C) {
  const int64_t k = (int64_t)blockIdx.x * BLK + threadIdx.x;
  if (k >= C.n) return;
  const KnotDesc& d = C.P.desc[k];
  CollectStart& s = C.start[k];
  s.x = (float)d.sx;
  s.y = (float)d.sy;
#pragma unroll
  for (int o = 0; o < 4; ++o) s.e[o] = exit_threshold<KIND, float>(C.P.coef, C.P.exit_rule, C.P.sqrt_h, d, o);
}

// The value carried out of the patch by a path that ended at (x, y) with Y, Z
// and the sides `fl` flagged.
template <int KIND>
__device__ __forceinline__ float exit_score(const CollectArgs& C, const KnotDesc& d, float x, float y, float Y, float Z,
                                            uint32_t fl) {
  const AsmParams& P = C.P;
  const bool fE = fl & 1u, fN = (fl >> 1) & 1u, fW = (fl >> 2) & 1u, fS = (fl >> 3) & 1u;
  const int o = choose_side<float>(x, y, fE, fN, fW, fS, d.line);
  const bool vert = (o == 0 || o == 2);
  const float along = vert ? y : x;
  const float lpos = (float)d.line[o];
  float uex;
  if ((d.bmask >> o) & 1) {
    const float a0 = vert ? (float)P.y0 : (float)P.x0, a1 = vert ? (float)P.y1 : (float)P.x1;
    const float pa = fminf(fmaxf(along, a0), a1);
    uex = vert ? g_at<KIND>(lpos, pa) : g_at<KIND>(pa, lpos);
  } else {
    int q0;
    float w;
    hat_weights<float, false>(along, vert ? (float)P.y0 : (float)P.x0, vert ? P.dy : P.dx,
                              vert ? P.inv_dy : P.inv_dx, d.clo[o], d.chi[o], q0, w);
    uex = 0.0f;
    for (int e = 0; e < 2; ++e) {
      const int q = q0 + e;
      const float wq = e == 0 ? 1.0f - w : w;
      float val;
      if (q == 0 || q == P.L) {
        const float qc = vert ? (float)P.y0 + (float)q * (float)P.dy : (float)P.x0 + (float)q * (float)P.dx;
        val = vert ? g_at<KIND>(lpos, qc) : g_at<KIND>(qc, lpos);
      } else {
        const int lx = vert ? d.at[o] : q, ly = vert ? q : d.at[o];
        val = (float)C.u0[P.lattice[(size_t)ly * (P.L + 1) + lx]];
      }
      uex += wq * val;
    }
  }
  return (isnan(x) || isnan(y)) ? NAN : Z + Y * uex;
}

struct ExitState {
  float x, y, Y, Z;
};

// Two steps of a path, the second unless the first exits: the flagged sides (0:
// goes on) and K after them.  Draw j, which is advanced.
template <int KIND>
__device__ __forceinline__ uint32_t step_pair(const CollectArgs& C, const double* line, const float (&e)[4], uint32_t k,
                                              uint32_t p, uint32_t& j, float& x, float& y, float& Y, float& Z,
                                              uint32_t& K) {
  const AsmParams& P = C.P;
  const U4 r = philox10(j, p, k, C.inst, P.key0, P.key1);
  float z0, z1;
  box_muller(uniform32(r.a), uniform32(r.b), z0, z1);
  em_step<KIND, float>(P.coef, (float)P.h, (float)P.sqrt_h, z0, z1, x, y, Y, Z);
  uint32_t fl = exit_sides<KIND, float>(P.coef, P.exit_rule, (float)P.sqrt_h, line, e, x, y);
  K = 2 * j + 1;
  if (fl == 0) {
    box_muller(uniform32(r.c), uniform32(r.d), z0, z1);
    em_step<KIND, float>(P.coef, (float)P.h, (float)P.sqrt_h, z0, z1, x, y, Y, Z);
    fl = exit_sides<KIND, float>(P.coef, P.exit_rule, (float)P.sqrt_h, line, e, x, y);
    K = 2 * j + 2;
  }
  ++j;
  if (fl == 0 && 2 * j >= (1u << 24) - 2) fl = 15u;   // step cap
  return fl;
}

// Each wave takes a contiguous range of the path ids.
template <int KIND>
__global__ __launch_bounds__(BLK) void k_collect_ends(CollectArgs C, int64_t waves) {
  __shared__ ExitState queue[BLK / 64][QCAP];
  __shared__ uint32_t queue_id[BLK / 64][QCAP], queue_kf[BLK / 64][QCAP];
  const AsmParams& P = C.P;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t wave = (int64_t)blockIdx.x * (BLK / 64) + wid;
  if (wave >= waves) return;
  const int64_t total = C.n * C.paths_per_knot;
  uint32_t next = (uint32_t)(total * wave / waves);
  const uint32_t stop = (uint32_t)(total * (wave + 1) / waves);
  ExitState* Q = queue[wid];
  uint32_t* Qi = queue_id[wid];
  uint32_t* Qk = queue_kf[wid];
  int qn = 0;
  auto resolve = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < qn; i += 64) {
      const ExitState r = Q[i];
      const uint32_t id = Qi[i], kf = Qk[i];
      const KnotDesc& d = P.desc[id / (uint32_t)C.paths_per_knot];
      CollectEnd e;
      e.v = exit_score<KIND>(C, d, r.x, r.y, r.Y, r.Z, kf & 15u);
      e.K = kf >> 4;
      C.end[id] = e;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    qn = 0;
  };
  bool active = false;
  uint32_t id = 0, k = 0, p = 0, j = 0;
  float x = 0, y = 0, Y = 0, Z = 0;
  float e[4] = {0, 0, 0, 0};
  while (true) {
    const uint64_t idle = __ballot(!active);
    const int n_idle = __popcll(idle);
    if (next < stop && (n_idle >= REFILL || idle == ~0ull)) {
      const uint32_t take = min((uint32_t)n_idle, stop - next);
      const uint32_t rank = (uint32_t)__popcll(idle & ((1ull << lane) - 1ull));
      if (!active && rank < take) {
        id = next + rank;
        k = id / (uint32_t)C.paths_per_knot;
        p = id - k * (uint32_t)C.paths_per_knot;
        const CollectStart& s = C.start[k];
        x = s.x; y = s.y; Y = 1.0f; Z = 0.0f;
#pragma unroll
        for (int o = 0; o < 4; ++o) e[o] = s.e[o];
        j = 0;
        active = true;
      }
      next += take;
    } else if (idle == ~0ull) {
      break;
    }
    uint32_t fl = 0, K = 0;
    if (active) fl = step_pair<KIND>(C, P.desc[k].line, e, k, p, j, x, y, Y, Z, K);
    const uint64_t em = __ballot(fl != 0);
    if (em != 0) {
      if (fl != 0) {
        const int i = qn + __popcll(em & ((1ull << lane) - 1ull));
        Q[i] = ExitState{x, y, Y, Z};
        Qi[i] = id;
        Qk[i] = (K << 4) | fl;
        active = false;
      }
      qn += __popcll(em);
      if (qn >= 64) resolve();
    }
  }
  if (qn > 0) resolve();
}

// The pairs of the paths [first, last), at most 64, one lane per path (id k, p,
// start x, y, end v, K): CHUNK points at a time, then the wave writes the chunk's
// slots, CHUNK consecutive lanes per path.
constexpr int CHUNK = 8;
struct PairStage {
  float2 xy[64 * (CHUNK + 1)];
  float t[64 * (CHUNK + 1)];
};
template <int KIND>
__device__ __forceinline__ void write_points(const CollectArgs& C, PairStage& stage, int64_t first, int64_t last, int lane,
                                             uint32_t k, uint32_t p, float x, float y, const CollectEnd& end) {
  const AsmParams& P = C.P;
  const int S = C.points_per_path;
  const int rec = (int)min(end.K, (uint32_t)S);
  float Y = 1.0f, Z = 0.0f;
  const float ux = (float)(1.0 / (P.x1 - P.x0)), uy = (float)(1.0 / (P.y1 - P.y0));
  for (int n0 = 0; n0 < S; n0 += CHUNK) {
    if (__ballot(n0 < rec) != 0) {
      U4 r{};
#pragma unroll
      for (int c = 0; c < CHUNK; ++c) {
        const int n = n0 + c;
        float2 at = make_float2(0.0f, 0.0f);
        float t = NAN;
        if (n < rec) {
          // the network's input: the point in the domain's unit coordinates
          at.x = (x - (float)P.x0) * ux;
          at.y = (y - (float)P.y0) * uy;
          t = (end.v - Z) / Y;
          if ((c & 1) == 0) r = philox10((uint32_t)n >> 1, p, k, C.inst, P.key0, P.key1);
          if (n + 1 < rec) {
            float z0, z1;
            box_muller(uniform32((c & 1) ? r.c : r.a), uniform32((c & 1) ? r.d : r.b), z0, z1);
            em_step<KIND, float>(P.coef, (float)P.h, (float)P.sqrt_h, z0, z1, x, y, Y, Z);
          }
        }
        stage.xy[lane * (CHUNK + 1) + c] = at;
        stage.t[lane * (CHUNK + 1) + c] = t;
      }
    } else {
#pragma unroll
      for (int c = 0; c < CHUNK; ++c) {
        stage.xy[lane * (CHUNK + 1) + c] = make_float2(0.0f, 0.0f);
        stage.t[lane * (CHUNK + 1) + c] = NAN;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < CHUNK; ++q) {
      const int path = q * (64 / CHUNK) + lane / CHUNK, c = lane % CHUNK;
      const int64_t slot = (first + path) * S + n0 + c;
      if (first + path < last && n0 + c < S) {
        const float2 at = stage.xy[path * (CHUNK + 1) + c];
        C.xy[2 * slot] = at.x;
        C.xy[2 * slot + 1] = at.y;
        C.target[slot] = stage.t[path * (CHUNK + 1) + c];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

template <int KIND>
__global__ __launch_bounds__(BLK) void k_collect_points(CollectArgs C) {
  __shared__ PairStage stage[BLK / 64];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t total = C.n * C.paths_per_knot;
  const int64_t first = ((int64_t)blockIdx.x * (BLK / 64) + wid) * 64;
  if (first >= total) return;
  const uint32_t id = (uint32_t)min(first + lane, total - 1);
  const uint32_t k = id / (uint32_t)C.paths_per_knot, p = id - k * (uint32_t)C.paths_per_knot;
  write_points<KIND>(C, stage[wid], first, min(first + 64, total), lane, k, p, C.start[k].x, C.start[k].y, C.end[id]);
}

// The same in one launch, a path per lane from its start to its pairs.
template <int KIND>
__global__ __launch_bounds__(BLK) void k_collect_whole(CollectArgs C) {
  __shared__ PairStage stage[BLK / 64];
  const AsmParams& P = C.P;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t total = C.n * C.paths_per_knot;
  const int64_t first = ((int64_t)blockIdx.x * (BLK / 64) + wid) * 64;
  if (first >= total) return;
  const uint32_t id = (uint32_t)min(first + lane, total - 1);
  const uint32_t k = id / (uint32_t)C.paths_per_knot, p = id - k * (uint32_t)C.paths_per_knot;
  const KnotDesc& d = P.desc[k];
  float e[4];
#pragma unroll
  for (int o = 0; o < 4; ++o) e[o] = exit_threshold<KIND, float>(P.coef, P.exit_rule, P.sqrt_h, d, o);
  float x = (float)d.sx, y = (float)d.sy, Y = 1.0f, Z = 0.0f;
  uint32_t j = 0, fl = 0;
  CollectEnd end{0.0f, 0u};
  while (fl == 0) fl = step_pair<KIND>(C, d.line, e, k, p, j, x, y, Y, Z, end.K);
  end.v = exit_score<KIND>(C, d, x, y, Y, Z, fl);
  write_points<KIND>(C, stage[wid], first, min(first + 64, total), lane, k, p, (float)d.sx, (float)d.sy, end);
}

template <int KIND>
hipError_t launch_kind(const CollectArgs& C, hipStream_t stream) {
  const int64_t total = C.n * C.paths_per_knot;
  if (!C.start) {
    hipLaunchKernelGGL(k_collect_whole<KIND>, dim3((unsigned)((total + BLK - 1) / BLK)), dim3(BLK), 0, stream, C);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_collect_start<KIND>, dim3((unsigned)((C.n + BLK - 1) / BLK)), dim3(BLK), 0, stream, C);
  const int64_t waves = std::min<int64_t>(COLLECT_WAVES, (total + 63) / 64);
  hipLaunchKernelGGL(k_collect_ends<KIND>, dim3((unsigned)((waves + BLK / 64 - 1) / (BLK / 64))), dim3(BLK), 0, stream, C,
                     waves);
  hipLaunchKernelGGL(k_collect_points<KIND>, dim3((unsigned)((total + BLK - 1) / BLK)), dim3(BLK), 0, stream, C);
  return hipGetLastError();
}

}  // namespace

bool collect_refills(double cell_steps, int64_t paths) {
  return cell_steps >= REFILL_STEPS && paths >= REFILL_PATHS;
}

hipError_t launch_collect(const AsmParams& P, int64_t n, int32_t paths_per_knot, int32_t points_per_path,
                          uint32_t inst, const double* u0, float* xy, void* scratch, float* target, hipStream_t stream) {
  CollectArgs C;
  C.inst = inst;
  C.P = P;
  C.n = n;
  C.paths_per_knot = paths_per_knot;
  C.points_per_path = points_per_path;
  C.u0 = u0;
  C.start = static_cast<CollectStart*>(scratch);
  C.end = scratch ? reinterpret_cast<CollectEnd*>(C.start + n) : nullptr;
  C.xy = xy;
  C.target = target;
  switch (P.coef.kind) {
    case PDD_COEF_POISSON: return launch_kind<PDD_COEF_POISSON>(C, stream);
    case PDD_COEF_VARCOEF: return launch_kind<PDD_COEF_VARCOEF>(C, stream);
    case PDD_COEF_AMPLITUDE: return launch_kind<PDD_COEF_AMPLITUDE>(C, stream);
    case PDD_COEF_LUT: return launch_kind<PDD_COEF_LUT>(C, stream);
    case PDD_COEF_CONSTSOL: return launch_kind<PDD_COEF_CONSTSOL>(C, stream);
    case PDD_COEF_EQ43: return launch_kind<PDD_COEF_EQ43>(C, stream);
    default: return launch_kind<PDD_COEF_EXITTIME>(C, stream);
  }
}

}  // namespace pdd
