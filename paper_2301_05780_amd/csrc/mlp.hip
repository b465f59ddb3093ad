// The control-variate network v(x) = w3 . tanh(W2 tanh(W1 x + b1) + b2) + b3
// (2 -> 64 -> 64 -> 1) on the GPU: pointwise evaluation with input gradient,
// the Adam trainer (float32 MFMA), the grad-v table bake, and the kernel
// that collects (path point, tail score) training pairs from the method's own
// paths.
//
// Any adapted F keeps the mean of the Feynman-Kac score (eq. 38); F = sigma^T
// grad u would remove the variance (eq. 11).  The network is fitted to
// pathwise estimates of u: for a point X_n of a path that exits at step K,
// E[(Z_K + Y_K u(X_K) - Z_n) / Y_n | X_n] = u(X_n), with u at the exit taken
// from the solved knot values (hat interpolation) or the boundary datum.
//
// Parameter layout (4417 float32): W1[64][2], b1[64], W2[64][64] (out, in),
// b2[64], w3[64], b3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <memory>

#include "context.h"
#include "device_common.h"
#include "grid_exchange.h"
#include "mlp.h"
#include "net_grad.h"

namespace pdd {

namespace {

constexpr int BLK = 256;

// tanh for the trainer: 1 - 2 / (exp(2z) + 1) (one exp, one reciprocal,
// exact limits +-1, absolute error about 1e-7), and for |z| < 1/16 the odd
// Taylor polynomial z - z^3/3 + 2 z^5/15 (relative error below 1e-8), where
// the first form would lose relative accuracy
__device__ __forceinline__ float tanh_f(float z) {
  const float e = __builtin_amdgcn_exp2f(z * 2.8853900817779268f);
  const float t = 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
  const float z2 = z * z;
  const float p = z * __builtin_fmaf(z2, __builtin_fmaf(z2, 0.13333333f, -0.33333333f), 1.0f);
  return __builtin_fabsf(z) < 0.0625f ? p : t;
}

// v and grad v at one point, float32 throughout, parameters from `th`
__device__ __forceinline__ void net_eval_f32(const float* __restrict__ th, float x, float y, float& v, float& gx,
                                             float& gy) {
  float h1[MLP_W];
#pragma unroll
  for (int k = 0; k < MLP_W; ++k)
    h1[k] = tanhf(th[OW1 + 2 * k] * x + th[OW1 + 2 * k + 1] * y + th[OB1 + k]);
  float g1[MLP_W];
#pragma unroll
  for (int k = 0; k < MLP_W; ++k) g1[k] = 0.0f;
  float vv = th[OB3];
  for (int j = 0; j < MLP_W; ++j) {
    float z = th[OB2 + j];
#pragma unroll
    for (int k = 0; k < MLP_W; ++k) z += th[OW2 + j * MLP_W + k] * h1[k];
    const float h2 = tanhf(z);
    vv += th[OW3 + j] * h2;
    const float g2 = (1.0f - h2 * h2) * th[OW3 + j];
#pragma unroll
    for (int k = 0; k < MLP_W; ++k) g1[k] += th[OW2 + j * MLP_W + k] * g2;
  }
  float ax = 0.0f, ay = 0.0f;
#pragma unroll
  for (int k = 0; k < MLP_W; ++k) {
    const float d = (1.0f - h1[k] * h1[k]) * g1[k];
    ax += th[OW1 + 2 * k] * d;
    ay += th[OW1 + 2 * k + 1] * d;
  }
  v = vv;
  gx = ax;
  gy = ay;
}

__global__ __launch_bounds__(BLK) void k_mlp_eval(const float* __restrict__ params, int64_t n, const float* __restrict__ xy,
                                                  float* __restrict__ v, float* __restrict__ g) {
  __shared__ float th[MLP_PARAMS];
  for (int i = threadIdx.x; i < MLP_PARAMS; i += BLK) th[i] = params[i];
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) {
    float vv, gx, gy;
    net_eval_f32(th, xy[2 * i], xy[2 * i + 1], vv, gx, gy);
    if (v) v[i] = vv;
    if (g) { g[2 * i] = gx; g[2 * i + 1] = gy; }
  }
}

// grad v through net_grad_mfma, the routine the float32 network control
// variate runs at every Euler step of the assembly: each wave takes 64
// consecutive points per pass.  Lanes past the end repeat the last point, so
// every lane of the wave takes part in the MFMA products, and store nothing.
__global__ __launch_bounds__(BLK) void k_mlp_grad_bf16(const float* __restrict__ params, int64_t n,
                                                       const float* __restrict__ xy, float* __restrict__ g) {
  __shared__ NetLds N;
  net_stage(&N, params);
  __syncthreads();
  const int lane = (int)(threadIdx.x & 63);
  const int64_t waves = (int64_t)gridDim.x * (BLK / 64);
  const int64_t wave = (int64_t)blockIdx.x * (BLK / 64) + (threadIdx.x >> 6);
  for (int64_t base = wave * 64; base < n; base += waves * 64) {      // wave-uniform bound
    const int64_t i = base + lane;
    const int64_t r = i < n ? i : n - 1;
    float gx, gy;
    net_grad_mfma(&N, xy[2 * r], xy[2 * r + 1], gx, gy);
    if (i < n) {
      g[2 * i] = gx;
      g[2 * i + 1] = gy;
    }
  }
}

// grad v on the node-centred grid of the domain: grad_lut[(j n + i) 2 + d]
__global__ __launch_bounds__(BLK) void k_mlp_bake(const float* __restrict__ params, int lut_n, double x0, double x1,
                                                  double y0, double y1, float* __restrict__ out) {
  __shared__ float th[MLP_PARAMS];
  for (int i = threadIdx.x; i < MLP_PARAMS; i += BLK) th[i] = params[i];
  __syncthreads();
  const int64_t total = (int64_t)lut_n * lut_n;
  for (int64_t q = (int64_t)blockIdx.x * BLK + threadIdx.x; q < total; q += (int64_t)gridDim.x * BLK) {
    const int i = (int)(q % lut_n), j = (int)(q / lut_n);
    // the network's input: the node in the domain's unit coordinates; the
    // gradient scaled back to the domain's
    const float x = (float)((double)i / (double)(lut_n - 1));
    const float y = (float)((double)j / (double)(lut_n - 1));
    float vv, gx, gy;
    net_eval_f32(th, x, y, vv, gx, gy);
    out[2 * q] = gx * (float)(1.0 / (x1 - x0));
    out[2 * q + 1] = gy * (float)(1.0 / (y1 - y0));
  }
}

// ---- trainer (float32 MFMA) -------------------------------------------------
// A step's minibatch is cut into units of points: a batch of up to WIDE_BATCH is
// one slice, a larger one slices of WIDE_SLICE points; unit v (0..3) of a slice
// takes its points 128 rd + 32 v + c, c < 32, rd = 0, 1, ...  A unit's gradient is
// one accumulation over its rounds, and the gradient of the step is the sum of
// the units of a slice in order, then of the slices in order: fixed, whatever
// workgroups compute them.
//
// The steps are sequential and a unit is little work (two rounds of a batch of
// 256: 192 MFMA per round), so a step on one workgroup was the four units' work
// on one CU, 31 us for a batch of 256 and 111 us for 1024.  Here one cooperative
// launch gives every unit a workgroup on a CU of its own for all the steps
// (grid_exchange.h).  Of a single slice every workgroup sums the published units and
// updates (Adam) all the parameters for itself, one exchange a step over two buffers
// in turn; of several slices each sums and updates its share and publishes it, two
// exchanges a step.  What bounds a step is that chain: per pair of rounds three
// products of 32 and more dependent MFMA and seven barriers, then the exchange and
// the update.  Per step (us; one workgroup for the batch, and above 1024 one launch
// for the slices' gradients and one for Adam, against this form):
//   batch      32    100    256   1024   4096   20,000   65,537
//   before   18.3   18.6   31.5    109    109      366     1163
//   now      10.7   13.0   14.1     37     21       48      112
// With shares of the parameters and two exchanges a single slice took 17.1 for 256.
//
// Eight waves per workgroup, two rounds (tiles of 32 points) at a time, points as
// the columns c = lane % 32 and the two half-waves h = lane / 32 splitting the
// contraction index:
//   h1 = tanh(W1 x + b1)                          all waves, 8 values per lane
//   z2^T = W2 h1^T                                waves 0-3 (tile, jb): v_mfma_f32_32x32x2_f32, K = 64
//   h2 = tanh(z2 + b2), v = w3 . h2 + b3, dv = (v - t) / B
//   dz2^T = dv (1 - h2^2) w3
//   gW2 += dz2^T h1                               waves 0-3 (jb, kb): MFMA, K = the 32 points of each tile
//   dh1^T = W2^T dz2^T, dz1 = dh1 (1 - h1^2)      waves 4-7 (tile, kb): MFMA, K = 64
//   gW1, gb1, gb2, gw3, gb3, loss                 sums over the points, one lane per unit or point
// The contraction order of z2 and dh1 follows the accumulator's row order
// (row = 8 (r / 4) + 4 h + r % 4 of register r).  Parameters and moments stay in LDS
// for the whole call.
struct TrainArgs {
  float* params;
  float* m;
  float* s;
  const float* xy;
  const float* target;
  const int32_t* order;
  int64_t n_order;
  int64_t n_points;       // order entries outside [0, n_points) are skipped
  int32_t batch;
  int32_t steps;
  int32_t step0;          // Adam step counter before this call
  float lr;
  int32_t update;         // 0: write the gradient of the first batch to grad_out only
  float* grad_out;
  float* losses;          // per step, nullable
  int32_t slice;          // points per slice
  int32_t units;          // units of the batch (four per slice; of a single slice, those with points)
  float* part;            // several workgroups: the published gradients, GPAD each,
  float* theta;           // several slices: the parameters, and at the end the moments, PARAM_PAD each,
  uint32_t* flags;        // and the epoch flags, none above
  uint32_t epoch;         // this
  uint32_t polls;         // of a wait between workgroups (grid_exchange.h)
};

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int WIDE_BATCH = 1024;      // larger batches are cut into slices
constexpr int WIDE_SLICE = 256;
constexpr int TT = 512;               // threads per workgroup
constexpr int TRAIN_G = 256;          // workgroups, at most
constexpr int H1S = 68;               // row stride of the h1 copy [point][unit] (16-byte aligned rows)
constexpr int DZS = 36;               // row stride of the [unit][point] copies
constexpr int PARAM_PAD = ((MLP_PARAMS + 3) / 4) * 4;
constexpr int GPAD = PARAM_PAD + 4;   // one unit's gradient (+ loss)

struct TrainTile {
  float h1[32 * H1S];                 // h1[c][k]
  float dz[64 * DZS];                 // dz2^T[j][c]
  float dh[64 * DZS];                 // dv_c h2[j][c]
  float dz1[64 * DZS];                // dz1^T[k][c]
  float x[32], y[32], t[32], ok[32];  // the points, and 1 (0: skipped)
  float vp[64];                       // w3 . h2 over the first 32 units, per lane
  float dv[32], res[32];
};
constexpr int MOMENTS = GPAD;         // items (owned parameter, lane) of a workgroup, at most
struct TrainLds {
  float th[PARAM_PAD];
  TrainTile tile[2];
  float sum[GPAD];                    // one workgroup or whole slices: the slice's sum so far
  float all[GPAD];                    // one workgroup: the batch's; several: the first moments,
  int32_t stop;
  float second[MOMENTS];              // and the second ones
};

// accumulator register r of a 32 x 32 tile holds row 8 (r / 4) + 4 h + r % 4
__device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// A point of the batch as loaded ahead of its round by the threads below 64.
struct TrainPoint {
  float x, y, t, ok;
};
__device__ __forceinline__ TrainPoint load_point(const TrainArgs& A, int step, int p, int pend) {
  TrainPoint q{0.0f, 0.0f, 0.0f, 0.0f};
  if (p < pend) {
    const int64_t oi = ((int64_t)step * A.batch + p) % A.n_order;
    const int32_t idx = A.order[oi];
    if (idx >= 0 && (int64_t)idx < A.n_points) {
      q.x = A.xy[2 * (int64_t)idx];
      q.y = A.xy[2 * (int64_t)idx + 1];
      q.t = A.target[idx];
      q.ok = 1.0f;
    }
  }
  return q;
}

// ONE: a single slice.  UNITS: several.  WHOLE: several, and a workgroup takes the
// four units of a slice in turn and publishes their sum.
enum TrainForm { ONE, UNITS, WHOLE };
// All the steps as workgroup `me` of G.  Only workgroup 0 writes to the caller's
// arrays: the losses as they come, and the parameters, moments or gradient at the
// very end.  False: a wait ran out, before that.
template <TrainForm form>
__device__ __forceinline__ bool train_steps(const TrainArgs& A, TrainLds& L, const int G, const int me) {
  float* th = L.th;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wt = w >> 1, wb = w & 1;    // waves 0-3: tile (or jb) and half of the units; 4-7: 2 + tile, half
  constexpr bool one = form == ONE, whole = form == WHOLE;
  const int nsl = one ? 1 : (A.batch + A.slice - 1) / A.slice;
  for (int i = tid; i < MLP_PARAMS; i += TT) th[i] = A.params[i];
  if (tid == 0) L.stop = 0;
  // this workgroup's parameters [q0, q0 + S), the loss counted as the last one: of a
  // single slice every workgroup sums and updates all of them, of several its share,
  // each summed over the slices by LP lanes.  Their moments in LDS (several slices on
  // one workgroup: in global memory)
  const int S = one ? MLP_PARAMS + 1 : (MLP_PARAMS + 1 + G - 1) / G;
  const int q0 = one ? 0 : me * S;
  const bool resident = one || G > 1;
  int LP = 1;
  if (!one && G > 1)
    while (LP < nsl && LP < 64 && 2 * LP * S <= MOMENTS) LP <<= 1;
  float* mom_m = L.all;
  float* mom_s = L.second;
  if (resident && A.update) {
    for (int item = tid; item < S * LP; item += TT) {
      const int q = q0 + item / LP;
      mom_m[item] = q < MLP_PARAMS ? A.m[q] : 0.0f;
      mom_s[item] = q < MLP_PARAMS ? A.s[q] : 0.0f;
    }
  }
  const float inv_b = 1.0f / (float)A.batch;
  uint32_t epoch = A.epoch;
  // this workgroup's units: `u0`, and the one after u
  const int u0 = whole ? 4 * me : me;
  auto after = [&](int u) __attribute__((always_inline)) -> int {
    return !whole ? u + G : (u & 3) != 3 ? u + 1 : u + 4 * G - 3;
  };
  const int t2 = tid >> 5 & 1;          // tile of the point that thread tid < 64 loads
  auto point_of = [&](int unit, int rd, int& pend) __attribute__((always_inline)) -> int {
    const int pbase = (unit >> 2) * A.slice;
    pend = min(A.batch, pbase + A.slice);
    return pbase + (rd + t2) * 128 + 32 * (unit & 3) + (tid & 31);
  };
  TrainPoint next{};
  if (tid < 64) {
    int pend;
    const int p = point_of(u0, 0, pend);
    next = load_point(A, 0, p, pend);
  }
  __syncthreads();

  bool late = false;
  for (int step = 0; step < A.steps; ++step) {
    for (int unit = u0; unit < A.units; unit = after(unit)) {
      f32x16 gw2 = f32x16{};
      float g_b2 = 0.0f, g_w3 = 0.0f, g_w1 = 0.0f, g_b3 = 0.0f, loss = 0.0f;
      int pend;
      const int rounds = (min(A.batch - (unit >> 2) * A.slice, A.slice) + 127) / 128;
      for (int rd = 0; rd < rounds; rd += 2) {
        const int tiles = min(2, rounds - rd);
        if (tid < 64) {
          TrainTile& T = L.tile[t2];
          T.x[tid & 31] = next.x; T.y[tid & 31] = next.y; T.t[tid & 31] = next.t; T.ok[tid & 31] = next.ok;
          // the next rounds' points, of this unit, the next one or the next step
          int u = unit, r2 = rd + 2, st = step;
          if (r2 >= rounds) {
            r2 = 0;
            u = after(unit);
            if (u >= A.units) {
              u = u0;
              ++st;
            }
          }
          const int p = point_of(u, r2, pend);
          next = st < A.steps ? load_point(A, st, p, pend) : TrainPoint{};
        }
        __syncthreads();
        // layer 1: wave (tile, units 16 q .. 16 q + 15), 8 units per lane
        {
          TrainTile& T = L.tile[w >> 2];
          const float x = T.x[c], y = T.y[c];
          const int k0 = 16 * (w & 3) + 8 * h;
          if ((w >> 2) < tiles) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int k = k0 + i;
              T.h1[c * H1S + k] = tanh_f(th[OW1 + 2 * k] * x + th[OW1 + 2 * k + 1] * y + th[OB1 + k]);
            }
          }
        }
        __syncthreads();
        // layer 2: wave (tile, jb): z2^T[j][c], contraction k(s, h) = 32 (s / 16) + acc_row(s % 16, h)
        const bool fwd = w < 4 && wt < tiles;
        f32x16 z = f32x16{};
        float dz2r[16];
        if (fwd) {
          TrainTile& T = L.tile[wt];
          const float* wrow = th + OW2 + (32 * wb + c) * MLP_W;
          const float* hrow = T.h1 + c * H1S;
#pragma unroll
          for (int q = 0; q < 8; ++q) {          // four steps s = 4q .. 4q+3 read four consecutive k
            const int k0 = 32 * (q >> 2) + 8 * (q & 3) + 4 * h;
            const float4 a4 = *reinterpret_cast<const float4*>(wrow + k0);
            const float4 b4 = *reinterpret_cast<const float4*>(hrow + k0);
            const float av[4] = {a4.x, a4.y, a4.z, a4.w};
            const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], bv[e], z, 0, 0, 0);
          }
          // rows j = 32 wb + acc_row(r, h) of column c
          float vpart = 0.0f;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = 32 * wb + acc_row(r, h);
            const float h2 = tanh_f(z[r] + th[OB2 + j]);
            if (wb == 0) vpart += th[OW3 + j] * h2;
            z[r] = h2;
            dz2r[r] = (1.0f - h2 * h2) * th[OW3 + j];
          }
          if (wb == 0) T.vp[lane] = vpart;
        }
        __syncthreads();
        // the sum w3 . h2 goes on over the second half of the units, then the residual
        if (fwd && wb == 1) {
          TrainTile& T = L.tile[wt];
          float vpart = T.vp[lane];
#pragma unroll
          for (int r = 0; r < 16; ++r) vpart += th[OW3 + 32 + acc_row(r, h)] * z[r];
          const float v = vpart + __shfl_xor(vpart, 32, 64) + th[OB3];
          const float res = T.ok[c] != 0.0f ? v - T.t[c] : 0.0f;
          if (h == 0) {
            T.res[c] = res;
            T.dv[c] = res * inv_b;
          }
        }
        __syncthreads();
        if (fwd) {
          TrainTile& T = L.tile[wt];
          const float dv = T.dv[c];
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = 32 * wb + acc_row(r, h);
            T.dz[j * DZS + c] = dz2r[r] * dv;
            T.dh[j * DZS + c] = dv * z[r];
          }
        }
        if (w == 7 && h == 0) {
          for (int t = 0; t < tiles; ++t) {
            const float res = L.tile[t].res[c];
            loss += 0.5f * res * res * inv_b;
            g_b3 = __builtin_fmaf(res, inv_b, g_b3);
          }
        }
        __syncthreads();
        if (w < 4) {
          // gW2[j][k] += sum_c dz2^T[j][c] h1[c][k], wave (jb, kb); contraction c(s, h) = 16 h + s
          for (int t = 0; t < tiles; ++t) {
            TrainTile& T = L.tile[t];
            const float* arow = T.dz + (32 * wt + c) * DZS + 16 * h;
            float av[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 a4 = *reinterpret_cast<const float4*>(arow + 4 * q);
              av[4 * q] = a4.x; av[4 * q + 1] = a4.y; av[4 * q + 2] = a4.z; av[4 * q + 3] = a4.w;
            }
#pragma unroll
            for (int s2 = 0; s2 < 16; ++s2)
              gw2 = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s2], T.h1[(16 * h + s2) * H1S + 32 * wb + c], gw2, 0, 0, 0);
            // gb2[j], gw3[j] for j = lane: sums over the 32 points
            if (w < 2) {
              const float4* src = reinterpret_cast<const float4*>((w == 0 ? T.dz : T.dh) + lane * DZS);
              float& g = w == 0 ? g_b2 : g_w3;
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                const float4 a4 = src[q];
                g += (a4.x + a4.y) + (a4.z + a4.w);
              }
            }
          }
        } else if (wt - 2 < tiles) {
          // dh1^T[k][c] = sum_j W2[j][k] dz2^T[j][c], wave (tile, kb); contraction j(s, h) as k(s, h) above
          TrainTile& T = L.tile[wt - 2];
          f32x16 d = f32x16{};
#pragma unroll
          for (int s2 = 0; s2 < 32; ++s2) {
            const int j = 32 * (s2 >> 4) + acc_row(s2 & 15, h);
            d = __builtin_amdgcn_mfma_f32_32x32x2f32(th[OW2 + j * MLP_W + 32 * wb + c], T.dz[j * DZS + c], d, 0, 0, 0);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int k = 32 * wb + acc_row(r, h);
            const float h1 = T.h1[c * H1S + k];
            T.dz1[k * DZS + c] = d[r] * (1.0f - h1 * h1);
          }
        }
        __syncthreads();
        // gW1[k][.] (waves 4, 5), gb1[k] (wave 6) for k = lane: sums over the 32 points
        if (w == 4 || w == 5) {
          for (int t = 0; t < tiles; ++t) {
            TrainTile& T = L.tile[t];
            const float4* dzr = reinterpret_cast<const float4*>(T.dz1 + lane * DZS);
            const float* xs = w == 4 ? T.x : T.y;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const float4 a4 = dzr[q];
              const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
              for (int e = 0; e < 4; ++e) g_w1 = __builtin_fmaf(av[e], xs[4 * q + e], g_w1);
            }
          }
        } else if (w == 6) {
          for (int t = 0; t < tiles; ++t) {
            const float4* dzr = reinterpret_cast<const float4*>(L.tile[t].dz1 + lane * DZS);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const float4 a4 = dzr[q];
              g_w1 = ((g_w1 + a4.x) + a4.y) + a4.z;
              g_w1 += a4.w;
            }
          }
        }
        __syncthreads();
      }
      // loss and gb3 of the unit (wave 7, lanes with h == 0 hold one point column each)
      if (w == 7) {
        for (int off = 32; off > 0; off >>= 1) {
          loss += __shfl_xor(loss, off, 64);
          g_b3 += __shfl_xor(g_b3, off, 64);
        }
      }
      // the unit's gradient: published, or added in unit and slice order
      const bool alone = G > 1 && !whole;
      float* out = G > 1 ? A.part + (size_t)(one ? unit + 4 * (step & 1) : whole ? unit >> 2 : unit) * GPAD : nullptr;
      const bool first = (unit & 3) == 0;
      auto put = [&](int q, float g) __attribute__((always_inline)) {
        if (alone) agent_store(out + q, g);
        else L.sum[q] = first ? g : L.sum[q] + g;
      };
      if (w < 4) {
#pragma unroll
        for (int r = 0; r < 16; ++r) put(OW2 + (32 * wt + acc_row(r, h)) * MLP_W + 32 * wb + c, gw2[r]);
      }
      if (w == 0) put(OB2 + lane, g_b2);
      if (w == 1) put(OW3 + lane, g_w3);
      if (w == 4) put(OW1 + 2 * lane, g_w1);
      if (w == 5) put(OW1 + 2 * lane + 1, g_w1);
      if (w == 6) put(OB1 + lane, g_w1);
      if (w == 7 && lane == 0) {
        put(OB3, g_b3);
        put(MLP_PARAMS, loss);
      }
      if (!one && !alone && (unit & 3) == 3) {
        __syncthreads();
        for (int q = tid; q <= MLP_PARAMS; q += TT) {
          if (G > 1) agent_store(out + q, L.sum[q]);
          else L.all[q] = ((unit >> 2) == 0 ? 0.0f : L.all[q]) + L.sum[q];
        }
        __syncthreads();
      }
    }
    const int tstep = A.step0 + step + 1;
    const float c1 = 1.0f - powf(0.9f, (float)tstep);
    const float c2 = 1.0f - powf(0.999f, (float)tstep);
    if ((late = !grid_exchange(A.flags, G, me, ++epoch, &L.stop, A.polls))) break;
    // sums of the units and slices in order, then Adam (bias-corrected), beta1 =
    // 0.9, beta2 = 0.999, eps = 1e-8.  The roundings of the step are written out:
    // which product the fused one takes is not left to the compiler.
    auto adam = [&](int q, float g, float* pm, float* ps) __attribute__((always_inline)) -> float {
      const float mg = 0.1f * g, sg = 0.001f * g;
      const float mq = one ? __builtin_fmaf(0.9f, *pm, mg) : __builtin_fmaf(0.1f, g, 0.9f * *pm);
      const float sq = one ? __builtin_fmaf(0.999f, *ps, sg * g) : __builtin_fmaf(g, sg, 0.999f * *ps);
      *pm = mq;
      *ps = sq;
      return th[q] - A.lr * (mq / c1) / (sqrtf(sq / c2) + 1e-8f);
    };
    if constexpr (one) {
      if (G > 1) {                        // (every thread reads back what it wrote itself)
        constexpr int ALL = (MLP_PARAMS + 1 + TT - 1) / TT;
        float p[ALL][4];
        const float* in = A.part + (size_t)(4 * (step & 1)) * GPAD;
#pragma unroll
        for (int i = 0; i < ALL; ++i)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            p[i][u] = u < A.units && tid + i * TT <= MLP_PARAMS ? agent_load(in + u * GPAD + tid + i * TT) : 0.0f;
#pragma unroll
        for (int i = 0; i < ALL; ++i)
          if (tid + i * TT <= MLP_PARAMS) L.sum[tid + i * TT] = ((p[i][0] + p[i][1]) + p[i][2]) + p[i][3];
      }
#pragma unroll 1
      for (int q = tid; q <= MLP_PARAMS; q += TT) {
        const float g = L.sum[q];
        if (q == MLP_PARAMS) {
          if (me == 0 && A.losses) A.losses[step] = g;
        } else if (!A.update) {
          if (me == 0) A.grad_out[q] = g;
        } else {
          th[q] = adam(q, g, mom_m + q, mom_s + q);
        }
      }
      if (!A.update) return true;                     // (the same for every workgroup)
      continue;       // the other buffer of gradients is free: all have read it before they published this step's
    }
    for (int i0 = 0; i0 < S * LP; i0 += TT) {           // (uniform)
      const int item = i0 + tid, q = q0 + item / LP, b = item & (LP - 1);
      const bool own = item < S * LP && q <= MLP_PARAMS;
      float g = 0.0f;
      if (G == 1) {
        if (own) g = L.all[q];
      } else {
        for (int base = 0; base < nsl; base += LP) {
          float p[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          if (own && base + b < nsl && whole) {
            p[0] = agent_load(A.part + (size_t)(base + b) * GPAD + q);
          } else if (own && base + b < nsl) {
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = agent_load(A.part + (size_t)(4 * (base + b) + u) * GPAD + q);
          }
          const float mine = ((p[0] + p[1]) + p[2]) + p[3];
          const int many = min(LP, nsl - base);
          for (int j = 0; j < many; ++j) g += __shfl(mine, (lane & ~(LP - 1)) + j, 64);
        }
      }
      if (own && q == MLP_PARAMS) {
        if (b == 0 && G > 1) agent_store(A.theta + q, g);
        else if (b == 0 && A.losses) A.losses[step] = g;
      } else if (own) {
        const float tq = adam(q, g, resident ? mom_m + item : A.m + q, resident ? mom_s + item : A.s + q);
        if (b == 0) {
          if (G > 1) {
            agent_store(A.theta + q, tq);
            if (step + 1 == A.steps) {     // the moments for workgroup 0
              agent_store(A.theta + PARAM_PAD + q, mom_m[item]);
              agent_store(A.theta + 2 * PARAM_PAD + q, mom_s[item]);
            }
          } else {
            th[q] = tq;
          }
        }
      }
    }
    if ((late = !grid_exchange(A.flags, G, me, ++epoch, &L.stop, A.polls))) break;
    if (G > 1) {
      constexpr int ALL = (MLP_PARAMS + TT - 1) / TT;
      float v[ALL];
#pragma unroll
      for (int i = 0; i < ALL; ++i) v[i] = tid + i * TT < MLP_PARAMS ? agent_load(A.theta + tid + i * TT) : 0.0f;
#pragma unroll
      for (int i = 0; i < ALL; ++i)
        if (tid + i * TT < MLP_PARAMS) th[tid + i * TT] = v[i];
      if (me == 0 && tid == 0 && A.losses) A.losses[step] = agent_load(A.theta + MLP_PARAMS);
    }
  }
  __syncthreads();
  if (late) return false;
  if constexpr (one) {
    if (me == 0) {
      for (int q = tid; q < MLP_PARAMS; q += TT) {
        A.m[q] = mom_m[q];
        A.s[q] = mom_s[q];
        A.params[q] = th[q];
      }
    }
    return true;
  }
  if (me == 0) {
    for (int q = tid; q < MLP_PARAMS; q += TT) {
      if (G > 1) {
        A.m[q] = agent_load(A.theta + PARAM_PAD + q);
        A.s[q] = agent_load(A.theta + 2 * PARAM_PAD + q);
      }
      A.params[q] = th[q];
    }
  }
  return true;
}

// Where a wait ran out (see grid_exchange.h) workgroup 0 does the call by itself,
// from the start and with the same bits; the others end.
template <TrainForm form>
__global__ __launch_bounds__(TT) void k_mlp_train(TrainArgs A) {
  extern __shared__ float tlds[];
  TrainLds& L = *reinterpret_cast<TrainLds*>(tlds);
  if (train_steps<form>(A, L, gridDim.x, blockIdx.x) || blockIdx.x != 0) return;
  __syncthreads();
  train_steps<form>(A, L, 1, 0);
}

// ---- one workgroup of four waves ----------------------------------------------
// For calls that a cooperative launch does not suit: a captured one (nothing
// says that a graph may hold such a launch), and a single step of 33 to 128 points,
// which is over before the launch of several workgroups has paid.  A wave per unit
// of the batch, a round of 32 points at a time; the same sums in the same order, the
// same bits.  us per call or step, the units one after the other on one workgroup
// of eight waves against this: one step of 96 points 43.6 (three workgroups), 38.2;
// the gradient of 100 points 58.3, 47.7; captured steps of 64 points 20.2, 18.6; 128 37.0,
// 18.7; 256 42.2, 31.5; 1024 143, 108.  Up to 32 points (one unit) the eight waves are
// faster: 11.9, 18.6.
// A captured batch above WIDE_BATCH takes two launches a step, a workgroup per slice for
// the gradients and one for Adam (4096 points 107 us, 631 on one workgroup; 20,000 363,
// 3070).
struct TrainWaveLds {
  float h1[32 * H1S];                 // h1[c][k]
  float dz[64 * DZS];                 // dz2^T[j][c], later dz1^T[k][c]
  float dh[64 * DZS];                 // dv_c h2[j][c]
  float xy[32][2];
};

constexpr int TW = 4;                 // waves per workgroup
constexpr size_t waves_lds_bytes() { return PARAM_PAD * sizeof(float) + TW * sizeof(TrainWaveLds); }
constexpr int OWN = (MLP_PARAMS + TW * 64 - 1) / (TW * 64);   // parameters per thread in Adam
constexpr int GSTRIDE = GPAD;                                  // one wave's gradient slice (+ loss)
static_assert(TW * GSTRIDE * sizeof(float) <= TW * sizeof(TrainWaveLds), "gradient slices fit the wave buffers");

// `slice` 0: the whole batch.  Else (A.update == 0, A.steps == 1) workgroup g takes the
// points [g slice, (g + 1) slice) of the batch of order step `order_step` and writes its
// gradient sum (and loss) to A.grad_out + g GPAD.
__global__ __launch_bounds__(TW * 64) void k_mlp_train_waves(TrainArgs A, int32_t slice, int32_t order_step) {
  extern __shared__ float tlds[];
  float* th = tlds;
  TrainWaveLds* WL = reinterpret_cast<TrainWaveLds*>(tlds + PARAM_PAD);
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, h = lane >> 5, c = lane & 31;
  TrainWaveLds& L = WL[w];
  for (int i = tid; i < MLP_PARAMS; i += TW * 64) th[i] = A.params[i];
  float mown[OWN], sown[OWN];           // Adam moments of parameters tid + i TW 64
#pragma unroll
  for (int i = 0; i < OWN; ++i) {
    const int q = tid + i * TW * 64;
    mown[i] = (q < MLP_PARAMS && A.update) ? A.m[q] : 0.0f;
    sown[i] = (q < MLP_PARAMS && A.update) ? A.s[q] : 0.0f;
  }
  __syncthreads();
  const float inv_b = 1.0f / (float)A.batch;
  // this workgroup's points of each batch: all of them, or one slice
  const int pbase = slice > 0 ? (int)blockIdx.x * slice : 0;
  const int pend = slice > 0 ? min(A.batch, pbase + slice) : A.batch;
  const int rounds = (pend - pbase + 32 * TW - 1) / (32 * TW);

  for (int step = 0; step < A.steps; ++step) {
    f32x16 gw2[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) gw2[a][b] = f32x16{};
    float g_b2 = 0.0f, g_w3 = 0.0f, g_w1x = 0.0f, g_w1y = 0.0f, g_b1 = 0.0f, g_b3 = 0.0f, loss = 0.0f;

    for (int rd = 0; rd < rounds; ++rd) {
      const int p = pbase + rd * 32 * TW + 32 * w + c;
      const bool inb = p < pend;
      const int64_t oi = ((int64_t)(step + order_step) * A.batch + p) % A.n_order;
      const int32_t oidx = inb ? A.order[oi] : -1;
      const bool valid = oidx >= 0 && (int64_t)oidx < A.n_points;
      const int32_t idx = valid ? oidx : 0;
      const float x = valid ? A.xy[2 * (int64_t)idx] : 0.0f;
      const float y = valid ? A.xy[2 * (int64_t)idx + 1] : 0.0f;
      const float t = valid ? A.target[idx] : 0.0f;
      if (h == 0) { L.xy[c][0] = x; L.xy[c][1] = y; }
      // layer 1: units k = 32 kb + acc_row(r, h) of point c
      float h1r[2][16];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int k = 32 * kb + acc_row(r, h);
          const float v = tanh_f(th[OW1 + 2 * k] * x + th[OW1 + 2 * k + 1] * y + th[OB1 + k]);
          h1r[kb][r] = v;
          L.h1[c * H1S + k] = v;
        }
      // layer 2: z2^T[j][c], contraction k(s, h) = 32 (s / 16) + acc_row(s % 16, h)
      f32x16 z[2];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
        z[jb] = f32x16{};
        const float* wrow = th + OW2 + (32 * jb + c) * MLP_W;
#pragma unroll
        for (int q = 0; q < 8; ++q) {          // four steps s = 4q .. 4q+3 read four consecutive k
          const float4 a4 = *reinterpret_cast<const float4*>(wrow + 32 * (q >> 2) + 8 * (q & 3) + 4 * h);
          const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int s2 = 4 * q + e;
            z[jb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], h1r[s2 >> 4][s2 & 15], z[jb], 0, 0, 0);
          }
        }
      }
      // output, residual and dz2 (registers: rows j = 32 jb + acc_row(r, h) of column c)
      float vpart = 0.0f;
      float dz2r[2][16];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = 32 * jb + acc_row(r, h);
          const float h2 = tanh_f(z[jb][r] + th[OB2 + j]);
          vpart += th[OW3 + j] * h2;
          z[jb][r] = h2;
          dz2r[jb][r] = (1.0f - h2 * h2) * th[OW3 + j];
        }
      const float v = vpart + __shfl_xor(vpart, 32, 64) + th[OB3];
      const float res = valid ? v - t : 0.0f;
      const float dv = res * inv_b;
      if (h == 0) { loss += 0.5f * res * res * inv_b; g_b3 += dv; }
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = 32 * jb + acc_row(r, h);
          dz2r[jb][r] *= dv;
          L.dz[j * DZS + c] = dz2r[jb][r];
          L.dh[j * DZS + c] = dv * z[jb][r];
        }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // gb2[j], gw3[j] for j = lane: sums over the 32 points
      {
        const float4* dzr = reinterpret_cast<const float4*>(L.dz + lane * DZS);
        const float4* dhr = reinterpret_cast<const float4*>(L.dh + lane * DZS);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float4 a4 = dzr[q], b4 = dhr[q];
          g_b2 += (a4.x + a4.y) + (a4.z + a4.w);
          g_w3 += (b4.x + b4.y) + (b4.z + b4.w);
        }
      }
      // gW2[j][k] += sum_c dz2^T[j][c] h1[c][k]; contraction c(s, h) = 16 h + s
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
        const float* arow = L.dz + (32 * jb + c) * DZS + 16 * h;
        float av[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 a4 = *reinterpret_cast<const float4*>(arow + 4 * q);
          av[4 * q] = a4.x; av[4 * q + 1] = a4.y; av[4 * q + 2] = a4.z; av[4 * q + 3] = a4.w;
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int s2 = 0; s2 < 16; ++s2)
            gw2[jb][kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s2], L.h1[(16 * h + s2) * H1S + 32 * kb + c],
                                                               gw2[jb][kb], 0, 0, 0);
      }
      // backward: dh1^T[k][c] = sum_j W2[j][k] dz2^T[j][c], contraction j(s, h) = 32 (s / 16) + acc_row(s % 16, h)
      float dz1r[2][16];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        f32x16 d = f32x16{};
#pragma unroll
        for (int s2 = 0; s2 < 32; ++s2) {
          const int j = 32 * (s2 >> 4) + acc_row(s2 & 15, h);
          d = __builtin_amdgcn_mfma_f32_32x32x2f32(th[OW2 + j * MLP_W + 32 * kb + c], dz2r[s2 >> 4][s2 & 15], d, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dz1r[kb][r] = d[r] * (1.0f - h1r[kb][r] * h1r[kb][r]);
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) L.dz[(32 * kb + acc_row(r, h)) * DZS + c] = dz1r[kb][r];
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // gW1[k][.], gb1[k] for k = lane: sums over the 32 points
      {
        const float4* dzr = reinterpret_cast<const float4*>(L.dz + lane * DZS);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float4 a4 = dzr[q];
          const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int cc = 4 * q + e;
            g_w1x += av[e] * L.xy[cc][0];
            g_w1y += av[e] * L.xy[cc][1];
            g_b1 += av[e];
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    // loss and gb3 of the wave (lanes with h == 0 hold one point each)
    for (int off = 32; off > 0; off >>= 1) {
      loss += __shfl_xor(loss, off, 64);
      g_b3 += __shfl_xor(g_b3, off, 64);
    }
    // the four waves' gradients into four slices of the (now free) wave
    // buffers, then summed per parameter in wave order (fixed, reproducible)
    __syncthreads();
    float* Gw = reinterpret_cast<float*>(WL) + w * GSTRIDE;
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) Gw[OW2 + (32 * jb + acc_row(r, h)) * MLP_W + 32 * kb + c] = gw2[jb][kb][r];
    Gw[OW1 + 2 * lane] = g_w1x;
    Gw[OW1 + 2 * lane + 1] = g_w1y;
    Gw[OB1 + lane] = g_b1;
    Gw[OB2 + lane] = g_b2;
    Gw[OW3 + lane] = g_w3;
    if (lane == 0) { Gw[OB3] = g_b3; Gw[MLP_PARAMS] = loss; }
    __syncthreads();
    const float* G0 = reinterpret_cast<const float*>(WL);
    auto gsum = [&](int q) __attribute__((always_inline)) {
      return ((G0[q] + G0[GSTRIDE + q]) + G0[2 * GSTRIDE + q]) + G0[3 * GSTRIDE + q];
    };
    if (!A.update) {
      if (slice > 0) {
        float* out = A.grad_out + (size_t)blockIdx.x * GPAD;
        for (int q = tid; q <= MLP_PARAMS; q += TW * 64) out[q] = gsum(q);
        return;
      }
      if (tid == 0 && A.losses) A.losses[step] = gsum(MLP_PARAMS);
      for (int q = tid; q < MLP_PARAMS; q += TW * 64) A.grad_out[q] = gsum(q);
      return;
    }
    if (tid == 0 && A.losses) A.losses[step] = gsum(MLP_PARAMS);
    // Adam (bias-corrected), beta1 = 0.9, beta2 = 0.999, eps = 1e-8; each
    // thread keeps the moments of the parameters it owns in registers
    const int tstep = A.step0 + step + 1;
    const float c1 = 1.0f - powf(0.9f, (float)tstep);
    const float c2 = 1.0f - powf(0.999f, (float)tstep);
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
      const int q = tid + i * TW * 64;
      if (q < MLP_PARAMS) {
        const float g = gsum(q);
        const float mq = 0.9f * mown[i] + 0.1f * g;
        const float sq = 0.999f * sown[i] + 0.001f * g * g;
        mown[i] = mq;
        sown[i] = sq;
        th[q] -= A.lr * (mq / c1) / (sqrtf(sq / c2) + 1e-8f);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < OWN; ++i) {
    const int q = tid + i * TW * 64;
    if (q < MLP_PARAMS && A.update) {
      A.m[q] = mown[i];
      A.s[q] = sown[i];
    }
  }
  for (int i = tid; i < MLP_PARAMS; i += TW * 64) A.params[i] = th[i];
}

// The update of a step over slices: their gradients in order, then Adam with the
// moments in global memory.
__global__ __launch_bounds__(256) void k_mlp_adam(float* __restrict__ params, float* __restrict__ m,
                                                  float* __restrict__ s, const float* __restrict__ part, int groups,
                                                  int tstep, float lr, float* losses) {
  const float c1 = 1.0f - powf(0.9f, (float)tstep);
  const float c2 = 1.0f - powf(0.999f, (float)tstep);
  for (int q = threadIdx.x; q <= MLP_PARAMS; q += 256) {
    float g = 0.0f;
    for (int b = 0; b < groups; ++b) g += part[(size_t)b * GPAD + q];
    if (q == MLP_PARAMS) {
      if (losses) *losses = g;
      continue;
    }
    const float mq = 0.9f * m[q] + 0.1f * g;
    const float sq = 0.999f * s[q] + 0.001f * g * g;
    m[q] = mq;
    s[q] = sq;
    params[q] -= lr * (mq / c1) / (sqrtf(sq / c2) + 1e-8f);
  }
}

__global__ void k_mlp_zero(uint32_t* flags) { flags[threadIdx.x] = 0u; }

// Glorot-uniform weights, zero biases: parameter i of a weight matrix with
// fan sum F is lim (2u - 1), lim = sqrt(6 / F), u the float64 uniform of the
// first word of Philox4x32-10 at counter (i, 0, 0, 0), key (seed lo, seed hi)
__global__ __launch_bounds__(BLK) void k_mlp_init(float* __restrict__ params, uint32_t k0, uint32_t k1) {
  const int i = blockIdx.x * BLK + threadIdx.x;
  if (i >= MLP_PARAMS) return;
  int fan = 0;
  if (i < OB1) fan = MLP_W + 2;
  else if (i >= OW2 && i < OB2) fan = 2 * MLP_W;
  else if (i >= OW3 && i < OB3) fan = MLP_W + 1;
  float w = 0.0f;
  if (fan) {
    const double u = uniform64(philox10((uint32_t)i, 0u, 0u, 0u, k0, k1).a);
    w = (float)(sqrt(6.0 / fan) * (2.0 * u - 1.0));
  }
  params[i] = w;
}

}  // namespace

pdd_status run_mlp_init(pdd_ctx* ctx, float* params, uint64_t seed) {
  hipLaunchKernelGGL(k_mlp_init, dim3((MLP_PARAMS + BLK - 1) / BLK), dim3(BLK), 0, ctx->stream, params,
                     (uint32_t)seed, (uint32_t)(seed >> 32));
  return check_hip(ctx, hipGetLastError(), "launch mlp_init");
}

pdd_status run_mlp_eval(pdd_ctx* ctx, const float* params, int64_t n, const float* xy, float* v, float* g) {
  const int grid = (int)std::min<int64_t>(4096, (n + BLK - 1) / BLK);
  hipLaunchKernelGGL(k_mlp_eval, dim3(std::max(grid, 1)), dim3(BLK), 0, ctx->stream, params, n, xy, v, g);
  return check_hip(ctx, hipGetLastError(), "launch mlp_eval");
}

pdd_status run_mlp_grad_bf16(pdd_ctx* ctx, const float* params, int64_t n, const float* xy, float* g) {
  const int64_t waves = (n + 63) / 64;
  const int grid = (int)std::min<int64_t>(2048, (waves + BLK / 64 - 1) / (BLK / 64));
  hipLaunchKernelGGL(k_mlp_grad_bf16, dim3(std::max(grid, 1)), dim3(BLK), 0, ctx->stream, params, n, xy, g);
  return check_hip(ctx, hipGetLastError(), "launch mlp_grad_bf16");
}

pdd_status run_mlp_bake(pdd_ctx* ctx, const float* params, const pdd_partition& part, int32_t lut_n, float* out) {
  const int64_t total = (int64_t)lut_n * lut_n;
  const int grid = (int)std::min<int64_t>(8192, (total + BLK - 1) / BLK);
  hipLaunchKernelGGL(k_mlp_bake, dim3(grid), dim3(BLK), 0, ctx->stream, params, lut_n, part.x0, part.x1, part.y0,
                     part.y1, out);
  return check_hip(ctx, hipGetLastError(), "launch mlp_bake");
}

namespace {

hipError_t waves_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp_train_waves), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)waves_lds_bytes());
}

pdd_status train_by_waves(pdd_ctx* ctx, const TrainArgs& A) {
  const hipError_t e = waves_lds();
  if (e != hipSuccess) return check_hip(ctx, e, "hipFuncSetAttribute(mlp_train)");
  hipLaunchKernelGGL(k_mlp_train_waves, dim3(1), dim3(TW * 64), waves_lds_bytes(), ctx->stream, A, 0, 0);
  return check_hip(ctx, hipGetLastError(), "launch mlp_train");
}

// The slices' gradients of captured calls: allocated by the calls that are not, each
// at least twice as large as the last, and kept with the context, so that a graph's
// buffer stays where it is.  Null: there is none of this size.
float* slice_gradients(pdd_ctx* ctx, size_t bytes, bool captured) {
  auto& all = ctx->mlp_slices;
  const size_t have = all.empty() ? 0 : all.back()->bytes;
  if (bytes > have) {
    if (captured) return nullptr;
    auto fresh = std::make_unique<DeviceBuffer>();
    if (fresh->reserve(std::max(bytes, 2 * have)) != hipSuccess) {
      (void)hipGetLastError();                      // no room: a captured call takes one workgroup
      return nullptr;
    }
    all.push_back(std::move(fresh));
  }
  return all.back()->as<float>();
}

pdd_status train_by_slices(pdd_ctx* ctx, TrainArgs A, int32_t slices, float* grads) {
  const hipError_t e = waves_lds();
  if (e != hipSuccess) return check_hip(ctx, e, "hipFuncSetAttribute(mlp_train)");
  const int32_t steps = A.steps;
  float* losses = A.losses;
  A.update = 0;
  A.steps = 1;
  A.losses = nullptr;
  A.grad_out = grads;
  for (int32_t st = 0; st < steps; ++st) {
    hipLaunchKernelGGL(k_mlp_train_waves, dim3(slices), dim3(TW * 64), waves_lds_bytes(), ctx->stream, A, WIDE_SLICE, st);
    hipLaunchKernelGGL(k_mlp_adam, dim3(1), dim3(256), 0, ctx->stream, A.params, A.m, A.s, A.grad_out, slices,
                       A.step0 + st + 1, A.lr, losses ? losses + st : nullptr);
  }
  return check_hip(ctx, hipGetLastError(), "launch mlp_train (slices)");
}

}  // namespace

pdd_status run_mlp_train(pdd_ctx* ctx, float* params, float* m, float* s, int64_t n_points, const float* xy,
                         const float* target, const int32_t* order, int64_t n_order, int32_t batch, int32_t steps,
                         int32_t step0, float lr, float* losses, float* grad_out) {
  TrainArgs A{};
  A.n_points = n_points;
  A.params = params; A.m = m; A.s = s; A.xy = xy; A.target = target; A.order = order;
  A.n_order = n_order; A.batch = batch; A.steps = steps; A.step0 = step0; A.lr = lr;
  A.update = grad_out ? 0 : 1;
  A.grad_out = grad_out;
  A.losses = losses;
  A.polls = ctx->wait_polls;
  // the gradient entry keeps one slice at any size
  A.slice = !grad_out && batch > WIDE_BATCH ? WIDE_SLICE : batch;
  const int64_t slices = ((int64_t)batch + A.slice - 1) / A.slice;
  A.units = slices > 1 ? (int32_t)(4 * slices) : std::min(4, (batch + 31) / 32);
  // with a slice for every workgroup whole slices keep them as busy, at a quarter of the gradients to exchange
  const bool whole = slices >= TRAIN_G;
  int G = (int)std::min<int64_t>({(int64_t)A.units, (int64_t)TRAIN_G, (int64_t)ctx->cu_count});
  // a captured call, and one step of at most a round of four units: see k_mlp_train_waves
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  const bool captured = hipStreamIsCapturing(ctx->stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusActive;
  if (slices > 1) {
    float* grads = slice_gradients(ctx, (size_t)slices * GPAD * sizeof(float), captured);
    if (captured && grads) return train_by_slices(ctx, A, (int32_t)slices, grads);
  }
  if (slices == 1 && A.units > 1 && (captured || (steps == 1 && batch <= 128))) return train_by_waves(ctx, A);
  if (captured) G = 1;
  const void* f = slices == 1 ? reinterpret_cast<const void*>(&k_mlp_train<ONE>)
                  : whole     ? reinterpret_cast<const void*>(&k_mlp_train<WHOLE>)
                              : reinterpret_cast<const void*>(&k_mlp_train<UNITS>);
  // more than 64 KiB of LDS for one workgroup (gfx950 allows 160 KiB)
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(TrainLds));
  if (e != hipSuccess) return check_hip(ctx, e, "hipFuncSetAttribute(mlp_train)");
  void* args[] = {&A};
  if (G == 1) {
    e = hipLaunchKernel(f, dim3(1), dim3(TT), args, sizeof(TrainLds), ctx->stream);
    return check_hip(ctx, e, "launch mlp_train");
  }
  const size_t part = (size_t)(whole ? slices : slices == 1 ? 8 : A.units) * GPAD;
  const size_t theta = slices == 1 ? 0 : 3 * PARAM_PAD;
  const size_t bytes = (TRAIN_G + theta + part) * sizeof(float);
  const bool fresh = bytes > ctx->mlp_wide.buf.bytes;
  pdd_status st = ctx->mlp_wide.acquire(ctx, bytes);
  if (st != PDD_OK) return st;
  A.flags = ctx->mlp_wide.buf.as<uint32_t>();
  A.theta = ctx->mlp_wide.buf.as<float>() + TRAIN_G;
  A.part = A.theta + theta;
  // Flags only grow: a call goes on from the epochs of the one before (also of one
  // that gave up), and they are cleared in a new buffer and before they would wrap.
  // A clearing kernel before each cooperative launch cost 12 us of a call's 57.
  const uint32_t epochs = 2u * (uint32_t)steps;
  if (fresh || ctx->mlp_epoch > UINT32_MAX - epochs) {
    hipLaunchKernelGGL(k_mlp_zero, dim3(1), dim3(TRAIN_G), 0, ctx->stream, A.flags);
    if ((e = hipGetLastError()) != hipSuccess) return check_hip(ctx, e, "launch mlp_zero");
    ctx->mlp_epoch = 0;
  }
  A.epoch = ctx->mlp_epoch;
  ctx->mlp_epoch += epochs;
  e = hipLaunchCooperativeKernel(f, dim3(G), dim3(TT), args, (unsigned)sizeof(TrainLds), ctx->stream);
  if (e == hipErrorCooperativeLaunchTooLarge) {     // a device that does not hold them all: one workgroup, the same bits
    (void)hipGetLastError();
    e = hipLaunchKernel(f, dim3(1), dim3(TT), args, sizeof(TrainLds), ctx->stream);
  }
  if (e != hipSuccess) return check_hip(ctx, e, "launch mlp_train");
  return ctx->mlp_wide.release(ctx);
}

}  // namespace pdd
