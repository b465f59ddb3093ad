// Solution of the assembled system G u = b (eq. 23): mixed-precision
// iterative refinement.  The outer loop keeps u and the residual
// r = b - G u in float64; each correction G d = r is solved by BiCGStab
// (van der Vorst, 1992) on float32 vectors and a float32 copy of G, with
// float64 dot products.  Scalars of the recurrence live on the device; the
// host reads the residual norm only every few iterations.
//
// Two forms of the same iteration.  Systems of up to SMALL_N unknowns run in
// one launch (k_solve_small): the whole refinement, without a host round
// trip.  Larger ones take a kernel per operation: CSR SpMV with one wave per
// row (rows hold 1 to a few hundred entries), fused vector updates that also
// produce per-block partial dot products, and a one-block reduction that
// finishes the dots and advances the scalars.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "context.h"
#include "grid_exchange.h"

namespace pdd {

namespace {

constexpr int RED_BLOCKS = 256;     // partial-dot blocks
constexpr int BLK = 256;
constexpr int MAX_DEVICES = 64;

// Scratch of pdd_solve_noalloc: a file-scope device array, one copy per GPU
// that runs the library, held until the process ends.  Host code uses only
// its per-device address from hipGetSymbolAddress (solve_noalloc_setup); the
// array's name on the host is a stand-in, not a device address.
__device__ __align__(256) char scratch[SOLVE_NOALLOC_BYTES];
void* g_scratch_ptr[MAX_DEVICES] = {};
std::mutex g_scratch_mu;

// Scalars of one BiCGStab recurrence (device).
struct Scal {
  double rho, rho_new, alpha, omega;
  double rv, ts, tt, rr;
  int32_t broke;                    // breakdown flag
  int32_t pad;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// block-level sum of up to 3 values into partial[q * RED_BLOCKS + blockIdx.x]
template <int NQ>
__device__ __forceinline__ void block_partials(double (&v)[NQ], double* partial) {
  __shared__ double sh[NQ][BLK / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double s = wave_sum(v[q]);
    if (lane == 0) sh[q][wid] = s;
  }
  __syncthreads();
  if (threadIdx.x < NQ) {
    double s = 0.0;
    for (int w = 0; w < BLK / 64; ++w) s += sh[threadIdx.x][w];
    partial[threadIdx.x * RED_BLOCKS + blockIdx.x] = s;
  }
}

// y = A x (one wave per row); optional fused dot d0 = <w, y>
template <typename TA, typename TX>
__global__ __launch_bounds__(BLK) void k_spmv(int64_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                              const TA* __restrict__ val, const TX* __restrict__ x, TX* __restrict__ y) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (BLK / 64) + (threadIdx.x >> 6);
  if (row >= n) return;
  double s = 0.0;
  for (int p = rp[row] + lane; p < rp[row + 1]; p += 64) s += (double)val[p] * (double)x[ci[p]];
  s = wave_sum(s);
  if (lane == 0) y[row] = (TX)s;
}

// r = b - A u (float64) and partial ||r||^2
__global__ __launch_bounds__(BLK) void k_residual(int64_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                                  const double* __restrict__ val, const double* __restrict__ u,
                                                  const double* __restrict__ b, double* __restrict__ r) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (BLK / 64) + (threadIdx.x >> 6);
  if (row >= n) return;
  double s = 0.0;
  for (int p = rp[row] + lane; p < rp[row + 1]; p += 64) s += val[p] * u[ci[p]];
  s = wave_sum(s);
  if (lane == 0) r[row] = b[row] - s;
}

// grid-stride helpers over n with RED_BLOCKS blocks
#define GRID_LOOP(i) for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)RED_BLOCKS * BLK)

__global__ __launch_bounds__(BLK) void k_norm2(int64_t n, const double* __restrict__ a, double* partial) {
  double v[1] = {0.0};
  GRID_LOOP(i) v[0] += a[i] * a[i];
  block_partials<1>(v, partial);
}

// inner start: x = 0, r = rhat = p = float(r64), v = 0; partials <rhat, r>, <r, r>
__global__ __launch_bounds__(BLK) void k_init(int64_t n, const double* __restrict__ r64, float* x, float* r, float* rhat,
                                              float* p, float* v, double* partial) {
  double acc[2] = {0.0, 0.0};
  GRID_LOOP(i) {
    const float ri = (float)r64[i];
    x[i] = 0.0f; r[i] = ri; rhat[i] = ri; p[i] = ri; v[i] = 0.0f;
    acc[0] += (double)ri * ri;
    acc[1] += (double)ri * ri;
  }
  block_partials<2>(acc, partial);
}

// finish partial sums: which = 0: rho_new, rr (start) | 1: rv | 2: ts, tt | 3: rho_next, rr
__global__ __launch_bounds__(BLK) void k_reduce(const double* __restrict__ partial, int nq, int which, Scal* S) {
  __shared__ double sh[3][BLK / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int q = 0; q < nq; ++q) {
    double s = 0.0;
    for (int i = threadIdx.x; i < RED_BLOCKS; i += BLK) s += partial[q * RED_BLOCKS + i];
    s = wave_sum(s);
    if (lane == 0) sh[q][wid] = s;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double t[3] = {0, 0, 0};
  for (int q = 0; q < nq; ++q)
    for (int w = 0; w < BLK / 64; ++w) t[q] += sh[q][w];
  if (which == 0) {
    S->rho = 1.0; S->alpha = 1.0; S->omega = 1.0; S->rho_new = t[0]; S->rr = t[1]; S->broke = 0;
  } else if (which == 1) {
    S->rv = t[0];
    if (!(t[0] != 0.0) || !isfinite(t[0])) S->broke = 1;
  } else if (which == 2) {
    S->ts = t[0]; S->tt = t[1];
    if (!isfinite(t[0]) || !isfinite(t[1])) S->broke = 1;
  } else {
    // an exact half-step solution (s = 0, omega = 0) ends the recurrence here
    S->rho = S->rho_new; S->rho_new = t[0]; S->rr = t[1];
    if (!(t[0] != 0.0) || !isfinite(t[0]) || S->omega == 0.0) S->broke = 1;
  }
}

// p = r + beta (p - omega v), beta = (rho_new / rho) (alpha / omega); first iteration p = r
__global__ __launch_bounds__(BLK) void k_update_p(int64_t n, int first, const Scal* S, const float* r, const float* v, float* p) {
  if (S->broke) return;
  const double beta = first ? 0.0 : (S->rho_new / S->rho) * (S->alpha / S->omega);
  const float fb = (float)beta, fo = (float)S->omega;
  GRID_LOOP(i) p[i] = r[i] + fb * (p[i] - fo * v[i]);
}

// alpha = rho_new / <rhat, v>; s = r - alpha v
__global__ __launch_bounds__(BLK) void k_update_s(int64_t n, Scal* S, const float* r, const float* v, float* s) {
  if (S->broke) return;
  const double alpha = S->rho_new / S->rv;
  if (blockIdx.x == 0 && threadIdx.x == 0) S->alpha = alpha;
  const float fa = (float)alpha;
  GRID_LOOP(i) s[i] = r[i] - fa * v[i];
}

// partial <t, s>, <t, t>
__global__ __launch_bounds__(BLK) void k_dots_ts(int64_t n, const float* t, const float* s, double* partial) {
  double acc[2] = {0.0, 0.0};
  GRID_LOOP(i) { acc[0] += (double)t[i] * s[i]; acc[1] += (double)t[i] * t[i]; }
  block_partials<2>(acc, partial);
}

// partial <rhat, v>
__global__ __launch_bounds__(BLK) void k_dot_rv(int64_t n, const float* rhat, const float* v, double* partial) {
  double acc[1] = {0.0};
  GRID_LOOP(i) acc[0] += (double)rhat[i] * v[i];
  block_partials<1>(acc, partial);
}

// omega = <t,s>/<t,t>; x += alpha p + omega s; r = s - omega t; partials <rhat, r>, <r, r>
__global__ __launch_bounds__(BLK) void k_update_xr(int64_t n, Scal* S, const float* p, const float* s, const float* t,
                                                   const float* rhat, float* x, float* r, double* partial) {
  double acc[2] = {0.0, 0.0};
  if (!S->broke) {
    const double omega = S->tt > 0.0 ? S->ts / S->tt : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) S->omega = omega;
    const float fa = (float)S->alpha, fo = (float)omega;
    GRID_LOOP(i) {
      x[i] = x[i] + fa * p[i] + fo * s[i];
      const float ri = s[i] - fo * t[i];
      r[i] = ri;
      acc[0] += (double)rhat[i] * ri;
      acc[1] += (double)ri * ri;
    }
  }
  block_partials<2>(acc, partial);
}

// u += x (float64)
__global__ __launch_bounds__(BLK) void k_accumulate(int64_t n, const float* x, double* u) {
  GRID_LOOP(i) u[i] += (double)x[i];
}

// CSR sanity, one wave per row: row_ptr from 0, non-decreasing and within
// nnz = row_ptr[n], column indices in [0, n).  The rows' entries go to the
// float32 copy on the way (val32).
__global__ __launch_bounds__(BLK) void k_check_csr(int64_t n, int32_t nnz, const int32_t* __restrict__ rp,
                                                   const int32_t* __restrict__ ci, const double* __restrict__ val,
                                                   float* __restrict__ val32, int32_t* bad) {
  const int lane = threadIdx.x & 63;
  for (int64_t i = (int64_t)blockIdx.x * (BLK / 64) + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * (BLK / 64)) {
    const int32_t a = rp[i], e = rp[i + 1];
    if ((i == 0 && a != 0) || a < 0 || e < a || e > nnz) {
      if (lane == 0) *bad = 1;
      continue;
    }
    bool off = false;
    for (int32_t p = a + lane; p < e; p += 64) {
      off |= ci[p] < 0 || ci[p] >= n;
      val32[p] = (float)val[p];
    }
    if (off) *bad = 1;
  }
}

__global__ __launch_bounds__(BLK) void k_zero(int64_t n, double* u) {
  GRID_LOOP(i) u[i] = 0.0;
}

__global__ void k_zero_words(int32_t* w, int32_t count) {
  if ((int)threadIdx.x < count) w[threadIdx.x] = 0;
}

// ---- the whole solve in one launch ------------------------------------------
// Bound by latency: a system of a few thousand unknowns is a chain of some
// forty iterations with two products and three reductions each, and as ten
// launches an iteration it took 60 us (1729 unknowns, 40 to 44 iterations: 2.6 ms;
// now 0.79 ms; 29 unknowns 0.57 ms, now 0.085; 15,105 5.9 ms, now 3.2).
// Here G workgroups (at most one per CU) each own a contiguous range of rows
// and keep the whole vectors r, p, v redundantly in registers (thread t
// holds the elements t + 1024 k, k < K), with rhat and the vector being
// multiplied in LDS.  Every update and dot product is then local to the
// workgroup, the same operations in the same order everywhere, so all
// workgroups hold the same bits and take the same branches; only the rows'
// products are exchanged, twice an iteration (G = 1: never).
//
// Exchange (grid_exchange.h): a buffer is rewritten only two exchanges later,
// after every workgroup has flagged that it finished reading it.  (Agent fences
// and plain loads instead: each fence drops the XCD's cached matrix, 2 to 6
// times slower.  Words carrying value and exchange number, polled without flags:
// 2 % slower at 1729 unknowns, 40 % at 15,105.)
// The launch is cooperative (the runtime keeps all workgroups resident
// together) and every wait is bounded: one that runs out ends the kernel and
// the solve is done by the kernel-per-operation form.
constexpr int SMALL_T = 1024;
constexpr int SMALL_N = 16 * SMALL_T;
constexpr int SMALL_G = 256;               // at most this many workgroups
constexpr int SMALL_ROWS = 2048;           // rows of one workgroup, at most
constexpr int INNER_MAX = 400;             // BiCGStab iterations of one correction
constexpr double INNER_TOL = 1e-5;         // and its residual against the correction's right-hand side
constexpr int OUTER_MAX = 50;

enum { SMALL_DONE = 0, SMALL_MALFORMED = 1, SMALL_TIMEOUT = 2 };
struct SmallResult {
  double rel;
  int32_t iters;
  int32_t state;
};

struct SmallArgs {
  int64_t n;
  const int32_t* rp;
  const int32_t* ci;
  const double* val;
  const float* val32;
  const double* b;
  double* u;
  double* r64;               // exchange buffers: residual, products v and t
  float* v;
  float* t;
  uint32_t* flags;           // SMALL_G epoch flags, zeroed before the launch
  const int32_t* bad;        // set by k_check_csr
  SmallResult* result;
  double tol;
  int32_t max_iter;
  uint32_t polls;            // of a wait between workgroups (grid_exchange.h)
};

// One DPP step of a sum: each lane adds the value of the lane the control
// selects (0 outside the row of 16 lanes, or in a row that is masked off).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
// Sum of a row of 16 lanes left in its last lane, by shifts of 1, 2, 4 and 8.
__device__ __forceinline__ double row_sum_last(double v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  return dpp_add<0x118, 0xf>(v);
}
// Wave sum left in lane 63: the rows, then their broadcasts.
__device__ __forceinline__ double wave_sum_last(double v) {
  v = row_sum_last(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// A matrix row's product with x (LDS) by 16 lanes, left in the last of them.
// FLY entries per lane are in flight at once: a row is a chain of L2 reads
// and LDS gathers, and a workgroup has only tens of rows (8 against 4: 5 %
// faster from 5661 unknowns, 5 % slower at 29).
template <int FLY, typename TA, typename TX>
__device__ __forceinline__ double row_product(const TA* __restrict__ val, const int32_t* __restrict__ ci, const TX* x,
                                              int begin, int end, int l16) {
  double s = 0.0;
  for (int q = begin + l16; q < end; q += 16 * FLY) {
    TA a[FLY];
    int32_t c[FLY];
#pragma unroll
    for (int j = 0; j < FLY; ++j) {
      const int at = q + 16 * j < end ? q + 16 * j : q;
      a[j] = val[at];
      c[j] = ci[at];
    }
#pragma unroll
    for (int j = 0; j < FLY; ++j)
      if (q + 16 * j < end) s += (double)a[j] * (double)x[c[j]];
  }
  return row_sum_last(s);
}

template <int K>
__global__ __launch_bounds__(SMALL_T) void k_solve_small(SmallArgs A) {
  extern __shared__ double lds[];              // the multiplied vector and rhat, or u (refinement)
  __shared__ double red[2][SMALL_T / 64][2];
  __shared__ int32_t rows[SMALL_ROWS + 1];
  __shared__ float local[SMALL_ROWS];          // G = 1: the product
  __shared__ float x[SMALL_ROWS];              // the correction, own rows
  __shared__ int32_t stop;
  float* g32 = reinterpret_cast<float*>(lds);
  float* rhat = g32 + A.n;                     // beside the multiplied vector
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = (int)A.n, G = gridDim.x, me = blockIdx.x;
  const int row0 = (int)(A.n * me / G), row1 = (int)(A.n * (me + 1) / G);
  if (*A.bad) {
    if (me == 0 && tid == 0) *A.result = SmallResult{0.0, 0, SMALL_MALFORMED};
    return;
  }
  for (int i = tid; i <= row1 - row0; i += SMALL_T) rows[i] = A.rp[row0 + i];
  if (tid == 0) stop = 0;
  __syncthreads();

  constexpr int FLY = K <= 2 ? 4 : 8;
  uint32_t epoch = 0;
  auto exchange = [&]() __attribute__((always_inline)) -> bool {
    return grid_exchange(A.flags, G, me, ++epoch, &stop, A.polls);
  };
  // sums of two values over the workgroup, the same bits in every thread
  int par = 0;
  auto block_sums = [&](double a, double b, double& sa, double& sb) __attribute__((always_inline)) {
    a = wave_sum_last(a);
    b = wave_sum_last(b);
    par ^= 1;                                  // two buffers: one barrier per reduction
    if (lane == 63) {
      red[par][w][0] = a;
      red[par][w][1] = b;
    }
    __syncthreads();
    // every row of 16 lanes sums the sixteen waves
    sa = readlane_f64(row_sum_last(red[par][lane & 15][0]), 15);
    sb = readlane_f64(row_sum_last(red[par][lane & 15][1]), 15);
  };
  static_assert(SMALL_T / 64 == 16, "sixteen waves per workgroup");
  // the thread's elements; its index is made opaque to each loop, or the
  // compiler keeps every element's address of every array in registers
  auto opaque = [](int t) __attribute__((always_inline)) -> int {
    __asm__ volatile("" : "+v"(t));
    return t;
  };
#define FOR_OWN(i) _Pragma("unroll") for (int k = 0, i = opaque(tid); k < K; ++k, i += SMALL_T) if (i < n)
  // float32 product of this workgroup's rows with the vector in LDS, published
  auto product = [&](float* out) __attribute__((always_inline)) {
    __syncthreads();
    for (int row = tid >> 4; row < row1 - row0; row += SMALL_T / 16) {
      const float s = (float)row_product<FLY>(A.val32, A.ci, g32, rows[row], rows[row + 1], tid & 15);
      if ((tid & 15) == 15) {
        if (G == 1) local[row] = s;
        else agent_store(out + row0 + row, s);
      }
    }
  };
  // every workgroup's products, this thread's elements; false: a wait ran out
  auto collect = [&](const float* in, float (&out)[K]) __attribute__((always_inline)) -> bool {
    if (!exchange()) return false;
    if (G == 1) {
      FOR_OWN(i) out[k] = local[i];
    } else {
      FOR_OWN(i) out[k] = agent_load(in + i);
    }
    return true;
  };

  double bb = 0.0, dummy;
  FOR_OWN(i) bb += A.b[i] * A.b[i];
  block_sums(bb, 0.0, bb, dummy);
  const double bnorm = sqrt(bb);
  int total = 0;
  double rel = 1.0;
  bool late = false;                           // a wait ran out
  for (int i = row0 + tid; i < row1; i += SMALL_T) agent_store(A.u + i, 0.0);
  if (bnorm == 0.0) rel = 0.0;
  float r[K], p[K], v[K];
  for (int outer = 0; bnorm != 0.0 && outer < OUTER_MAX && !late; ++outer) {
    // ---- float64 residual of the iterate (b itself for u = 0) --------------
    double rr = 0.0, rr32 = 0.0;
    if (outer > 0) {
      if ((late = !exchange())) break;
      for (int i = tid; i < n; i += SMALL_T) lds[i] = agent_load(A.u + i);
      __syncthreads();
      for (int row = tid >> 4; row < row1 - row0; row += SMALL_T / 16) {
        const double s = row_product<FLY>(A.val, A.ci, lds, rows[row], rows[row + 1], tid & 15);
        if ((tid & 15) == 15) agent_store(A.r64 + row0 + row, A.b[row0 + row] - s);
      }
      if ((late = !exchange())) break;
    }
    FOR_OWN(i) {
      const double ri = outer > 0 ? agent_load(A.r64 + i) : A.b[i];
      rr += ri * ri;
      r[k] = (float)ri;
      rr32 += (double)r[k] * r[k];
    }
    block_sums(rr, rr32, rr, rr32);
    rel = sqrt(rr) / bnorm;
    if (!(rel > A.tol) || total >= A.max_iter) break;
    // ---- BiCGStab on G d = r -------------------------------------------------
    FOR_OWN(i) {
      if (i >= row0 && i < row1) x[i - row0] = 0.0f;
      rhat[i] = r[k];
      p[k] = r[k];
      v[k] = 0.0f;
    }
    const double r0 = sqrt(rr);
    double rho = 1.0, rho_new = rr32, alpha = 1.0, omega = 1.0;
    rr = rr32;
    bool broke = false;
    for (int it = 0; it < INNER_MAX && total < A.max_iter; ++it, ++total) {
      if (!broke) {
        // p = r + beta (p - omega v)
        const float fb = it == 0 ? 0.0f : (float)((rho_new / rho) * (alpha / omega)), fo = (float)omega;
        FOR_OWN(i) {
          p[k] = r[k] + fb * (p[k] - fo * v[k]);
          g32[i] = p[k];
        }
        product(A.v);
        double rv = 0.0, ts = 0.0, tt = 0.0, rh = 0.0;
        if ((late = !collect(A.v, v))) break;
        FOR_OWN(i) rv += (double)rhat[i] * v[k];
        block_sums(rv, 0.0, rv, dummy);
        if (!(rv != 0.0) || !isfinite(rv)) broke = true;
        if (!broke) {
          // s = r - alpha v, kept in r
          alpha = rho_new / rv;
          const float fa = (float)alpha;
          FOR_OWN(i) {
            r[k] = r[k] - fa * v[k];
            g32[i] = r[k];
          }
          product(A.t);
          float t[K];
          if ((late = !collect(A.t, t))) break;
          FOR_OWN(i) {
            ts += (double)t[k] * r[k];
            tt += (double)t[k] * t[k];
          }
          block_sums(ts, tt, ts, tt);
          if (!isfinite(ts) || !isfinite(tt)) broke = true;
          if (!broke) {
            omega = tt > 0.0 ? ts / tt : 0.0;
            const float fw = (float)omega;
            rr = 0.0;
            FOR_OWN(i) {
              if (i >= row0 && i < row1) x[i - row0] = x[i - row0] + fa * p[k] + fw * r[k];
              r[k] = r[k] - fw * t[k];
              rh += (double)rhat[i] * r[k];
              rr += (double)r[k] * r[k];
            }
            block_sums(rh, rr, rh, rr);
            rho = rho_new;
            rho_new = rh;
            // an exact half-step solution (s = 0, omega = 0) ends the recurrence here
            if (!(rho_new != 0.0) || !isfinite(rho_new) || omega == 0.0) broke = true;
          }
        }
      }
      if ((it & 3) == 3 && (broke || sqrt(rr) <= INNER_TOL * r0)) { ++total; break; }
    }
    if (late) break;
    // u += x, each workgroup its rows
    FOR_OWN(i) {
      if (i >= row0 && i < row1) agent_store(A.u + i, agent_load(A.u + i) + (double)x[i - row0]);
    }
  }
#undef FOR_OWN
  if (late && tid == 0) A.result->state = SMALL_TIMEOUT;
  if (!late && me == 0 && tid == 0) {
    A.result->rel = rel;
    A.result->iters = total;
  }
}

template <int K>
hipError_t launch_small_k(SmallArgs& A, int G, hipStream_t stream) {
  const void* f = reinterpret_cast<const void*>(&k_solve_small<K>);
  const size_t lds = (size_t)A.n * sizeof(double);
  hipError_t e;
  if (lds > 32768 && (e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) != hipSuccess)
    return e;
  void* args[] = {&A};
  if (G == 1) return hipLaunchKernel(f, dim3(G), dim3(SMALL_T), args, lds, stream);
  return hipLaunchCooperativeKernel(f, dim3(G), dim3(SMALL_T), args, (unsigned)lds, stream);
}

// Workgroups.  More of them shorten the products and lengthen the exchanges:
// a product of about 4000 entries per workgroup (four per thread) takes 1.3 us,
// an exchange 1.7 us among 31 and 2.1 us among 122 workgroups.  Measured: 53 k
// entries best at 13 to 26 workgroups (0.31 ms; 7: 0.35), 250 k at 31 (0.76 ms;
// 61: 0.82, 122: 0.94, 16: 1.0), 1.6 M at 100 (1.71 ms; 199: 1.82), 4.4 M at the
// device's 256.  Below 2048 entries one workgroup needs no exchange.
int small_groups(int64_t n, int32_t nnz, int cu_count) {
  const int64_t few = std::min<int64_t>(32, ((int64_t)nnz + 2047) / 2048);
  const int64_t want = std::max(few, ((int64_t)nnz + 16383) / 16384);
  const int64_t least = (n + SMALL_ROWS - 1) / SMALL_ROWS;
  return (int)std::max(least, std::min<int64_t>({want, (int64_t)SMALL_G, (int64_t)cu_count, n}));
}

hipError_t launch_small(SmallArgs& A, int G, hipStream_t stream) {
  if (G < 1 || G > SMALL_G || A.n > SMALL_N || (A.n + G - 1) / G > SMALL_ROWS) return hipErrorInvalidValue;
  if (A.n <= 2 * SMALL_T) return launch_small_k<2>(A, G, stream);
  if (A.n <= 4 * SMALL_T) return launch_small_k<4>(A, G, stream);
  if (A.n <= 8 * SMALL_T) return launch_small_k<8>(A, G, stream);
  return launch_small_k<16>(A, G, stream);
}

// Bytes of solver scratch for n unknowns and nnz entries: float32 matrix,
// 7 float32 vectors, float64 residual, partials, scalars (and padding).
size_t solve_bytes(int64_t n, int64_t nnz) {
  return ((size_t)nnz + 7 * (size_t)n) * sizeof(float) + ((size_t)n + 3 * RED_BLOCKS) * sizeof(double) +
         sizeof(Scal) + 256;
}

// nnz = row_ptr[n] (synchronises the stream)
pdd_status read_nnz(pdd_ctx* ctx, int64_t n, const int32_t* rp, int32_t* nnz) {
  hipError_t e;
  if ((e = hipMemcpyAsync(ctx->host_words, rp + n, sizeof(int32_t), hipMemcpyDeviceToHost, ctx->stream)) != hipSuccess)
    return check_hip(ctx, e, "read nnz");
  if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) return check_hip(ctx, e, "hipStreamSynchronize");
  *nnz = *static_cast<const int32_t*>(ctx->host_words);
  if (*nnz < 1) {
    ctx->err = "pdd_solve: empty matrix (row_ptr[n] < 1)";
    return PDD_EINVAL;
  }
  return PDD_OK;
}

// Validate the CSR structure on the device before any kernel indexes with it,
// and fill the float32 copy of its values (flag: one device int32, cleared
// here by a kernel along with `extra` words behind it).
hipError_t launch_check(pdd_ctx* ctx, int64_t n, int32_t nnz, const int32_t* rp, const int32_t* ci, const double* val,
                        float* val32, int32_t* flag, int32_t words) {
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(1024), 0, ctx->stream, flag, words);
  const int64_t waves = (n + BLK / 64 - 1) / (BLK / 64);
  hipLaunchKernelGGL(k_check_csr, dim3((unsigned)std::min<int64_t>(4096, waves)), dim3(BLK), 0, ctx->stream, n, nnz, rp,
                     ci, val, val32, flag);
  return hipGetLastError();
}

pdd_status malformed(pdd_ctx* ctx) {
  ctx->err = "pdd_solve: malformed CSR (row_ptr not monotone from 0, or a column outside [0, n))";
  return PDD_EINVAL;
}

pdd_status finish(pdd_ctx* ctx, double tol, int32_t total, double rel, int32_t* iters, double* relres) {
  *iters = total;
  *relres = rel;
  if (!(rel <= tol)) {
    ctx->err = "pdd_solve: tolerance not reached within max_iter";
    return PDD_ENOTCONV;
  }
  return PDD_OK;
}

// The solve in one launch, on scratch as solve_body's.  *late: a wait
// between the workgroups ran out and nothing has been decided.
pdd_status solve_small(pdd_ctx* ctx, int64_t n, int32_t nnz, const int32_t* rp, const int32_t* ci, const double* val,
                       const double* b, double* u, double tol, int32_t max_iter, int32_t* iters, double* relres,
                       char* base, bool* late) {
  *late = false;
  hipError_t e;
  SmallArgs A{};
  A.n = n;
  A.rp = rp; A.ci = ci; A.val = val; A.b = b; A.u = u;
  A.tol = tol;
  A.max_iter = max_iter;
  A.polls = ctx->wait_polls;
  // result and flags first (cleared together), then the buffers
  int32_t* words = reinterpret_cast<int32_t*>(base);
  A.result = reinterpret_cast<SmallResult*>(base);
  int32_t* bad = words + 4;
  A.bad = bad;
  A.flags = reinterpret_cast<uint32_t*>(words + 64);
  A.r64 = reinterpret_cast<double*>(base + 2048);
  A.v = reinterpret_cast<float*>(A.r64 + n);
  A.t = A.v + n;
  float* val32 = A.t + n;
  A.val32 = val32;
  static_assert(sizeof(SmallResult) == 16 && (64 + SMALL_G) * 4 <= 2048, "scratch head");
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(1024), 0, ctx->stream, words, 64 + SMALL_G);
  const int64_t waves = (n + BLK / 64 - 1) / (BLK / 64);
  hipLaunchKernelGGL(k_check_csr, dim3((unsigned)waves), dim3(BLK), 0, ctx->stream, n, nnz, rp, ci, val, val32, bad);
  if ((e = hipGetLastError()) != hipSuccess) return check_hip(ctx, e, "launch csr check");
  e = launch_small(A, small_groups(n, nnz, ctx->cu_count), ctx->stream);
  if (e == hipErrorCooperativeLaunchTooLarge) {
    (void)hipGetLastError();
    *late = true;
    return PDD_OK;
  }
  if (e != hipSuccess) return check_hip(ctx, e, "launch solve");
  SmallResult h;
  if ((e = hipMemcpyAsync(ctx->host_words, A.result, sizeof(h), hipMemcpyDeviceToHost, ctx->stream)) != hipSuccess) return check_hip(ctx, e, "read result");
  if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) return check_hip(ctx, e, "hipStreamSynchronize");
  h = *static_cast<const SmallResult*>(ctx->host_words);
  if (h.state == SMALL_MALFORMED) return malformed(ctx);
  if (h.state == SMALL_TIMEOUT) {
    *late = true;
    return PDD_OK;
  }
  return finish(ctx, tol, h.iters, h.rel, iters, relres);
}

// The refinement loop on caller-provided scratch of solve_bytes(n, nnz) bytes
// (256-byte aligned); allocates nothing.
pdd_status solve_body(pdd_ctx* ctx, int64_t n, int32_t nnz, const int32_t* rp, const int32_t* ci, const double* val,
                      const double* b, double* u, double tol, int32_t max_iter, int32_t* iters, double* relres,
                      char* base) {
  hipError_t e;
  if (n <= SMALL_N) {
    bool late = false;
    const pdd_status st = solve_small(ctx, n, nnz, rp, ci, val, b, u, tol, max_iter, iters, relres, base, &late);
    if (!late) return st;
  }
  hipStream_t st = ctx->stream;
  double* r64 = reinterpret_cast<double*>(base);
  double* partial = r64 + n;
  Scal* S = reinterpret_cast<Scal*>(partial + 3 * RED_BLOCKS);
  float* val32 = reinterpret_cast<float*>(reinterpret_cast<char*>(S) + 128);
  float* x = val32 + nnz;
  float* r = x + n;
  float* rhat = r + n;
  float* p = rhat + n;
  float* v = p + n;
  float* s = v + n;
  float* t = s + n;

  const unsigned rows_grid = (unsigned)((n + BLK / 64 - 1) / (BLK / 64));
  auto L = [&](const char* what) -> pdd_status { return check_hip(ctx, hipGetLastError(), what); };
  pdd_status ps;

  int32_t* flag = reinterpret_cast<int32_t*>(partial);       // free until the first norm
  if ((e = launch_check(ctx, n, nnz, rp, ci, val, val32, flag, 1)) != hipSuccess) return check_hip(ctx, e, "launch csr check");
  int32_t hbad = 0;
  if ((e = hipMemcpyAsync(&hbad, flag, sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess) return check_hip(ctx, e, "read flag");
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return check_hip(ctx, e, "hipStreamSynchronize");
  if (hbad) return malformed(ctx);
  hipLaunchKernelGGL(k_zero, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, u);
  hipLaunchKernelGGL(k_norm2, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, b, partial);
  if ((ps = L("solve setup")) != PDD_OK) return ps;
  double hp[RED_BLOCKS];
  if ((e = hipMemcpyAsync(hp, partial, RED_BLOCKS * sizeof(double), hipMemcpyDeviceToHost, st)) != hipSuccess) return check_hip(ctx, e, "read |b|");
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return check_hip(ctx, e, "hipStreamSynchronize");
  double bb = 0.0;
  for (double q : hp) bb += q;
  const double bnorm = std::sqrt(bb);
  if (bnorm == 0.0) {
    *iters = 0;
    *relres = 0.0;
    return PDD_OK;   // u = 0 solves G u = 0
  }

  int total = 0;
  double rel = 1.0;
  for (int outer = 0; outer < OUTER_MAX; ++outer) {
    // float64 residual of the current iterate
    hipLaunchKernelGGL(k_residual, dim3(rows_grid), dim3(BLK), 0, st, n, rp, ci, val, u, b, r64);
    hipLaunchKernelGGL(k_norm2, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, r64, partial);
    if ((ps = L("residual")) != PDD_OK) return ps;
    if ((e = hipMemcpyAsync(hp, partial, RED_BLOCKS * sizeof(double), hipMemcpyDeviceToHost, st)) != hipSuccess) return check_hip(ctx, e, "read residual");
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return check_hip(ctx, e, "hipStreamSynchronize");
    double rr = 0.0;
    for (double q : hp) rr += q;
    rel = std::sqrt(rr) / bnorm;
    if (!(rel > tol) || total >= max_iter) break;

    // BiCGStab on G d = r (float32 vectors), d accumulated into u
    hipLaunchKernelGGL(k_init, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, r64, x, r, rhat, p, v, partial);
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(BLK), 0, st, partial, 2, 0, S);
    const double r0 = std::sqrt(rr);
    for (int it = 0; it < INNER_MAX && total < max_iter; ++it, ++total) {
      hipLaunchKernelGGL(k_update_p, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, it == 0 ? 1 : 0, S, r, v, p);
      hipLaunchKernelGGL((k_spmv<float, float>), dim3(rows_grid), dim3(BLK), 0, st, n, rp, ci, val32, p, v);
      hipLaunchKernelGGL(k_dot_rv, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, rhat, v, partial);
      hipLaunchKernelGGL(k_reduce, dim3(1), dim3(BLK), 0, st, partial, 1, 1, S);
      hipLaunchKernelGGL(k_update_s, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, S, r, v, s);
      hipLaunchKernelGGL((k_spmv<float, float>), dim3(rows_grid), dim3(BLK), 0, st, n, rp, ci, val32, s, t);
      hipLaunchKernelGGL(k_dots_ts, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, t, s, partial);
      hipLaunchKernelGGL(k_reduce, dim3(1), dim3(BLK), 0, st, partial, 2, 2, S);
      hipLaunchKernelGGL(k_update_xr, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, S, p, s, t, rhat, x, r, partial);
      hipLaunchKernelGGL(k_reduce, dim3(1), dim3(BLK), 0, st, partial, 2, 3, S);
      if ((ps = L("bicgstab")) != PDD_OK) return ps;
      if ((it & 3) == 3) {
        Scal hs;
        if ((e = hipMemcpyAsync(&hs, S, sizeof(Scal), hipMemcpyDeviceToHost, st)) != hipSuccess) return check_hip(ctx, e, "read scalars");
        if ((e = hipStreamSynchronize(st)) != hipSuccess) return check_hip(ctx, e, "hipStreamSynchronize");
        if (hs.broke || std::sqrt(hs.rr) <= INNER_TOL * r0) { ++total; break; }
      }
    }
    hipLaunchKernelGGL(k_accumulate, dim3(RED_BLOCKS), dim3(BLK), 0, st, n, x, u);
    if ((ps = L("accumulate")) != PDD_OK) return ps;
  }
  return finish(ctx, tol, total, rel, iters, relres);
}

}  // namespace

pdd_status run_solve(pdd_ctx* ctx, int64_t n, const int32_t* rp, const int32_t* ci, const double* val,
                     const double* b, double* u, double tol, int32_t max_iter, int32_t* iters, double* relres) {
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return check_hip(ctx, e, "hipSetDevice");
  int32_t nnz = 0;
  pdd_status ps = read_nnz(ctx, n, rp, &nnz);
  if (ps != PDD_OK) return ps;
  if ((e = ctx->solve_scratch.reserve(solve_bytes(n, nnz))) != hipSuccess) return check_hip(ctx, e, "hipMalloc(solve scratch)");
  return solve_body(ctx, n, nnz, rp, ci, val, b, u, tol, max_iter, iters, relres, ctx->solve_scratch.as<char>());
}

hipError_t solve_noalloc_setup(int device) {
  if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = ptr;
  return hipSuccess;
}

pdd_status run_solve_noalloc(pdd_ctx* ctx, int64_t n, const int32_t* rp, const int32_t* ci, const double* val,
                             const double* b, double* u, double tol, int32_t max_iter, int32_t* iters,
                             double* relres) {
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return check_hip(ctx, e, "hipSetDevice");
  if ((e = solve_noalloc_setup(ctx->device)) != hipSuccess) return check_hip(ctx, e, "hipGetSymbolAddress(solve scratch)");
  char* base = static_cast<char*>(g_scratch_ptr[ctx->device]);
  int32_t nnz = 0;
  pdd_status ps = read_nnz(ctx, n, rp, &nnz);
  if (ps != PDD_OK) return ps;
  if (solve_bytes(n, nnz) + 256 > SOLVE_NOALLOC_BYTES) {
    ctx->err = "pdd_solve_noalloc: n and nnz need more than the static 128 MiB of scratch "
               "(4 (nnz + 7 n) + 8 n bytes plus 7 KiB)";
    return PDD_EINVAL;
  }
  return solve_body(ctx, n, nnz, rp, ci, val, b, u, tol, max_iter, iters, relres, base);
}

}  // namespace pdd
