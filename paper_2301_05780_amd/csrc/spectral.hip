// Pseudospectral subdomain solves (Sec. 3.3, Sec. 5.1) and the global u0(x)
// they define (Sec. 4.3, Phase I), for constant-coefficient operators
// 1/2 a_xx u_xx + 1/2 a_yy u_yy + c u = f.
//
// Every square of the partition carries the tensor grid of the p + 1
// Chebyshev-Gauss-Lobatto points per direction.  Its side values come from
// the knot values (hat or inverse-multiquadric cardinal interpolation along
// the grid line over the side's extended stencil) or from g on the domain
// boundary; the interior values solve the collocation system
//   ax E U + ay U E^T + c U = F,   E = D2[1..p-1][1..p-1],
// F the source at the interior points minus the boundary columns of D2
// applied to the side values.  With E = V diag(lam) V^{-1} (host, once per
// p) the solve is four dense products and a pointwise division:
//   U = V [(V^{-1} F V^{-T}) / (ax lam_i + ay lam_j + c)] V^T,
// run per square by one workgroup of sixteen waves on the float64 matrix
// cores (v_mfma_f64_16x16x4_f64) with 64 x 64 tiles in LDS.  Two more products
// give the grid derivatives (2/S) D U and U ((2/S) D)^T.
//
// Grid layout (device, float64): grid[s][f][i][j], square s = a + H c (a
// along x), field f = 0 (u), 1 (du/dx), 2 (du/dy), i the x index and j the y
// index of the point (x_a + S (t_i + 1) / 2, y_c + S (t_j + 1) / 2).
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "spectral.h"

namespace pdd {

namespace {

constexpr int LDT = SPEC_T + 1;     // LDS row stride (doubles): spreads a fragment over the banks
typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double* gfield(const SpecArgs& A, int64_t s, int f) {
  const int N = A.p + 1;
  return A.grid + ((size_t)s * 3 + f) * (size_t)N * N;
}

// lattice value of the line at lattice coordinate `at` (vertical: x = const)
// at along-line lattice point q: g on the domain boundary, else the knot value
template <int KIND>
__device__ __forceinline__ double lattice_value(const SpecArgs& A, bool vert, int at, int q) {
  const AsmParams& P = A.P;
  if (q == 0 || q == P.L) {
    const double lx = vert ? P.x0 + (double)at * P.dx : P.x0 + (double)q * P.dx;
    const double ly = vert ? P.y0 + (double)q * P.dy : P.y0 + (double)at * P.dy;
    return g_at<KIND>(lx, ly);
  }
  const int ix = vert ? at : q, iy = vert ? q : at;
  return A.u_knots[P.lattice[(size_t)iy * (P.L + 1) + ix]];
}

// Side values and the source, one launch.  The first `side_blocks`
// workgroups: one wave per (square, side); side o = 0 (S), 1 (N), 2 (W),
// 3 (E).  The horizontal sides take all p + 1 points (the corners included),
// the vertical sides the p - 1 interior ones.  The other workgroups: one
// thread per interior point, whose source value waits in the grid's u field
// for k_spec_solve.  The source is float64 transcendentals (EQ43: four
// sincos and a tanh per point, 384,400 points for 100 squares at p = 63) and
// would keep the solve's few workgroups busy for two thirds of their time;
// here every CU takes part (17 us for both, the sides alone 8 us).
template <int KIND>
__global__ __launch_bounds__(256) void k_spec_sides(SpecArgs A, int32_t smax, int32_t side_blocks) {
  extern __shared__ double sv[];
  const AsmParams& P = A.P;
  if ((int)blockIdx.x >= side_blocks) {
    const int n = A.p - 1;
    const int64_t q = (int64_t)((int)blockIdx.x - side_blocks) * 256 + threadIdx.x;
    if (q >= (int64_t)A.H * A.H * n * n) return;
    const int j = (int)(q % n), i = (int)((q / n) % n);
    const int64_t sq = q / ((int64_t)n * n);
    const int a = (int)(sq % A.H), c = (int)(sq / A.H);
    const double Sx = (P.x1 - P.x0) / A.H, Sy = (P.y1 - P.y0) / A.H;
    const double x = P.x0 + a * Sx + Sx * (A.T.nodes[i + 1] + 1.0) * 0.5;
    const double y = P.y0 + c * Sy + Sy * (A.T.nodes[j + 1] + 1.0) * 0.5;
    Coef<double> cf;
    coef_at<KIND>(P.coef, x, y, cf);
    gfield(A, sq, 0)[(size_t)(i + 1) * (A.p + 1) + j + 1] = cf.f;
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= 4LL * A.H * A.H) return;
  const int64_t s = w >> 2;
  const int o = (int)(w & 3);
  const int a = (int)(s % A.H), c = (int)(s / A.H);
  const int p = A.p, N = p + 1, m = A.m, L = P.L;
  const bool vert = o >= 2;
  const int at = vert ? (o == 2 ? a * m : (a + 1) * m) : (o == 0 ? c * m : (c + 1) * m);
  const int lo = vert ? c * m : a * m, hi = lo + m;
  const double Sx = (P.x1 - P.x0) / A.H, Sy = (P.y1 - P.y0) / A.H;
  const double xa = P.x0 + a * Sx, ya = P.y0 + c * Sy;
  double* U = gfield(A, s, 0);
  const bool bnd = at == 0 || at == L;
  const int clo = max(0, lo - A.ext), chi = min(L, hi + A.ext);
  const double a0 = vert ? P.y0 : P.x0, d = vert ? P.dy : P.dx;
  double* v = sv + (size_t)(threadIdx.x >> 6) * 2 * smax;
  double* al = v + smax;
  const int S = chi - clo + 1;
  if (!bnd && A.rbf) {
    // alpha = Phi^{-1} v over the side's stencil
    for (int i = lane; i < S; i += 64) v[i] = lattice_value<KIND>(A, vert, at, clo + i);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const double* Mi = P.rbf_inv + (vert ? P.rbf_half : 0) + rbf_block_offset(S);
    for (int i = lane; i < S; i += 64) {
      double acc = 0.0;
      for (int j = 0; j < S; ++j) acc = fma(Mi[(size_t)j * S + i], v[j], acc);
      al[i] = acc;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  const int first = vert ? 1 : 0, last = vert ? p - 1 : p;
  for (int k = first + lane; k <= last; k += 64) {
    const double t = A.T.nodes[k];
    const double xk = vert ? (o == 2 ? xa : xa + Sx) : xa + Sx * (t + 1.0) * 0.5;
    const double yk = vert ? ya + Sy * (t + 1.0) * 0.5 : (o == 0 ? ya : ya + Sy);
    double val;
    if (bnd) {
      val = g_at<KIND>(xk, yk);
    } else {
      const double z = vert ? yk : xk;
      if (A.rbf) {
        double acc = 0.0;
        for (int q = 0; q < S; ++q) {
          const double r = z - (a0 + (double)(clo + q) * d);
          acc = fma(al[q], 1.0 / sqrt(fma(r, r, P.rbf_c2)), acc);
        }
        val = acc;
      } else {
        double tt = (z - a0) / d;
        tt = fmin(fmax(tt, (double)clo), (double)chi);
        const double i0 = fmin(floor(tt), (double)(chi - 1));
        const double wt = tt - i0;
        const int q0 = (int)i0;
        val = (1.0 - wt) * lattice_value<KIND>(A, vert, at, q0) + wt * lattice_value<KIND>(A, vert, at, q0 + 1);
      }
    }
    const int i = vert ? (o == 2 ? 0 : p) : k, j = vert ? k : (o == 0 ? 0 : p);
    U[(size_t)i * N + j] = val;
  }
}

// The 16 x 16 tile of C = A B (64 x 64 operands) that wave w of 16 owns: rows
// 16 (w / 4) .., columns 16 (w % 4) ...  Operands per lane l and K step:
// A[row0 + l % 16][k0 + l / 16] and B[k0 + l / 16][col0 + l % 16]; the float64
// accumulator holds element q of lane l at row row0 + l / 16 + 4 q, column
// col0 + l % 16.
constexpr int SOLVE_WAVES = 16;

struct Tile {
  int row0, col0, r, kq;
};
__device__ __forceinline__ Tile my_tile() {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  return Tile{16 * (w >> 2), 16 * (w & 3), lane & 15, lane >> 4};
}

// The lane's sixteen K-step values T[row0 + l % 16][4 s + l / 16] of a 64 x 64
// table: the A operand of T X, or the B operand of X T^T.  The tables are
// stored in this order (spec_frag), so a wave's loads are 512 contiguous
// bytes each; from row-major tables every load touched 16 lines.
__device__ __forceinline__ void load_frag(const double* __restrict__ T, int row0, double (&f)[16]) {
  const double* src = T + row0 * SPEC_T + (threadIdx.x & 63);
#pragma unroll
  for (int s = 0; s < 16; ++s) f[s] = src[64 * s];
}

// T X: the table's fragment from registers, X from LDS
__device__ __forceinline__ v4d tile_left(const double (&f)[16], const double* X, const Tile& t) {
  v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 16; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s], X[(4 * s + t.kq) * LDT + t.col0 + t.r], acc, 0, 0, 0);
  return acc;
}

// X T^T
__device__ __forceinline__ v4d tile_right(const double* X, const double (&f)[16], const Tile& t) {
  v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 16; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[(t.row0 + t.r) * LDT + 4 * s + t.kq], f[s], acc, 0, 0, 0);
  return acc;
}

template <class F>
__device__ __forceinline__ void tile_for_each(const v4d& acc, const Tile& t, F f) {
#pragma unroll
  for (int q = 0; q < 4; ++q) f(t.row0 + t.kq + 4 * q, t.col0 + t.r, acc[q]);
}

// Interior solve and grid derivatives of one square per workgroup.  Bound by
// latency (a partition has tens to a few hundred squares and each is a chain
// of six products), so sixteen waves share the 64 x 64 tiles, one 16 x 16
// tile per wave and product, and every product's table fragment is loaded
// while the previous product runs.  100 squares at p = 63 take 30 us (four
// waves with a 16-row strip each and the source evaluated here: 72 us; the
// same sixteen waves with row-major tables: 55 us).
__global__ __launch_bounds__(64 * SOLVE_WAVES) void k_spec_solve(SpecArgs A) {
  __shared__ double B[SPEC_T * LDT];
  const AsmParams& P = A.P;
  const int64_t s = blockIdx.x;
  const int p = A.p, N = p + 1, n = p - 1;
  const double Sx = (P.x1 - P.x0) / A.H, Sy = (P.y1 - P.y0) / A.H;
  double* U = gfield(A, s, 0);
  const double* D2b = A.T.D2b;
  const Tile t = my_tile();
  // F: source at the interior points minus the boundary columns of the operator
  for (int e = threadIdx.x; e < SPEC_T * SPEC_T; e += blockDim.x) {
    const int i = e / SPEC_T, j = e % SPEC_T;
    double f = 0.0;
    if (i < n && j < n) {
      f = U[(size_t)(i + 1) * N + j + 1] - A.ax * (D2b[2 * i] * U[(size_t)0 * N + j + 1] + D2b[2 * i + 1] * U[(size_t)p * N + j + 1]) -
          A.ay * (D2b[2 * j] * U[(size_t)(i + 1) * N] + D2b[2 * j + 1] * U[(size_t)(i + 1) * N + p]);
    }
    B[i * LDT + j] = f;
  }
  auto put = [&](const v4d& acc) __attribute__((always_inline)) {
    __syncthreads();                 // every wave has read the previous tile
    tile_for_each(acc, t, [&](int i, int j, double v) { B[i * LDT + j] = v; });
    __syncthreads();
  };
  double f0[16], f1[16];
  load_frag(A.T.Vinv, t.row0, f0);
  __syncthreads();
  v4d acc;
  // V^{-1} F
  load_frag(A.T.Vinv, t.col0, f1);
  acc = tile_left(f0, B, t);
  put(acc);
  // (V^{-1} F) V^{-T}, divided by ax lam_i + ay lam_j + c
  load_frag(A.T.V, t.row0, f0);
  acc = tile_right(B, f1, t);
  const double* lam = A.T.lam;
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = acc[q] / (A.ax * lam[t.row0 + t.kq + 4 * q] + A.ay * lam[t.col0 + t.r] + A.c);
  put(acc);
  // V (.)
  load_frag(A.T.V, t.col0, f1);
  acc = tile_left(f0, B, t);
  put(acc);
  // (.) V^T: the interior values
  load_frag(A.T.D, t.row0, f0);
  acc = tile_right(B, f1, t);
  load_frag(A.T.D, t.col0, f1);
  __syncthreads();
  // the whole grid into LDS (zero-padded): interior from the product, sides from global
  tile_for_each(acc, t, [&](int i, int j, double v) {
    if (i < n && j < n) {
      B[(i + 1) * LDT + j + 1] = v;
      U[(size_t)(i + 1) * N + j + 1] = v;
    }
  });
  for (int e = threadIdx.x; e < SPEC_T * SPEC_T; e += blockDim.x) {
    const int i = e / SPEC_T, j = e % SPEC_T;
    if (i >= N || j >= N) B[i * LDT + j] = 0.0;
    else if (i == 0 || i == p || j == 0 || j == p) B[i * LDT + j] = U[(size_t)i * N + j];
  }
  __syncthreads();
  const double sx = 2.0 / Sx, sy = 2.0 / Sy;
  double* Gx = gfield(A, s, 1);
  double* Gy = gfield(A, s, 2);
  // du/dx = (2/S) D U
  acc = tile_left(f0, B, t);
  tile_for_each(acc, t, [&](int i, int j, double v) {
    if (i < N && j < N) Gx[(size_t)i * N + j] = sx * v;
  });
  // du/dy = U ((2/S) D)^T
  acc = tile_right(B, f1, t);
  tile_for_each(acc, t, [&](int i, int j, double v) {
    if (i < N && j < N) Gy[(size_t)i * N + j] = sy * v;
  });
}

template <int KIND>
hipError_t launch_kind(const SpecArgs& A, hipStream_t stream) {
  const int64_t waves = 4LL * A.H * A.H;
  const int smax = min(A.m + 2 * A.ext, A.P.L) + 1;
  const size_t lds = (size_t)4 * 2 * smax * sizeof(double);
  const int64_t side_blocks = (waves + 3) / 4;
  const int64_t points = (int64_t)A.H * A.H * (A.p - 1) * (A.p - 1);
  hipLaunchKernelGGL((k_spec_sides<KIND>), dim3((unsigned)(side_blocks + (points + 255) / 256)), dim3(256), lds, stream,
                     A, smax, (int32_t)side_blocks);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_spec_solve, dim3((unsigned)(A.H * A.H)), dim3(64 * SOLVE_WAVES), 0, stream, A);
  return hipGetLastError();
}

// wave sum, every lane receiving it
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// barycentric basis value of node `lane` at reference coordinate z (exact at a node)
__device__ __forceinline__ double bary_basis(const double* nodes, const double* bw, int p, double z) {
  const int lane = threadIdx.x & 63;
  const bool mine = lane <= p;
  const double dz = mine ? z - nodes[lane] : 1.0;
  const uint64_t hit = __ballot(mine && dz == 0.0);
  if (hit) return (int)__builtin_ctzll(hit) == lane ? 1.0 : 0.0;
  const double r = mine ? bw[lane] / dz : 0.0;
  return r / wave_sum(r);
}

// Node `i` of n in [lo, hi]: its coordinate and its square of H (side S), as
// for any point (monotone in i, so a square owns a range of nodes).
__device__ __forceinline__ double node_at(double lo, double hi, int i, int n) {
  return lo + (hi - lo) * (double)i / (double)(n - 1);
}
__device__ __forceinline__ int square_of(double x, double lo, double S, int H) {
  return min(max((int)floor((x - lo) / S), 0), H - 1);
}

// One wave per point: 2-D barycentric interpolation of u, du/dx, du/dy on the
// point's square.  Points are either xy[2 n] (outputs u[n], grad[2 n], each
// nullable) or, with lut_n > 0, the lut_n^2 nodes of the domain's node grid
// (output grad_lut[(j lut_n + i) 2 + d] in float32).
__global__ __launch_bounds__(256) void k_spec_eval(SpecDev T, int32_t p, int32_t H, double x0, double x1, double y0,
                                                   double y1, const double* __restrict__ grid, int64_t n_pts,
                                                   const double* __restrict__ xy, int32_t lut_n, double* u,
                                                   double* grad, float* grad_lut) {
  __shared__ double lys[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int N = p + 1;
  const double Sx = (x1 - x0) / H, Sy = (y1 - y0) / H;
  for (int64_t q = (int64_t)blockIdx.x * 4 + wv; q < n_pts; q += (int64_t)gridDim.x * 4) {
    const double x = lut_n > 0 ? node_at(x0, x1, (int)(q % lut_n), lut_n) : xy[2 * q];
    const double y = lut_n > 0 ? node_at(y0, y1, (int)(q / lut_n), lut_n) : xy[2 * q + 1];
    const int a = square_of(x, x0, Sx, H), c = square_of(y, y0, Sy, H);
    const double zx = 2.0 * (x - (x0 + a * Sx)) / Sx - 1.0;
    const double zy = 2.0 * (y - (y0 + c * Sy)) / Sy - 1.0;
    const double lx = bary_basis(T.nodes, T.bw, p, zx);
    const double ly = bary_basis(T.nodes, T.bw, p, zy);
    lys[wv][lane] = ly;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const size_t sq = (size_t)(a + (int64_t)H * c) * 3 * N * N;
    double out[3];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      double r = 0.0;
      if (lane < N && lx != 0.0) {
        const double* row = grid + sq + (size_t)f * N * N + (size_t)lane * N;
        for (int j = 0; j < N; ++j) r = fma(lys[wv][j], row[j], r);
      }
      out[f] = wave_sum(lx * r);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) {
      if (u) u[q] = out[0];
      if (grad) {
        grad[2 * q] = out[1];
        grad[2 * q + 1] = out[2];
      }
      if (grad_lut) {
        grad_lut[2 * q] = (float)out[1];
        grad_lut[2 * q + 1] = (float)out[2];
      }
    }
  }
}

// ---- gradient table -----------------------------------------------------------
// The nodes of the table that fall in one square form a tensor grid there, so
// the interpolation of a field G on it is two matrix products,
//   out[j][i] = sum_l By[j][l] M[l][i],   M[l][i] = sum_k G[k][l] Bx[i][k],
// with the barycentric bases Bx, By of the square's x and y nodes, on the
// float64 matrix cores: 4 N^2 (1 + nodes / N) flops per node column instead of
// the 4 N^2 per node (and two divisions per basis value and node) of a sum
// per node.  One workgroup per 64 x 64 nodes of a square, a strip of 16 node
// columns i per wave; M never leaves the registers: its accumulators, rows
// l / 16 + 4 q of the K step (tile, q), are the second product's B operand
// with the contraction taken in that order.  A 1025^2 table over 100 squares
// at p = 63 takes 42 us (one wave and two 64-lane sums per node: 10.8 ms);
// what remains is the basis divisions and the last, partly filled tiles.  Tiles and
// K steps go up to the grid's size (p = 8, 65 nodes, 4 squares: 18.4 us at 64 grid
// points, now 7.4), and tables of few nodes keep k_spec_eval, see few_nodes.
constexpr int TAB = 64;             // nodes per workgroup and direction

// first node whose square is at least a (n for a = H)
__device__ __forceinline__ int first_node(double lo, double hi, double S, int H, int n, int a) {
  if (a <= 0) return 0;
  if (a >= H) return n;
  int g = (int)min((int64_t)n - 1, ((int64_t)a * (n - 1) + H - 1) / H);
  while (g > 0 && square_of(node_at(lo, hi, g - 1, n), lo, S, H) >= a) --g;
  while (g < n && square_of(node_at(lo, hi, g, n), lo, S, H) < a) ++g;
  return g;
}

// Barycentric basis of the reference coordinate z shared by the four lanes
// of equal l % 16: this lane's values at the grid points 4 s + l / 16.
// *hit: the grid point that z equals exactly (the basis is then that unit
// vector), or -1.
template <int K>
__device__ __forceinline__ void bary_frag(const SpecDev& T, int N, int kq, double z, double (&b)[K], int* hit) {
  int at = -1;
  double sum = 0.0;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const int k = 4 * s + kq;
    double r = 0.0;
    if (k < N) {
      const double dz = z - T.nodes[k];
      if (dz == 0.0) at = k;
      r = T.bw[k] / dz;
    }
    b[s] = r;
    sum += r;
  }
  at = max(at, __shfl_xor(at, 16, 64));
  at = max(at, __shfl_xor(at, 32, 64));
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
#pragma unroll
  for (int s = 0; s < K; ++s) b[s] = at >= 0 ? (4 * s + kq == at ? 1.0 : 0.0) : b[s] / sum;
  *hit = at;
}

// NT: sixteens of grid points per direction, (p + 16) / 16.
template <int NT>
__global__ __launch_bounds__(256) void k_spec_table(SpecDev T, int32_t p, int32_t H, double x0, double x1, double y0,
                                                    double y1, const double* __restrict__ grid, int32_t lut_n,
                                                    int32_t tiles, float* __restrict__ out) {
  __shared__ double By[TAB * LDT];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int N = p + 1;
  const double Sx = (x1 - x0) / H, Sy = (y1 - y0) / H;
  int64_t blk = blockIdx.x;
  const int ti = (int)(blk % tiles);
  blk /= tiles;
  const int tj = (int)(blk % tiles);
  blk /= tiles;
  const int a = (int)(blk % H), c = (int)(blk / H);
  const int i0 = first_node(x0, x1, Sx, H, lut_n, a) + TAB * ti;
  const int j0 = first_node(y0, y1, Sy, H, lut_n, c) + TAB * tj;
  const int ni = min(TAB, first_node(x0, x1, Sx, H, lut_n, a + 1) - i0);
  const int nj = min(TAB, first_node(y0, y1, Sy, H, lut_n, c + 1) - j0);
  if (ni <= 0 || nj <= 0) return;                  // uniform: an edge tile that holds no node
  constexpr int K = 4 * NT;                        // K steps of four grid points
  double b[K];
  int hit;
  // the strip w of the y nodes, into LDS
  if (16 * w < nj) {
    const double y = node_at(y0, y1, j0 + min(16 * w + r, nj - 1), lut_n);
    bary_frag(T, N, kq, 2.0 * (y - (y0 + c * Sy)) / Sy - 1.0, b, &hit);
#pragma unroll
    for (int s = 0; s < K; ++s) By[(16 * w + r) * LDT + 4 * s + kq] = b[s];
  }
  __syncthreads();
  if (16 * w >= ni) return;                        // no barrier follows
  const int i = i0 + min(16 * w + r, ni - 1);
  bary_frag(T, N, kq, 2.0 * (node_at(x0, x1, i, lut_n) - (x0 + a * Sx)) / Sx - 1.0, b, &hit);
  v4d o[2][4];
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    const double* G = grid + ((size_t)(a + (int64_t)H * c) * 3 + 1 + d) * (size_t)N * N;
    v4d M[NT];
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      M[rt] = v4d{0.0, 0.0, 0.0, 0.0};
      const int l = 16 * rt + r;
      double g[K];
#pragma unroll
      for (int s = 0; s < K; ++s) g[s] = (l < N && 4 * s + kq < N) ? G[(size_t)(4 * s + kq) * N + l] : 0.0;
#pragma unroll
      for (int s = 0; s < K; ++s) M[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[s], b[s], M[rt], 0, 0, 0);
    }
    // a node on a grid column takes that column's values alone
    if (hit >= 0) {
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int l = 16 * rt + kq + 4 * q;
          M[rt][q] = l < N ? G[(size_t)hit * N + l] : 0.0;
        }
    }
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) {
      o[d][jt] = v4d{0.0, 0.0, 0.0, 0.0};
      if (16 * jt < nj) {
#pragma unroll
        for (int rt = 0; rt < NT; ++rt)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            o[d][jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(By[(16 * jt + r) * LDT + 16 * rt + 4 * q + kq], M[rt][q],
                                                            o[d][jt], 0, 0, 0);
      }
    }
  }
  if (16 * w + r < ni) {
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int jl = 16 * jt + kq + 4 * q;
        if (jl < nj) {
          float* to = out + 2 * ((size_t)(j0 + jl) * lut_n + i);
          to[0] = (float)o[0][jt][q];
          to[1] = (float)o[1][jt][q];
        }
      }
  }
}

// Range of the fields 0..5 (sxx, sxy, syy, dx, dy, c) of a LUT: per-block
// minima and maxima, then one block combines them into out[12] (min, max).
constexpr int RANGE_BLOCKS = 1024;
__global__ __launch_bounds__(256) void k_lut_range_part(const float* __restrict__ lut, int64_t nodes,
                                                        double* __restrict__ part) {
  __shared__ double red[256][12];
  double mn[6], mx[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    mn[q] = INFINITY;
    mx[q] = -INFINITY;
  }
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nodes; i += (int64_t)gridDim.x * 256) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const double v = lut[(size_t)i * PDD_LUT_STRIDE + q];
      mn[q] = fmin(mn[q], v);
      mx[q] = fmax(mx[q], v);
    }
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    red[threadIdx.x][q] = mn[q];
    red[threadIdx.x][6 + q] = mx[q];
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    const int q = threadIdx.x;
    double v = red[0][q];
    for (int t = 1; t < 256; ++t) v = q < 6 ? fmin(v, red[t][q]) : fmax(v, red[t][q]);
    part[(size_t)blockIdx.x * 12 + q] = v;
  }
}

__global__ void k_lut_range_final(const double* __restrict__ part, int blocks, double* __restrict__ out) {
  if (threadIdx.x < 12) {
    const int q = threadIdx.x;
    double v = part[q];
    for (int b = 1; b < blocks; ++b) v = q < 6 ? fmin(v, part[(size_t)b * 12 + q]) : fmax(v, part[(size_t)b * 12 + q]);
    out[q] = v;
  }
}

}  // namespace

hipError_t launch_spectral_solve(const SpecArgs& A, hipStream_t stream) {
  switch (A.P.coef.kind) {
    case PDD_COEF_POISSON: return launch_kind<PDD_COEF_POISSON>(A, stream);
    case PDD_COEF_EXITTIME: return launch_kind<PDD_COEF_EXITTIME>(A, stream);
    case PDD_COEF_EQ43: return launch_kind<PDD_COEF_EQ43>(A, stream);
    case PDD_COEF_LUT: return launch_kind<PDD_COEF_LUT>(A, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_spectral_eval(const SpecDev& T, int32_t p, int32_t H, double x0, double x1, double y0, double y1,
                                const double* grid, int64_t n_pts, const double* xy, double* u, double* grad,
                                hipStream_t stream) {
  const unsigned blocks = (unsigned)std::min<int64_t>((n_pts + 3) / 4, 65536);
  hipLaunchKernelGGL(k_spec_eval, dim3(std::max(blocks, 1u)), dim3(256), 0, stream, T, p, H, x0, x1, y0, y1, grid, n_pts,
                     xy, 0, u, grad, nullptr);
  return hipGetLastError();
}

// A wave per node, all resident at once, against a chain of bases and two products
// in a workgroup per square, of which some thousand run at once.  us, node by node
// and by squares: 17^2 nodes 6.2 and 7.7 (p = 3, 64 squares), 6.2 and 11.2 (p = 31);
// 65^2 7.7 and 8.2 (p = 8, 64), 9.4 and 10.5 (p = 16, 16), 14.6 and 15.0 (p = 32, 256), 6.8
// and 39 (p = 8, 4096); 101^2 11.7 and 7.4 (p = 2, 4), 12.8 and 40 (p = 8, 4096); 200^2
// 35 and 39 (p = 2, 4096).
bool few_nodes(int32_t p, int32_t H, int64_t lut_n) { return lut_n * lut_n * (p + 9) < 65536 + (int64_t)128 * H * H; }

hipError_t launch_spectral_table(const SpecDev& T, int32_t p, int32_t H, double x0, double x1, double y0, double y1,
                                 const double* grid, int32_t lut_n, float* grad_lut, hipStream_t stream) {
  if (few_nodes(p, H, lut_n)) {
    const int64_t nodes = (int64_t)lut_n * lut_n;
    hipLaunchKernelGGL(k_spec_eval, dim3((unsigned)std::min<int64_t>((nodes + 3) / 4, 65536)), dim3(256), 0, stream, T, p,
                       H, x0, x1, y0, y1, grid, nodes, nullptr, lut_n, nullptr, nullptr, grad_lut);
    return hipGetLastError();
  }
  // a square holds at most (lut_n - 1) / H + 2 nodes per direction
  const int64_t tiles = ((lut_n - 1) / H + 2 + TAB - 1) / TAB;
  const int64_t blocks = (int64_t)H * H * tiles * tiles;
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream, T, p, H, x0, x1, y0, y1, grid, lut_n,
                       (int32_t)tiles, grad_lut);
    return hipGetLastError();
  };
  switch ((p + 16) / 16) {
    case 1: return launch(k_spec_table<1>);
    case 2: return launch(k_spec_table<2>);
    case 3: return launch(k_spec_table<3>);
    default: return launch(k_spec_table<4>);
  }
}

hipError_t launch_lut_field_range(const float* lut, int64_t nodes, double* out, hipStream_t stream) {
  // out[0..11] = min, max of fields 0..5; out + 12 holds RANGE_BLOCKS * 12 partials
  double* part = out + 12;
  hipLaunchKernelGGL(k_lut_range_part, dim3(RANGE_BLOCKS), dim3(256), 0, stream, lut, nodes, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lut_range_final, dim3(1), dim3(64), 0, stream, part, RANGE_BLOCKS, out);
  return hipGetLastError();
}

}  // namespace pdd
