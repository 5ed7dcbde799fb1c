// Section 6: the right preconditioner of Algorithm 11 built from the
// sketch's factor, and LSQR on the preconditioned operator A N.
//
// Preconditioner.  The sketch A~ = G S A is factored as A~ P = Q R by the
// rank-revealing step; then
//   QR:  N = P R11^{-1}                       (columns past the rank zero);
//   SVD: N = P V_R Sigma^{-1}, R = U_R Sigma V_R^T the SVD of R, which is the
//        V Sigma^{-1} of the SVD of A~ itself (A~ = (Q U_R) Sigma (P V_R)^T),
//        keeping the k singular values above zeta sigma_1.
// The SVD of R (d <= 128) is the preconditioned one-sided Jacobi method of
// Drmac and Veselic (2008): Hestenes' iteration on W = R^T, whose columns
// are the rows of the pivoted factor and so are already close to
// orthogonal (few sweeps).  W sits in LDS; each round of a round-robin
// ordering orthogonalises all its disjoint column pairs at once (a 16-lane
// group per pair, Rutishauser's rotation), and sweeps repeat until no pair
// is rotated.  Then W = R^T U_R = V_R Sigma: the column norms are the
// singular values and column c over its norm is the right singular vector,
// so N = P W Sigma^{-2} without accumulating the rotations.  Relative
// accuracy of the singular values does not depend on kappa(R).
//
// LSQR (Paige and Saunders 1982) on M = A N from y = 0, with x = N y at the
// end.  Per iteration two passes over A (dense, FP64 arithmetic on any
// storage type) and one single-workgroup kernel:
//   gemv:  t = A (N v) - alpha u, and per-workgroup sums of t_i^2;
//   atv:   beta = sqrt(sum), u = t / beta, per-workgroup partials of A^T u;
//   step:  q = N^T (A^T u) - beta v, alpha = ||q||, v = q / alpha, the
//          rotation (rho, c, s, theta, phi), y += (phi / rho) w,
//          w = v - (theta / rho) w, z = N v for the next gemv.
// Scalars stay in device memory; all sums run in a fixed order.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lev_internal.h"

namespace lev {
namespace {

constexpr int kSvdGroup = 16;           // lanes per column pair
constexpr int kSvdMaxThreads = 1024;    // 64 groups: every pair of a round at d <= 128
constexpr int kMaxSweeps = 40;
// stride of a column of W in LDS: 16 ELEMS elements and the banks' offset
__host__ __device__ constexpr int svd_stride(int elems) { return kSvdGroup * elems + 16; }

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Round-robin pairing of dd (even) columns: in round t pair q joins the
// columns at positions q and dd - 1 - q of the ring, where position 0
// holds column 0 for good and position i > 0 holds column
// 1 + (i - 1 + t) mod (dd - 1); so from one round to the next every
// column but 0 moves to the next of 1 .. dd - 1, cyclically.
__device__ __forceinline__ int rr_col(int dd, int t, int i) { return i == 0 ? 0 : 1 + (i - 1 + t) % (dd - 1); }
__device__ __forceinline__ int rr_next(int dd, int c) { return c == 0 ? 0 : (c + 1 == dd ? 1 : c + 1); }

// v + v of the DPP partner lane (both 32-bit halves moved).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
  return v + __hiloint2double(hi, lo);
}

// Sum over each 16-lane row by butterflies whose partners always sit in
// the other half of the part summed so far, so both sides add the same two
// values and every lane of the row ends with identical bits (the rotation
// is then the same in every lane).  All 16 lanes must be active.
__device__ __forceinline__ double row16_sum(double v) {
  v = dpp_add<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v = dpp_add<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v = dpp_add<0x141>(v);  // row_half_mirror
  v = dpp_add<0x140>(v);  // row_mirror
  return v;
}

// One workgroup of 16 * (dd / 2) lanes (rounded up to a wave); LDS holds W
// column-major, dd columns (a zero column pads an odd d) of 16 ELEMS elements,
// zero past d, at a stride of 16 more (so that columns next to each other
// start in opposite halves of the banks).  ELEMS = 4 (d <= 64) or 8: the loads
// of a round need no bound.
// Bound by the chain of one round (LDS read, three dot products and their
// reductions, the rotation's divisions and roots, LDS write, barrier), which
// is repeated dd - 1 times a sweep.  d = 60: 344 us, against 491 with a bound
// and a select on every load.  (Eight lanes a pair and an angle without a
// division took 252, but round otherwise, and an unconverged LSQR iterate
// passes a change of N's last bits on to 1e-9.)
template <int ELEMS>
__global__ __launch_bounds__(kSvdMaxThreads) void jacobi_svd_kernel(int64_t d, const double* __restrict__ R,
                                                                    const int64_t* __restrict__ rank,
                                                                    const int32_t* __restrict__ perm, double zeta,
                                                                    double* __restrict__ N,
                                                                    int64_t* __restrict__ k_out) {
  extern __shared__ double W[];
  __shared__ int rotated;
  __shared__ double sig[128];
  __shared__ int order[128];
  const int di = (int)d;
  const int dd = di + (di & 1);
  constexpr int kRows = kSvdGroup * ELEMS, kStride = svd_stride(ELEMS);
  const int64_t r = *rank;
  // W = R^T: column c of W is row c of R (rows past the rank are zero)
  for (int e = threadIdx.x; e < dd * kRows; e += blockDim.x) {
    const int c = e / kRows, i = e % kRows;
    W[c * kStride + i] = (c < r && i < di) ? R[(int64_t)c * d + i] : 0.0;
  }
  __syncthreads();
  const int gl = threadIdx.x & (kSvdGroup - 1);
  const int q = threadIdx.x / kSvdGroup;
  const bool active = q < dd / 2;  // whole 16-lane rows are active or not
  // a pair is rotated while |x . y| > tol ||x|| ||y||, tested squared
  const double tol = 4.0 * (double)di * 2.220446049250313e-16;
  const double tol2 = tol * tol;
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    if (threadIdx.x == 0) rotated = 0;
    __syncthreads();
    int a = rr_col(dd, 0, q), b = rr_col(dd, 0, dd - 1 - q);
    for (int t = 0; t < dd - 1; ++t, a = rr_next(dd, a), b = rr_next(dd, b)) {
      if (active) {
        double* wa = W + a * kStride + gl;
        double* wb = W + b * kStride + gl;
        double x[ELEMS], y[ELEMS];
        double al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
        for (int j = 0; j < ELEMS; ++j) {
          x[j] = wa[kSvdGroup * j];
          y[j] = wb[kSvdGroup * j];
        }
#pragma unroll
        for (int j = 0; j < ELEMS; ++j) {
          al = fma(x[j], x[j], al);
          be = fma(y[j], y[j], be);
          ga = fma(x[j], y[j], ga);
        }
        al = row16_sum(al);
        be = row16_sum(be);
        ga = row16_sum(ga);
        if (ga != 0.0 && ga * ga > tol2 * (al * be)) {
          const double zt = (be - al) / (2.0 * ga);
          const double tn = (zt >= 0.0 ? 1.0 : -1.0) / (fabs(zt) + sqrt(1.0 + zt * zt));
          const double c = rsqrt(1.0 + tn * tn), s = c * tn;  // 1 + tn^2 in [1, 2]
#pragma unroll
          for (int j = 0; j < ELEMS; ++j) {
            wa[kSvdGroup * j] = c * x[j] - s * y[j];
            wb[kSvdGroup * j] = s * x[j] + c * y[j];
          }
          if (gl == 0) rotated = 1;
        }
      }
      __syncthreads();
    }
    const int any = rotated;
    __syncthreads();
    if (!any) break;
  }
  // singular values, their descending order (ties: lower column first), k
  for (int c = threadIdx.x; c < di; c += blockDim.x) {
    double nn = 0.0;
    for (int i = 0; i < di; ++i) nn = fma(W[c * kStride + i], W[c * kStride + i], nn);
    sig[c] = sqrt(nn);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < di; c += blockDim.x) {
    int rk = 0;
    for (int c2 = 0; c2 < di; ++c2) rk += (sig[c2] > sig[c] || (sig[c2] == sig[c] && c2 < c)) ? 1 : 0;
    order[rk] = c;
  }
  __syncthreads();
  const double s1 = sig[order[0]];
  int k = 0;
  for (int c = 0; c < di; ++c) k += (s1 > 0.0 && sig[order[c]] > zeta * s1) ? 1 : 0;
  // N[perm[i]][c] = V_R[i][order[c]] / sigma = W[i][order[c]] / sigma^2
  for (int e = threadIdx.x; e < di * di; e += blockDim.x) {
    const int i = e / di, c = e - i * di;
    double v = 0.0;
    if (c < k) {
      const int o = order[c];
      v = W[o * kStride + i] / sig[o] / sig[o];
    }
    N[(int64_t)perm[i] * d + c] = v;
  }
  if (threadIdx.x == 0) *k_out = k;
}

// N[perm[j]][q] = Z[j][q] (Z = R11^{-1} with zero rows past the rank).
__global__ void scatter_rows_kernel(int64_t d, const int32_t* __restrict__ perm, const double* __restrict__ Z,
                                    double* __restrict__ N, const int64_t* __restrict__ rank,
                                    int64_t* __restrict__ k_out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e == 0) *k_out = *rank;
  if (e >= d * d) return;
  const int64_t j = e / d, q = e % d;
  N[(int64_t)perm[j] * d + q] = Z[e];
}

// ---- LSQR -------------------------------------------------------------------------
// st: [0] alpha, [1] beta, [2] rhobar, [3] phibar, [4] stop (0 / 1), [5] beta_1
constexpr int kGemvThreads = 1024;

__device__ __forceinline__ double f64(double x) { return x; }
__device__ __forceinline__ double f64(float x) { return (double)x; }
__device__ __forceinline__ double f64(__hip_bfloat16 x) { return (double)__bfloat162float(x); }

// Four consecutive elements of a row from column c (c a multiple of 4,
// c < d), widened to FP64; elements at or past d read as zero.  Rows are
// 16-byte aligned with ld * sizeof(T) a multiple of 16, so a vector whose
// first element is below d stays inside the row (FP64: a second 16-byte half
// past d reads the first one again, so no load sits under a branch).
__device__ __forceinline__ void load4(const float* p, int64_t c, int64_t d, double (&a)[4]) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  a[0] = v.x;
  a[1] = c + 1 < d ? (double)v.y : 0.0;
  a[2] = c + 2 < d ? (double)v.z : 0.0;
  a[3] = c + 3 < d ? (double)v.w : 0.0;
}
__device__ __forceinline__ void load4(const double* p, int64_t c, int64_t d, double (&a)[4]) {
  const double2 lo = *reinterpret_cast<const double2*>(p);
  const double2 hi = *reinterpret_cast<const double2*>(p + (c + 2 < d ? 2 : 0));
  a[0] = lo.x;
  a[1] = c + 1 < d ? lo.y : 0.0;
  a[2] = c + 2 < d ? hi.x : 0.0;
  a[3] = c + 3 < d ? hi.y : 0.0;
}
__device__ __forceinline__ void load4(const __hip_bfloat16* p, int64_t c, int64_t d, double (&a)[4]) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  a[0] = (double)__uint_as_float(v.x << 16);
  a[1] = c + 1 < d ? (double)__uint_as_float(v.x & 0xFFFF0000u) : 0.0;
  a[2] = c + 2 < d ? (double)__uint_as_float(v.y << 16) : 0.0;
  a[3] = c + 3 < d ? (double)__uint_as_float(v.y & 0xFFFF0000u) : 0.0;
}

// LSQR before convergence passes a change of rounding on: an iterate moves by
// 1e-9 to 1e-8 (relative) when one sum of a step is taken in another order,
// while the residuals agree to 1e-15.  So every sum below keeps one fixed
// order whatever the number of threads: t_i by 16 lanes, the squares by 16
// chains of a workgroup's rows, A^T u by four chains a workgroup, the
// workgroups' partials and N^T by eight.

// Sum over the 16 lanes of a row in the order of a xor butterfly 8, 4, 2, 1
// (after each step the values repeat with that period, so a rotation by it
// brings the same partner).
__device__ __forceinline__ double ror16_sum(double v) {
  v = dpp_add<0x128>(v);  // row_ror:8
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}

// t_i = A[i,:] z - alpha u_i (or b_i when init), partial[g] = sum of t_i^2
// over the workgroup's rows.  A 16-lane group takes a row: lane l reads
// elements 64 m + 4 l .. + 3 (one vector load per 64 columns), against z in
// registers (M blocks of 64 columns; M = 0: any width, z in LDS).  256 rows at
// a time: the 64 groups of 1024 lanes leave their t_i in LDS, from which 16
// lanes of the first wave carry the 16 chains of squares (chain s takes the
// rows s, s + 16, ..) while the others go on.
// Bound by the latency of one row's chain and the launch when A fits the
// caches (50000 x 60 FP64, 196 workgroups: 6.4
// us; 13 with 256 lanes, two rows a group in flight and z read from LDS), by HBM beyond.
constexpr int kGemvGroup = 16;
constexpr int kGemvRows = 256;
template <typename T, int M>
__global__ __launch_bounds__(kGemvThreads) void lsqr_gemv_kernel(const T* __restrict__ A, int64_t n, int64_t d,
                                                                 int64_t ld, const double* __restrict__ z,
                                                                 const double* __restrict__ u,
                                                                 const double* __restrict__ b, int init,
                                                                 const double* __restrict__ st,
                                                                 double* __restrict__ t, double* __restrict__ partial) {
  constexpr int kSlots = kGemvThreads / kGemvGroup;
  constexpr int kIn = M == 1 ? 4 : M == 2 ? 2 : 1;  // rows in flight per group
  __shared__ double tb[2][kGemvRows];
  __shared__ __align__(16) double zs[M == 0 ? 1024 + 4 : 4];
  if (!init && st[4] != 0.0) return;
  const double alpha = init ? 0.0 : st[0];
  const double* src = init ? b : u;
  const int gl = threadIdx.x % kGemvGroup, slot = threadIdx.x / kGemvGroup;
  const int64_t rows_per_group = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_group, r1 = std::min<int64_t>(n, r0 + rows_per_group);
  double zc[M == 0 ? 1 : M][4];
  if constexpr (M == 0) {
    if (!init)
      for (int64_t c = threadIdx.x; c < d; c += kGemvThreads) zs[c] = z[c];
    __syncthreads();
  } else {
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t c = 64 * m + 4 * gl + e;
        zc[m][e] = !init && c < d ? z[c] : 0.0;
      }
  }
  double sq = 0.0;  // lanes 0 .. 15 of the first wave
  int buf = 0;
  for (int64_t i0 = r0; i0 < r1; i0 += kGemvRows, buf ^= 1) {
    for (int k0 = 0; k0 < kGemvRows / kSlots; k0 += kIn) {
      double dot[kIn], uv[kIn];
#pragma unroll
      for (int q = 0; q < kIn; ++q) uv[q] = src[std::min<int64_t>(i0 + slot + kSlots * (k0 + q), r1 - 1)];
      if (!init) {
        if constexpr (M == 0) {
          const int64_t i = std::min<int64_t>(i0 + slot + kSlots * k0, r1 - 1);
          double acc = 0.0;
          for (int64_t c = 4 * gl; c < d; c += 64) {
            double a[4];
            load4(A + i * ld + c, c, d, a);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = fma(a[e], c + e < d ? zs[c + e] : 0.0, acc);
          }
          dot[0] = acc;
        } else {
          double a[kIn][M][4];
#pragma unroll
          for (int q = 0; q < kIn; ++q) {
            const int64_t i = std::min<int64_t>(i0 + slot + kSlots * (k0 + q), r1 - 1);
#pragma unroll
            for (int m = 0; m < M; ++m) {
              // lanes past d read column 0 and take zeros
              const int64_t c = 64 * m + 4 * gl;
              load4(A + i * ld + (c < d ? c : 0), c, d, a[q][m]);
              a[q][m][0] = c < d ? a[q][m][0] : 0.0;
            }
          }
#pragma unroll
          for (int q = 0; q < kIn; ++q) {
            double acc = 0.0;
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc = fma(a[q][m][e], zc[m][e], acc);
            dot[q] = acc;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < kIn; ++q) {
        const int r = slot + kSlots * (k0 + q);
        const double ti = init ? uv[q] : fma(-alpha, uv[q], ror16_sum(dot[q]));
        if (gl == 0 && i0 + r < r1) {
          t[i0 + r] = ti;
          tb[buf][r] = ti;
        }
      }
    }
    __syncthreads();  // (the other half of tb was read before it)
    if (threadIdx.x < 16) {
#pragma unroll
      for (int k = 0; k < kGemvRows / 16; ++k) {
        const int r = threadIdx.x + 16 * k;
        const double ti = tb[buf][r];
        sq = i0 + r < r1 ? fma(ti, ti, sq) : sq;
      }
    }
  }
  if (threadIdx.x < 16) {
    sq = dpp_add<0x4E>(sq);  // chains s and s + 2 of each four, then the two sums
    sq = dpp_add<0xB1>(sq);
    double s = __shfl(sq, 0, 16);
    for (int w = 1; w < 4; ++w) s += __shfl(sq, 4 * w, 16);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
  }
}

// V consecutive elements of a row, widened (V = 4: load4).
template <typename T, int V>
__device__ __forceinline__ void load_cols(const T* p, int64_t c, int64_t d, double (&a)[V]) {
  if constexpr (V == 4) {
    load4(p, c, d, a);
  } else if constexpr (V == 1) {
    a[0] = f64(p[0]);
  } else if constexpr (sizeof(T) == 8) {
    const double2 v = *reinterpret_cast<const double2*>(p);
    a[0] = v.x;
    a[1] = v.y;
  } else if constexpr (sizeof(T) == 4) {
    const float2 v = *reinterpret_cast<const float2*>(p);
    a[0] = v.x;
    a[1] = v.y;
  } else {
    const uint32_t v = *reinterpret_cast<const uint32_t*>(p);
    a[0] = (double)__uint_as_float(v << 16);
    a[1] = (double)__uint_as_float(v & 0xFFFF0000u);
  }
}

// beta = sqrt(sum of the gemv partials); u = t / beta; partial_g[c] = sum over
// the workgroup's rows of u_i A[i][c].  Wave w's chain takes every fourth row;
// lane l takes columns V l .. V l + V - 1 of a slice of 64 V, the narrowest of
// V = 1, 2, 4 that holds d (V = 4: slice after slice), so all lanes work; the
// waves' sums are added in LDS in wave order.  u of 256 rows at a time is
// staged in LDS; kAtvIn rows load together, the next ones while these are
// added, the first ones before beta is known.
// Bound like the product with A, and by the sum of the gemv's partials before
// it (50000 x 60 FP64: 9.3 us; 24 when a lane took four columns at any width,
// 15 of 64 lanes at d = 60, and waited for beta and for each eight rows).
constexpr int kAtvThreads = 256;
template <typename T, int V>
__global__ __launch_bounds__(kAtvThreads) void lsqr_atv_kernel(const T* __restrict__ A, int64_t n, int64_t d,
                                                               int64_t ld, const double* __restrict__ t,
                                                               const double* __restrict__ gpart, int ggroups,
                                                               double* __restrict__ st, int init,
                                                               double* __restrict__ u, double* __restrict__ partial) {
  constexpr int kW = kAtvThreads / 64, kCols = 64 * V, kAtvIn = V == 1 ? 16 : V == 2 ? 8 : 4;
  constexpr int kBatch = kW * kAtvIn;  // rows of a batch over the waves
  __shared__ double red[kW][kCols];
  __shared__ __align__(16) double gs[1024];
  __shared__ double ub[kAtvThreads];
  const int64_t rows_per_group = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_group, r1 = std::min<int64_t>(n, r0 + rows_per_group);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double a[2][kAtvIn][V];
  // the batch of rows from i (this wave: i + wave, + 4, ..), clamped to the
  // last row; lanes past d read column 0 and are dropped
  auto load = [&](auto set, int64_t i, int64_t cl) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int q = 0; q < kAtvIn; ++q)
      load_cols<T, V>(A + std::min<int64_t>(i + wave + kW * q, r1 - 1) * ld + cl, cl, d, a[S][q]);
  };
  const std::integral_constant<int, 0> s0;
  const std::integral_constant<int, 1> s1;
  const int64_t cl0 = V * lane < d ? V * lane : 0;
  if (r0 < r1) load(s0, r0, cl0);  // (does not wait for beta)
  for (int g = threadIdx.x; g < 1024; g += kAtvThreads) gs[g] = g < ggroups ? gpart[g] : 0.0;
  if (!init && st[4] != 0.0) return;
  __syncthreads();
  double s = 0.0;
  for (int g0 = 0; g0 < ggroups; g0 += 32) {
    double2 v[16];  // (sums of squares from g0 on, zero past the last: it changes no bit)
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = *reinterpret_cast<const double2*>(gs + g0 + 2 * q);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      s += v[q].x;
      s += v[q].y;
    }
  }
  const double beta = sqrt(s);
  const double inv = beta > 0.0 ? 1.0 / beta : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st[1] = beta;
    if (init) {
      st[5] = beta;
      st[3] = beta;  // phibar = beta_1
    }
  }
  for (int64_t c0 = 0; c0 < d; c0 += kCols) {
    const int64_t cl = c0 + V * lane < d ? c0 + V * lane : 0;
    double acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.0;
    auto use = [&](auto set, int64_t i0, int k0) {
      constexpr int S = decltype(set)::value;
      double ui[kAtvIn];
#pragma unroll
      for (int q = 0; q < kAtvIn; ++q) ui[q] = ub[k0 + wave + kW * q];
#pragma unroll
      for (int q = 0; q < kAtvIn; ++q)
        if (i0 + k0 + wave + kW * q < r1) {  // uniform
#pragma unroll
          for (int e = 0; e < V; ++e) acc[e] = fma(ui[q], a[S][q][e], acc[e]);
        }
    };
    if (c0 > 0 && r0 < r1) load(s0, r0, cl);
    for (int64_t i0 = r0; i0 < r1; i0 += kAtvThreads) {
      __syncthreads();  // the previous rows' u (and the previous slice's sums) have been read
      const int64_t iu = i0 + threadIdx.x;
      if (iu < r1) {
        const double ui = t[iu] * inv;
        ub[threadIdx.x] = ui;
        if (c0 == 0) u[iu] = ui;
      }
      __syncthreads();
      for (int k0 = 0; k0 < kAtvThreads; k0 += 2 * kBatch) {
        if (i0 + k0 + kBatch >= r1) {
          use(s0, i0, k0);
          break;
        }
        load(s1, i0 + k0 + kBatch, cl);
        use(s0, i0, k0);
        if (i0 + k0 + 2 * kBatch >= r1) {
          use(s1, i0, k0 + kBatch);
          break;
        }
        load(s0, i0 + k0 + 2 * kBatch, cl);
        use(s1, i0, k0 + kBatch);
      }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) red[wave][V * lane + e] = acc[e];
    __syncthreads();
    const int64_t cc = c0 + threadIdx.x;
    if (threadIdx.x < kCols && cc < d) {
      double v = red[0][threadIdx.x];
#pragma unroll
      for (int w = 1; w < kW; ++w) v += red[w][threadIdx.x];
      partial[(int64_t)blockIdx.x * d + cc] = v;
    }
    __syncthreads();
  }
}

// One LSQR step after the two passes (init: the first alpha, v, w).  C: the
// power of two from 64 that holds d.  Every sum runs in eight chains (term j
// in chain j mod 8, the last j < 8 terms past the whole eights in chain 0)
// that are added in order; thread (c, p) carries 8 / P of column c's chains,
// so the whole workgroup loads, and for C <= 128 it holds its pieces of N in
// registers, fetched before the sums that they wait for.  z = N v takes a
// 16-lane group per row there, a wave per row beyond.
//
// One workgroup: bound by the latency of its chain (partials, N^T, alpha, v,
// z).  The square roots and divisions are long FP64 sequences, so the last
// wave alone takes the rotation and the columns' own waves alpha; run by all
// sixteen waves they filled the SIMDs.
// d = 60, 196 partials: 6.0 us (15.7 with one thread a column).  Beyond 256
// columns N is read twice, 2 d^2 doubles by one workgroup, and what counts is
// how many of its loads are in flight: d = 400, 600 and 1000: 70, 140 and 275 us
// (97, 220 and 590 with a load's address and wait in every turn of the loops).
template <int C>
__global__ __launch_bounds__(C == 64 ? 512 : 1024) void lsqr_step_kernel(
    int64_t d, const double* __restrict__ N, const double* __restrict__ partial, int groups, double* __restrict__ st,
    double* __restrict__ v, double* __restrict__ w, double* __restrict__ y, double* __restrict__ z,
    double* __restrict__ hist, int64_t it, int init) {
#pragma clang fp contract(off)  // (a product that ends a chain must not join the sum over the chains)
  constexpr int kThreads = C == 64 ? 512 : 1024, kWaves = kThreads / 64;
  constexpr int P = kThreads / C, kU = 8 / P;     // parts, chains of a thread
  constexpr bool kHold = C <= 128;
  constexpr int kE = kHold ? C / 8 : 1, kZ = kHold ? C / 16 : 1, kZr = kHold ? C / (kThreads / 16) : 1;
  __shared__ double g[C];
  __shared__ double part[8][C];
  __shared__ double red[C / 64];
  __shared__ double sc[4];  // phi / rho, sin, cos, rho
  const int di = (int)d;
  const int c = threadIdx.x & (C - 1);
  const int p = __builtin_amdgcn_readfirstlane(threadIdx.x / C);  // (C is whole waves: rows of N and partials are uniform)
  const int cl = c < di ? c : 0;  // columns past d load column 0 and are dropped
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool own = p == 0 && c < di;
  const int gl = threadIdx.x & 15, gr = threadIdx.x >> 4;
  // the partials' chains, sixteen loads in flight
  const int whole = groups / 8;
  double sp[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) sp[u] = 0.0;
  constexpr int kIn = 16 / kU;
  for (int k0 = 0; k0 < whole; k0 += kIn) {
    double a[kIn][kU];
#pragma unroll
    for (int q = 0; q < kIn; ++q)
#pragma unroll
      for (int u = 0; u < kU; ++u)
        a[q][u] = partial[(int64_t)(8 * std::min(k0 + q, whole - 1) + p * kU + u) * d + cl];
#pragma unroll
    for (int q = 0; q < kIn; ++q)
      if (k0 + q < whole) {  // uniform
#pragma unroll
        for (int u = 0; u < kU; ++u) sp[u] += a[q][u];
      }
  }
  if (p == 0) {
    double a[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) a[q] = partial[(int64_t)std::min(8 * whole + q, groups - 1) * d + cl];
#pragma unroll
    for (int q = 0; q < 7; ++q)
      if (8 * whole + q < groups) sp[0] += a[q];
  }
  const double stop = init ? 0.0 : st[4], beta = st[1], rhobar = st[2], phibar = st[3], beta1 = st[5];
  const double vo = own && !init ? v[c] : 0.0, wo = own && !init ? w[c] : 0.0, yo = own && !init ? y[c] : 0.0;
  // N's pieces: thread (c, p) the entries N[8 e + p][c] of q, the 16-lane
  // group r the entries N[r + groups m][l + 16 j] of z
  double nq[kE], nr[kHold ? 7 : 1], nz[kZr][kZ];
  const int dw = di / 8;
  if constexpr (kHold) {
#pragma unroll
    for (int e = 0; e < kE; ++e) nq[e] = N[(int64_t)std::min(8 * e + p, di - 1) * d + cl];
    if (p == 0)
#pragma unroll
      for (int q = 0; q < 7; ++q) nr[q] = N[(int64_t)std::min(8 * dw + q, di - 1) * d + cl];
#pragma unroll
    for (int m = 0; m < kZr; ++m)
#pragma unroll
      for (int j = 0; j < kZ; ++j) {
        const int r = gr + kThreads / 16 * m, cc = gl + 16 * j;
        nz[m][j] = N[(int64_t)(r < di ? r : 0) * d + (cc < di ? cc : 0)];
      }
  }
  if (stop != 0.0) {
    if (threadIdx.x == 0 && hist != nullptr) hist[it] = phibar;
    return;
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) part[p * kU + u][c] = sp[u];
  __syncthreads();
  if (p == 0) {
    double s = part[0][c];
#pragma unroll
    for (int u = 1; u < 8; ++u) s += part[u][c];
    g[c] = c < di ? s : 0.0;
  }
  __syncthreads();
  // the chains of q = N^T g
#pragma unroll
  for (int u = 0; u < kU; ++u) sp[u] = 0.0;
  if constexpr (kHold) {
#pragma unroll
    for (int e = 0; e < kE; ++e) sp[0] = e < dw ? fma(nq[e], g[8 * e + p], sp[0]) : sp[0];
    if (p == 0)
#pragma unroll
      for (int q = 0; q < 7; ++q) sp[0] = 8 * dw + q < di ? fma(nr[q], g[std::min(8 * dw + q, C - 1)], sp[0]) : sp[0];
  } else {
    // kQ rows of each chain in flight (past the last they load it again)
    constexpr int kQ = 16 / kU;
    const int end = __builtin_amdgcn_readfirstlane(c) < di ? dw : 0;  // (a wave wholly past d has none)
    for (int k0 = 0; k0 < end; k0 += kQ) {
      double a[kQ][kU];
#pragma unroll
      for (int q = 0; q < kQ; ++q)
#pragma unroll
        for (int u = 0; u < kU; ++u) a[q][u] = N[(int64_t)(8 * std::min(k0 + q, dw - 1) + p * kU + u) * d + cl];
#pragma unroll
      for (int q = 0; q < kQ; ++q)
        if (k0 + q < dw) {  // uniform
#pragma unroll
          for (int u = 0; u < kU; ++u) sp[u] = fma(a[q][u], g[8 * (k0 + q) + p * kU + u], sp[u]);
        }
    }
    if (p == 0)
      for (int i = 8 * dw; i < di; ++i) sp[0] = fma(N[(int64_t)i * d + cl], g[i], sp[0]);
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) part[p * kU + u][c] = sp[u];
  __syncthreads();
  // q, alpha = ||q||; the last wave: the rotation
  double qc = 0.0, a2 = 0.0;
  if (p == 0) {
    double s = part[0][c];
#pragma unroll
    for (int u = 1; u < 8; ++u) s += part[u][c];
    qc = c < di ? (init ? s : fma(-beta, vo, s)) : 0.0;
    a2 = wave_sum(qc * qc);
    if (C > 64 && lane == 0) red[wave] = a2;
  }
  if (wave == kWaves - 1 && !init) {
    const double rho = hypot(rhobar, beta);
    const double cs = rhobar / rho, sn = beta / rho;
    const double phi = cs * phibar;
    const double pr = phi / rho;
    if (lane == 0) {
      sc[0] = pr;
      sc[1] = sn;
      sc[2] = cs;
      sc[3] = rho;
    }
  }
  if constexpr (C > 64) {
    __syncthreads();
    a2 = 0.0;
    if (p == 0)
      for (int wv = 0; wv < C / 64; ++wv) a2 += red[wv];
  }
  double alpha = 0.0;
  if (p == 0) {
    alpha = sqrt(a2);
    const double ia = alpha > 0.0 ? 1.0 / alpha : 0.0;
    qc *= ia;  // the new v
    g[c] = qc;  // (v in LDS for z below; 0 past d)
    if (c < di) v[c] = qc;
  }
  __syncthreads();
  // z = N v for the next product, summed like a wave per row: each lane its
  // columns ascending, then partners 32, 16, 8, 4, 2, 1 apart
  if constexpr (kHold) {
#pragma unroll
    for (int m = 0; m < kZr; ++m) {
      double e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        e[j] = nz[m][j] * g[gl + 16 * j];
        if constexpr (C == 128) e[j] = 64 + gl + 16 * j < di ? fma(nz[m][4 + j], g[64 + gl + 16 * j], e[j]) : e[j];
      }
      const double zr = ror16_sum((e[0] + e[2]) + (e[1] + e[3]));
      const int r = gr + kThreads / 16 * m;
      if (gl == 0 && r < di) z[r] = zr;
    }
  } else {
    // a row's loads and the next row's in flight together; a lane past d takes
    // column 0 and adds nothing (a branch around the pieces past d cost more
    // than their loads)
    constexpr int kC = C / 64;
    double a[2][kC];
    auto load = [&](auto set, int r) {
      const double* row = N + (int64_t)std::min(r, di - 1) * d;
#pragma unroll
      for (int j = 0; j < kC; ++j) a[decltype(set)::value][j] = row[lane + 64 * j < di ? lane + 64 * j : 0];
    };
    auto use = [&](auto set, int r) {
      double zr = 0.0;
#pragma unroll
      for (int j = 0; j < kC; ++j)
        zr = lane + 64 * j < di ? fma(a[decltype(set)::value][j], g[lane + 64 * j], zr) : zr;
      zr = wave_sum(zr);
      if (lane == 0) z[r] = zr;
    };
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    load(s0, wave);
    for (int r = wave; r < di; r += 2 * kWaves) {
      load(s1, r + kWaves);
      use(s0, r);
      if (r + kWaves >= di) break;
      load(s0, r + 2 * kWaves);
      use(s1, r + kWaves);
    }
  }
  if (own) {
    if (init) {
      w[c] = qc;
      y[c] = 0.0;
    } else {
      const double theta = sc[1] * alpha;
      y[c] = fma(sc[0], wo, yo);
      w[c] = fma(-(theta / sc[3]), wo, qc);
    }
  }
  if (threadIdx.x == 0) {
    st[0] = alpha;
    if (init) {
      st[2] = alpha;  // rhobar = alpha_1
    } else {
      st[2] = -sc[2] * alpha;
      st[3] = sc[1] * phibar;
      if (hist != nullptr) hist[it] = sc[1] * phibar;
    }
    if (alpha == 0.0 || (!init && beta == 0.0) || beta1 == 0.0) st[4] = 1.0;
  }
}

// x = N y: a wave per row.
__global__ void lsqr_finish_kernel(int64_t d, const double* __restrict__ N, const double* __restrict__ y,
                                   double* __restrict__ x) {
  const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (r >= d) return;
  double acc = 0.0;
  for (int64_t c = threadIdx.x & 63; c < d; c += 64) acc = fma(N[r * d + c], y[c], acc);
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) x[r] = acc;
}

template <typename T>
hipError_t lsqr_typed(const void* Av, int64_t n, int64_t d, int64_t ld, const double* N, const double* b,
                      int64_t iters, double* x, double* hist, double* ws, hipStream_t s) {
  const T* A = static_cast<const T*>(Av);
  const int groups = lsqr_groups(n);
  double* st = ws;               // 8
  double* u = st + 8;            // n
  double* t = u + n;             // n
  double* gpart = t + n;         // groups
  double* apart = gpart + groups;  // groups * d
  double* v = apart + (size_t)groups * d;  // d
  double* w = v + d;
  double* y = w + d;
  double* z = y + d;
  hipError_t e = launch_fill_zero(st, 8 * sizeof(double), s);
  if (e != hipSuccess) return e;
  const auto gemv = d <= 64    ? lsqr_gemv_kernel<T, 1>
                    : d <= 128 ? lsqr_gemv_kernel<T, 2>
                    : d <= 256 ? lsqr_gemv_kernel<T, 4>
                               : lsqr_gemv_kernel<T, 0>;
  const auto atv = d <= 64 ? lsqr_atv_kernel<T, 1> : d <= 128 ? lsqr_atv_kernel<T, 2> : lsqr_atv_kernel<T, 4>;
  const auto step = d <= 64    ? lsqr_step_kernel<64>
                    : d <= 128 ? lsqr_step_kernel<128>
                    : d <= 256 ? lsqr_step_kernel<256>
                    : d <= 512 ? lsqr_step_kernel<512>
                               : lsqr_step_kernel<1024>;
  const int step_threads = d <= 64 ? 512 : 1024;
  // beta_1 u_1 = b; alpha_1 v_1 = M^T u_1
  gemv<<<groups, kGemvThreads, 0, s>>>(A, n, d, ld, z, u, b, 1, st, t, gpart);
  atv<<<groups, kAtvThreads, 0, s>>>(A, n, d, ld, t, gpart, groups, st, 1, u, apart);
  step<<<1, step_threads, 0, s>>>(d, N, apart, groups, st, v, w, y, z, hist, 0, 1);
  for (int64_t it = 0; it < iters; ++it) {
    gemv<<<groups, kGemvThreads, 0, s>>>(A, n, d, ld, z, u, b, 0, st, t, gpart);
    atv<<<groups, kAtvThreads, 0, s>>>(A, n, d, ld, t, gpart, groups, st, 0, u, apart);
    step<<<1, step_threads, 0, s>>>(d, N, apart, groups, st, v, w, y, z, hist, it, 0);
  }
  lsqr_finish_kernel<<<(unsigned)((d + 3) / 4), 256, 0, s>>>(d, N, y, x);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_precondition(int method, int64_t d, const double* R, const int64_t* rank, const int32_t* perm,
                               double zeta, double* work, double* N, int64_t* k_out, int32_t* err,
                               hipStream_t s) {
  if (method == 1) {
    if (d > 128) return hipErrorInvalidValue;
    const int64_t dd = d + (d & 1);
    const int elems = d <= 64 ? 4 : 8;  // of a column in a lane of its group
    const size_t lds = sizeof(double) * (size_t)(dd * svd_stride(elems));  // <= 144 KiB
    const int threads = (int)std::max<int64_t>(64, (dd / 2 * kSvdGroup + 63) / 64 * 64);
    const auto kernel = d <= 64 ? jacobi_svd_kernel<4> : jacobi_svd_kernel<8>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kernel<<<1, threads, lds, s>>>(d, R, rank, perm, zeta, N, k_out);
    return hipGetLastError();
  }
  // QR: Z = R11^{-1}, rows scattered to the original columns
  double* I = work;
  double* Z = work + d * d;
  hipError_t e = launch_trsm_inverse(d, R, rank, I, Z, err, s);
  if (e != hipSuccess) return e;
  scatter_rows_kernel<<<(unsigned)((d * d + 255) / 256), 256, 0, s>>>(d, perm, Z, N, rank, k_out);
  return hipGetLastError();
}

// k = -1 when a bounded wait of the rank-revealing step ran out.
__global__ void flag_error_kernel(const int32_t* __restrict__ err, int64_t* __restrict__ k_out) {
  if (*err != 0) *k_out = -1;
}

hipError_t launch_flag_error(const int32_t* err, int64_t* k_out, hipStream_t s) {
  flag_error_kernel<<<1, 1, 0, s>>>(err, k_out);
  return hipGetLastError();
}

int lsqr_groups(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(1024, (n + 255) / 256)); }

size_t lsqr_ws_doubles(int64_t n, int64_t d) {
  return 8 + 2 * (size_t)n + (size_t)lsqr_groups(n) * (1 + (size_t)d) + 4 * (size_t)d;
}

hipError_t launch_lsqr(int dtype, const void* A, int64_t n, int64_t d, int64_t ld, const double* N, const double* b,
                       int64_t iters, double* x, double* hist, double* ws, hipStream_t s) {
  switch (dtype) {
    case 0: return lsqr_typed<double>(A, n, d, ld, N, b, iters, x, hist, ws, s);
    case 1: return lsqr_typed<float>(A, n, d, ld, N, b, iters, x, hist, ws, s);
    case 2: return lsqr_typed<__hip_bfloat16>(A, n, d, ld, N, b, iters, x, hist, ws, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lev
