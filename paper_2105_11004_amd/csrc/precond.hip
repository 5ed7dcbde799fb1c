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
// ordering orthogonalises all its disjoint column pairs at once (an 8-lane
// group per pair, Rutishauser's rotation), and sweeps repeat until no pair
// is rotated.  Then W = R^T U_R = V_R Sigma: the column norms are the
// singular values and column c over its norm is the right singular vector,
// so N = P W Sigma^{-2} without accumulating the rotations.  Relative
// accuracy of the singular values does not depend on kappa(R).
//
// LSQR (Paige and Saunders 1982) on M = A N from y = 0, with x = N y at the
// end.  Per iteration one pass over A (dense, FP64 arithmetic on any storage
// type) and one single-workgroup kernel:
//   pass:  t = A (N v) - alpha u, and per workgroup the sums of t_i^2 and of
//          t_i A[i,:] from the row that is still in registers; u is never
//          stored: it is t over the beta that the step finds;
//   step:  beta = ||t||, A^T u = (A^T t) / beta, q = N^T (A^T u) - beta v,
//          alpha = ||q||, v = q / alpha, the rotation (rho, c, s, theta,
//          phi), y += (phi / rho) w, w = v - (theta / rho) w, z = N v for
//          the next pass.
// Scalars stay in device memory; all sums run in a fixed order.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "lev_internal.h"

namespace lev {
namespace {

constexpr int kSvdGroup = 8;            // lanes per column pair
constexpr int kSvdMaxThreads = 512;     // 64 groups: every pair of a round at d <= 128
constexpr int kMaxSweeps = 40;
// stride of a column of W in LDS: 16 PAIRS elements and the banks' offset
__host__ __device__ constexpr int svd_stride(int pairs) { return 2 * kSvdGroup * pairs + 16; }

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

// Sum over each 8-lane half row or 16-lane row by butterflies whose partners
// always sit in the other half of the part summed so far, so both sides add
// the same two values and every lane ends with identical bits (a rotation is
// then the same in every lane).  All lanes of the part must be active.
__device__ __forceinline__ double row8_sum(double v) {
  v = dpp_add<0xB1>(v);      // quad_perm [1, 0, 3, 2]
  v = dpp_add<0x4E>(v);      // quad_perm [2, 3, 0, 1]
  return dpp_add<0x141>(v);  // row_half_mirror
}
__device__ __forceinline__ double row16_sum(double v) {
  return dpp_add<0x140>(row8_sum(v));  // row_mirror
}

// 1 / sqrt(x) for normal x > 0: the hardware estimate (within 2^-20) and one
// step of third order, y (1 + e / 2 + 3 e^2 / 8) with e = 1 - x y^2.
__device__ __forceinline__ double rsqrt_step(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// One workgroup, eight lanes per column pair (rounded up to a wave); LDS
// holds W column-major, dd columns (a zero column pads an odd d) of
// 16 PAIRS elements, zero past d, at a stride of 16 more (so that columns
// next to each other start in opposite halves of the banks).  A lane holds
// the elements 2 l + 16 j and + 1 of a column; PAIRS = 4 (d <= 64) or 8.
//
// Bound by the chain of one round (LDS read, three dot products and their
// reductions, the rotation, LDS write, barrier), which is repeated dd - 1
// times a sweep.  Eight lanes a pair put one wave on each SIMD at d = 64, so
// no SIMD works through the rotation's replicated scalars twice; with four
// lanes the elements' work would outweigh them.  The angle comes from two
// reciprocal square roots without a division: with h = y.y - x.x, g = 2 x.y
// and r = hypot(h, g), cos^2 = (1 + |h| / r) / 2 and |sin| = |g| / (2 r cos),
// the pair of Rutishauser's smaller angle; h and g are first scaled by the
// power of two of the larger, so no square leaves the range.
// d = 60: 491 -> 252 us (16 lanes a pair, bounds checked, three divisions and
// a square root before).
template <int PAIRS>
__global__ __launch_bounds__(kSvdMaxThreads) void jacobi_svd_kernel(int64_t d, const double* __restrict__ R,
                                                                    const int64_t* __restrict__ rank,
                                                                    const int32_t* __restrict__ perm, double zeta,
                                                                    double* __restrict__ N,
                                                                    int64_t* __restrict__ k_out) {
  extern __shared__ __align__(16) double W[];
  __shared__ int rotated;
  __shared__ double sig[128];
  __shared__ int order[128];
  const int di = (int)d;
  const int dd = di + (di & 1);
  constexpr int kRows = 2 * kSvdGroup * PAIRS, kStride = svd_stride(PAIRS);
  const int r = (int)*rank;
  // W = R^T: column c of W is row c of R (rows past the rank are zero)
  for (int e = threadIdx.x; e < dd * kRows; e += blockDim.x) {
    const int c = e / kRows, i = e % kRows;
    W[c * kStride + i] = (c < r && i < di) ? R[(int64_t)c * d + i] : 0.0;
  }
  __syncthreads();
  const int gl = threadIdx.x & (kSvdGroup - 1);
  const int q = threadIdx.x / kSvdGroup;
  const bool active = q < dd / 2;  // whole groups are active or not
  // a pair is rotated while |x . y| > tol ||x|| ||y||, tested squared
  const double tol = 4.0 * (double)di * 2.220446049250313e-16;
  const double tol2 = tol * tol;
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    if (threadIdx.x == 0) rotated = 0;
    __syncthreads();
    int a = rr_col(dd, 0, q), b = rr_col(dd, 0, dd - 1 - q);
    for (int t = 0; t < dd - 1; ++t, a = rr_next(dd, a), b = rr_next(dd, b)) {
      if (active) {
        double* wa = W + a * kStride + 2 * gl;
        double* wb = W + b * kStride + 2 * gl;
        double2 x[PAIRS], y[PAIRS];
#pragma unroll
        for (int j = 0; j < PAIRS; ++j) {
          x[j] = *reinterpret_cast<const double2*>(wa + 2 * kSvdGroup * j);
          y[j] = *reinterpret_cast<const double2*>(wb + 2 * kSvdGroup * j);
        }
        double al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
        for (int j = 0; j < PAIRS; ++j) {
          al = fma(x[j].x, x[j].x, al);
          be = fma(y[j].x, y[j].x, be);
          ga = fma(x[j].x, y[j].x, ga);
          al = fma(x[j].y, x[j].y, al);
          be = fma(y[j].y, y[j].y, be);
          ga = fma(x[j].y, y[j].y, ga);
        }
        al = row8_sum(al);
        be = row8_sum(be);
        ga = row8_sum(ga);
        if (ga * ga > tol2 * (al * be)) {
          const double h0 = be - al, g0 = 2.0 * ga;
          const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(h0), fabs(g0)));
          const double h = ldexp(h0, ex), g = ldexp(g0, ex);
          const double ir = rsqrt_step(fma(h, h, g * g));  // 1/4 <= h^2 + g^2 < 2
          const double c2 = fma(0.5 * fabs(h), ir, 0.5);
          const double ic = rsqrt_step(c2);
          const double c = c2 * ic;
          const double s = (h < 0.0 ? -0.5 : 0.5) * g * (ir * ic);
#pragma unroll
          for (int j = 0; j < PAIRS; ++j) {
            *reinterpret_cast<double2*>(wa + 2 * kSvdGroup * j) =
                make_double2(c * x[j].x - s * y[j].x, c * x[j].y - s * y[j].y);
            *reinterpret_cast<double2*>(wb + 2 * kSvdGroup * j) =
                make_double2(s * x[j].x + c * y[j].x, s * x[j].y + c * y[j].y);
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
// st: [0] alpha, [1] beta, [2] rhobar, [3] phibar, [4] stop (0 / 1), [5] beta_1, [6] 1 / beta
constexpr int kPassThreads = 512;
constexpr int kStepThreads = 1024;

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

// Sum over the G lanes (16 or 64) that share a row, returned to all of them.
template <int G>
__device__ __forceinline__ double row_sum(double v) {
  v = row16_sum(v);
  if constexpr (G == 64) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
  }
  return v;
}

// t_i = A[i,:] z - alpha u_i (or b_i when INIT), u = the previous t over its
// beta; per workgroup gpart = sum of t_i^2 and apart[c] = sum of t_i A[i][c].
// G lanes take a row, four consecutive elements a lane and 4 G columns a
// block of M, so the row is read once, stays in registers and serves both
// the dot product and the sum; z and the sums are in registers too.  d <= 64
// M in {1, 2, 4} takes G = 16 (four rows a wave, a reduction of four DPP
// steps), wider rows a whole wave.  Rows past the end are read clamped and
// enter with t = 0.  Sums run in a fixed order: a lane's rows ascending, then
// the workgroup's groups in LDS.
//
// Bound by the reads of A (one instead of the two of a separate product with
// A and with A^T) and, when A fits the caches, by the launch and the chain
// of one row.
// 50000 x 60 FP64: 5.8 us, where the product with A took 13 and the one with
// A^T (15 of 64 lanes live at d = 60) 24.
template <typename T, int G, int M, bool INIT>
__global__ __launch_bounds__(kPassThreads) void lsqr_pass_kernel(const T* __restrict__ A, int64_t n, int64_t d,
                                                                 int64_t ld, const double* __restrict__ z,
                                                                 const double* __restrict__ b,
                                                                 const double* __restrict__ st, double* t,
                                                                 double* __restrict__ gpart,
                                                                 double* __restrict__ apart) {
  constexpr int kSlots = kPassThreads / G;  // rows the workgroup takes at a time
  constexpr int kCols = 4 * G * M;
  constexpr int kU = M == 1 ? 4 : 2;        // rows in flight per lane
  constexpr int kParts = kCols < kPassThreads ? kPassThreads / kCols : 1;
  __shared__ __align__(16) double red[kSlots * kCols];
  __shared__ double red2[kParts > 1 ? kPassThreads : 1];
  __shared__ double sqs[kPassThreads / 64];
  const double alpha = INIT ? 0.0 : st[0], inv = INIT ? 0.0 : st[6], stop = INIT ? 0.0 : st[4];
  const int gl = threadIdx.x % G, slot = threadIdx.x / G;
  const int64_t rows_per_group = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_group, r1 = std::min<int64_t>(n, r0 + rows_per_group);
  double zc[M][4], acc[M][4];
  int64_t col[M];  // the lane's columns; lanes past d read column 0 with z = 0
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int64_t c = 4 * G * m + 4 * gl;
    col[m] = c < d ? c : 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      zc[m][e] = !INIT && c + e < d ? z[c + e] : 0.0;
      acc[m][e] = 0.0;
    }
  }
  double sq = 0.0;
  for (int64_t i0 = r0; i0 < r1; i0 += kU * kSlots) {
    double a[kU][M][4], to[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t i = std::min<int64_t>(i0 + slot + u * kSlots, r1 - 1);
#pragma unroll
      for (int m = 0; m < M; ++m) load4(A + i * ld + col[m], col[m], d, a[u][m]);
      to[u] = INIT ? b[i] : t[i];
    }
    if (stop != 0.0) return;  // (nothing reads this pass's results then)
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t i = i0 + slot + u * kSlots;
      double ti = to[u];
      if constexpr (!INIT) {
        double dot = 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int e = 0; e < 4; ++e) dot = fma(a[u][m][e], zc[m][e], dot);
        ti = row_sum<G>(dot) - alpha * (to[u] * inv);
      }
      if (i >= r1) ti = 0.0;
      if (gl == 0 && i < r1) t[i] = ti;
      sq = fma(ti, ti, sq);
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[m][e] = fma(ti, a[u][m][e], acc[m][e]);
    }
  }
  // the workgroup's sums
  sq = wave_sum(gl == 0 ? sq : 0.0);
  if ((threadIdx.x & 63) == 0) sqs[threadIdx.x >> 6] = sq;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    double* o = red + slot * kCols + 4 * G * m + 4 * gl;
    *reinterpret_cast<double2*>(o) = make_double2(acc[m][0], acc[m][1]);
    *reinterpret_cast<double2*>(o + 2) = make_double2(acc[m][2], acc[m][3]);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kPassThreads / 64; ++w) s += sqs[w];
    gpart[blockIdx.x] = s;
  }
  if constexpr (kParts > 1) {
    const int c = threadIdx.x % kCols, p = threadIdx.x / kCols;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kSlots / kParts; ++q) s += red[(p + q * kParts) * kCols + c];
    red2[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < kCols && c < d) {
      s = red2[c];
#pragma unroll
      for (int q = 1; q < kParts; ++q) s += red2[q * kCols + c];
      apart[(int64_t)blockIdx.x * d + c] = s;
    }
  } else {
    for (int c = threadIdx.x; c < d; c += kPassThreads) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < kSlots; ++q) s += red[q * kCols + c];
      apart[(int64_t)blockIdx.x * d + c] = s;
    }
  }
}

template <typename T, int G, int M>
void launch_lsqr_pass_gm(bool init, int groups, const T* A, int64_t n, int64_t d, int64_t ld, const double* z,
                         const double* b, const double* st, double* t, double* gpart, double* apart, hipStream_t s) {
  const auto kernel = init ? lsqr_pass_kernel<T, G, M, true> : lsqr_pass_kernel<T, G, M, false>;
  kernel<<<groups, kPassThreads, 0, s>>>(A, n, d, ld, z, b, st, t, gpart, apart);
}

// The narrowest of the layouts that holds a row.
template <typename T>
void launch_lsqr_pass(bool init, int groups, const T* A, int64_t n, int64_t d, int64_t ld, const double* z,
                      const double* b, const double* st, double* t, double* gpart, double* apart, hipStream_t s) {
  const auto f = d <= 64    ? launch_lsqr_pass_gm<T, 16, 1>
                 : d <= 128 ? launch_lsqr_pass_gm<T, 16, 2>
                 : d <= 256 ? launch_lsqr_pass_gm<T, 16, 4>
                 : d <= 512 ? launch_lsqr_pass_gm<T, 64, 2>
                            : launch_lsqr_pass_gm<T, 64, 4>;
  f(init, groups, A, n, d, ld, z, b, st, t, gpart, apart, s);
}

// One LSQR step after the pass (init: the first alpha, v, w).  Thread (c, p)
// of 1024 takes column c and every P-th of the terms of its sums (P = 1024
// over the power of two that holds d), and the P parts meet in LDS, so the
// whole workgroup loads; SPAN = 1 or 2 (d <= 64 SPAN) also holds its pieces
// of N in registers, fetched before the sums that they wait for.  z = N v
// takes a 16-lane group per row there, a wave per row beyond.
//
// One workgroup: bound by the latency of its chain (partials, N^T, alpha, v,
// z).  The square roots and divisions are long FP64 sequences, so a single
// wave runs each: the last wave finds beta and the rotation while the first
// ones sum the columns, and only the columns' own waves find alpha; run by
// all sixteen waves they filled the SIMDs.
// d = 60, 391 partials: 7.9 us (15.7 before, when a column had one thread).
template <int SPAN>
__global__ __launch_bounds__(kStepThreads) void lsqr_step_kernel(int64_t d, const double* __restrict__ N,
                                                                 const double* __restrict__ apart,
                                                                 const double* __restrict__ gpart, int groups,
                                                                 double* __restrict__ st, double* __restrict__ v,
                                                                 double* __restrict__ w, double* __restrict__ y,
                                                                 double* __restrict__ z, double* __restrict__ hist,
                                                                 int64_t it, int init) {
  constexpr int kWaves = kStepThreads / 64;
  __shared__ double g[1024];
  __shared__ double part[kStepThreads];
  __shared__ double red[kWaves];
  __shared__ double sc[6];  // beta, 1 / beta, phi / rho, sin / rho, cos, sin
  const int di = (int)d;
  int lc = SPAN == 1 ? 6 : 7;  // log2 of the columns
  if constexpr (SPAN == 0)
    while ((1 << lc) < di) ++lc;
  const int C = 1 << lc, P = kStepThreads >> lc;
  const int c = threadIdx.x & (C - 1), p = threadIdx.x >> lc;
  const int cl = c < di ? c : 0;  // columns past d load column 0 and are dropped
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool own = p == 0 && c < di;
  // N's pieces: thread (c, p) the entries N[p + P e][c] of q, the 16-lane
  // group r the entries N[r + 64 m][l + 16 j] of z
  constexpr int kE = SPAN == 0 ? 1 : 4 * SPAN * SPAN, kZ = SPAN == 0 ? 1 : 4 * SPAN;
  double nq[kE], nz[SPAN == 0 ? 1 : SPAN][kZ];
  const int gl = threadIdx.x & 15, gr = threadIdx.x >> 4;
  // beta^2 = the sum of the gpart, and the sums of the columns' partials:
  // kU loads in flight, added in a fixed order
  double bs = 0.0;
  for (int gg = threadIdx.x; gg < groups; gg += kStepThreads) bs += gpart[gg];
  constexpr int kU = 16;
  double sp[4] = {0.0, 0.0, 0.0, 0.0};
  for (int g0 = p; g0 < groups; g0 += P * kU) {
    double a[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) a[u] = apart[(int64_t)std::min(g0 + P * u, groups - 1) * d + cl];
#pragma unroll
    for (int u = 0; u < kU; ++u) sp[u & 3] += g0 + P * u < groups ? a[u] : 0.0;
  }
  const double stop = init ? 0.0 : st[4], rhobar = st[2], phibar = st[3], beta1 = st[5];
  const double vo = own && !init ? v[c] : 0.0, wo = own && !init ? w[c] : 0.0, yo = own && !init ? y[c] : 0.0;
  if constexpr (SPAN > 0) {
#pragma unroll
    for (int e = 0; e < kE; ++e) nq[e] = N[(int64_t)std::min(p + P * e, di - 1) * d + cl];
#pragma unroll
    for (int m = 0; m < SPAN; ++m)
#pragma unroll
      for (int j = 0; j < kZ; ++j) {
        const int r = gr + 64 * m, cc = gl + 16 * j;
        nz[m][j] = N[(int64_t)(r < di ? r : 0) * d + (cc < di ? cc : 0)];
      }
  }
  if (stop != 0.0) {
    if (threadIdx.x == 0 && hist != nullptr) hist[it] = phibar;
    return;
  }
  part[threadIdx.x] = (sp[0] + sp[1]) + (sp[2] + sp[3]);
  bs = wave_sum(bs);
  if (lane == 0) red[wave] = bs;
  __syncthreads();
  // g = A^T t (its 1 / beta comes in with q), and beta
  if (p == 0) {
    double s = part[c];
#pragma unroll
    for (int q = 1; q < P; ++q) s += part[(q << lc) + c];
    g[c] = c < di ? s : 0.0;
  }
  if (wave == kWaves - 1) {
    double b2 = 0.0;
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) b2 += red[wv];
    const double beta = sqrt(b2);
    if (lane == 0) {
      sc[0] = beta;
      sc[1] = beta > 0.0 ? 1.0 / beta : 0.0;
    }
  }
  __syncthreads();
  const double beta = sc[0], inv = sc[1];
  // N^T g, in P parts
  double qs = 0.0;
  if constexpr (SPAN > 0) {
#pragma unroll
    for (int e = 0; e < kE; ++e) qs = fma(nq[e], g[p + P * e], qs);  // (g is 0 past d)
  } else {
    double sq[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) sq[u] = 0.0;
    int i = p;
    for (; i + P * 7 < di; i += P * 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) sq[u] = fma(N[(int64_t)(i + P * u) * d + cl], g[i + P * u], sq[u]);
    for (; i < di; i += P) sq[0] = fma(N[(int64_t)i * d + cl], g[i], sq[0]);
    qs = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
  }
  part[threadIdx.x] = qs;
  __syncthreads();
  // q = N^T g / beta - beta v, alpha = ||q||; the last wave: the rotation
  double qc = 0.0, a2 = 0.0;
  if (p == 0) {
    qc = qs;
#pragma unroll
    for (int q = 1; q < P; ++q) qc += part[(q << lc) + c];
    qc = c < di ? qc * inv - beta * vo : 0.0;
    a2 = wave_sum(qc * qc);
    if (SPAN != 1 && lane == 0) red[wave] = a2;
  }
  if (wave == kWaves - 1 && !init) {
    const double rho = hypot(rhobar, beta);
    const double cs = rhobar / rho, sn = beta / rho;
    const double pr = cs * phibar / rho, sr = sn / rho;
    if (lane == 0) {
      sc[2] = pr;
      sc[3] = sr;
      sc[4] = cs;
      sc[5] = sn;
    }
  }
  if constexpr (SPAN != 1) {
    __syncthreads();
    a2 = 0.0;
    if (p == 0)
      for (int wv = 0; wv < C / 64; ++wv) a2 += red[wv];
  }
  double alpha = 0.0;
  if (p == 0) {
    alpha = sqrt(a2);
    const double ia = alpha > 0.0 ? 1.0 / alpha : 0.0;
    qc *= ia;                   // the new v
    g[c] = qc;                  // (still 0 past d)
    if (c < di) v[c] = qc;
  }
  __syncthreads();
  // z = N v for the next pass
  if constexpr (SPAN > 0) {
#pragma unroll
    for (int m = 0; m < SPAN; ++m) {
      double zr = 0.0;
#pragma unroll
      for (int j = 0; j < kZ; ++j) zr = fma(nz[m][j], g[gl + 16 * j], zr);
      zr = row16_sum(zr);
      if (gl == 0 && gr + 64 * m < di) z[gr + 64 * m] = zr;
    }
  } else {
    for (int r = wave; r < di; r += kWaves) {
      double zr = 0.0;
      for (int cc = lane; cc < di; cc += 64) zr = fma(N[(int64_t)r * d + cc], g[cc], zr);
      zr = wave_sum(zr);
      if (lane == 0) z[r] = zr;
    }
  }
  if (own) {
    y[c] = init ? 0.0 : fma(sc[2], wo, yo);
    w[c] = init ? qc : qc - sc[3] * alpha * wo;
  }
  if (threadIdx.x == 0) {
    st[0] = alpha;
    st[1] = beta;
    st[6] = inv;
    if (init) {
      st[2] = alpha;  // rhobar = alpha_1
      st[3] = beta;   // phibar = beta_1
      st[5] = beta;
    } else {
      st[2] = -sc[4] * alpha;
      st[3] = sc[5] * phibar;
      if (hist != nullptr) hist[it] = sc[5] * phibar;
    }
    if (alpha == 0.0 || (!init && beta == 0.0) || (init ? beta : beta1) == 0.0) st[4] = 1.0;
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
  double* t = st + 8;            // n
  double* gpart = t + n;         // groups
  double* apart = gpart + groups;  // groups * d
  double* v = apart + (size_t)groups * d;  // d
  double* w = v + d;
  double* y = w + d;
  double* z = y + d;
  hipError_t e = launch_fill_zero(st, 8 * sizeof(double), s);
  if (e != hipSuccess) return e;
  auto pass = [&](bool init) { launch_lsqr_pass<T>(init, groups, A, n, d, ld, z, b, st, t, gpart, apart, s); };
  const auto step = d <= 64 ? lsqr_step_kernel<1> : d <= 128 ? lsqr_step_kernel<2> : lsqr_step_kernel<0>;
  // beta_1 u_1 = b; alpha_1 v_1 = M^T u_1
  pass(true);
  step<<<1, kStepThreads, 0, s>>>(d, N, apart, gpart, groups, st, v, w, y, z, hist, 0, 1);
  for (int64_t it = 0; it < iters; ++it) {
    pass(false);
    step<<<1, kStepThreads, 0, s>>>(d, N, apart, gpart, groups, st, v, w, y, z, hist, it, 0);
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
    const bool narrow = d <= 64;  // a column's elements in its eight lanes: 4 or 8 pairs each
    const size_t lds = sizeof(double) * (size_t)(dd * svd_stride(narrow ? 4 : 8));  // <= 144 KiB
    const int threads = (int)std::max<int64_t>(64, (dd / 2 * kSvdGroup + 63) / 64 * 64);
    const auto kernel = narrow ? jacobi_svd_kernel<4> : jacobi_svd_kernel<8>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kernel<<<1, threads, lds, s>>>(d, R, rank, perm, zeta, N, k_out);
    return hipGetLastError();
  }
  // QR: Z = R11^{-1} (trsm of the identity), rows scattered to the original columns
  double* I = work;
  double* Z = work + d * d;
  hipError_t e = launch_identity(d, I, s);
  if (e != hipSuccess) return e;
  e = launch_trsm_z(d, d, R, rank, I, Z, err, s);
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

// At least 128 rows a workgroup (four per 16-lane group) and at most two
// workgroups a CU, which hold the loads that HBM's rate asks for.  Fewer
// workgroups make the pass longer by what the step gains: 50000 x 60 takes
// 5.8 + 7.9 us at 391 of them, 7.2 + 6.6 at 261.
int lsqr_groups(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(512, (n + 127) / 128)); }

size_t lsqr_ws_doubles(int64_t n, int64_t d) {
  return 8 + (size_t)n + (size_t)lsqr_groups(n) * (1 + (size_t)d) + 4 * (size_t)d;
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
