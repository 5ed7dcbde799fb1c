// B = A^T A of a tall dense A with d <= 256 columns on the FP64 matrix cores
// (Algorithm 5's Gram, for the exact scores of Algorithm 7).
//
// Bound: FP64 matrix work, 2 n d^2 / 2 flops on and above the diagonal (a
// large FP64 product reaches 70 TFLOP/s on this card); A is read once.
//
// One workgroup of 8 waves holds the whole upper triangle in accumulators
// and walks its share of the rows, so that A is staged (and FP32 / BF16
// widened) once and not once per output tile.  The triangle is cut into units
// of 16 rows x 64 columns (4 MFMA blocks); a wave owns U units, and where the
// triangle has fewer than 8 U units (d <= 128) the waves also split the rows
// of a step KG ways.  A step is kRows rows in LDS, double-buffered, the next
// step's global loads in flight during the current step's MFMAs; the operand
// reads of a unit are issued before the MFMAs of the unit before it.  LDS rows
// are padded by 16 elements, which puts the four k rows of an operand read on
// different banks.  Measured at 2^20 x 256 FP32: 1.45 ms, 59 TFLOP/s of the
// units' products (the tiled form, which reads and widens A five times over
// with per-element addresses: 5.18 ms).
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "lev_internal.h"
#include "tall_stage.h"

namespace lev {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kRows = 32;  // rows of A per step

// Unit u of the triangle of d columns, in order of (64-column block J, 16-row
// block i): i runs over the row blocks on and above J's last row, below d.
__device__ __forceinline__ bool unit_of(int u, int d, int* i_out, int* J_out) {
  const int rb = (d + 15) / 16;
  for (int J = 0; 64 * J < d; ++J) {
    const int cnt = 4 * (J + 1) < rb ? 4 * (J + 1) : rb;
    if (u < cnt) {
      *i_out = u;
      *J_out = J;
      return true;
    }
    u -= cnt;
  }
  *i_out = 0;
  *J_out = 0;
  return false;
}

// Index of (i, j), i <= j, in the packed upper triangle of d columns.
__device__ __forceinline__ int64_t packed(int i, int j, int d) { return (int64_t)i * d - (int64_t)i * (i - 1) / 2 + (j - i); }

// TB: 64-column blocks (d <= 64 TB).  Workgroup w adds rows
// [w chunk, (w + 1) chunk) and writes its packed triangle to partial + w tri.
template <typename TI, int TB, int U, int KG>
__global__ __launch_bounds__(kThreads) void gram_tall_kernel(const TI* __restrict__ A, int64_t n, int d, int64_t ld,
                                                             int64_t chunk, double* __restrict__ partial) {
  constexpr int stride = tall_stride(TB);
  constexpr int UG = kWaves / KG;  // waves that share a row group
  __shared__ __align__(16) tall_lds_t<TI> L[2][kRows * stride];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ug = wave % UG, kg = wave / UG;
  const int g = lane >> 4, c = lane & 15;
  const int64_t kb = (int64_t)blockIdx.x * chunk, ke = std::min<int64_t>(n, kb + chunk);

  int ui[U], uj[U];
  bool live[U];
#pragma unroll
  for (int u = 0; u < U; ++u) live[u] = unit_of(ug * U + u, d, &ui[u], &uj[u]);
  v4d acc[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[u][b] = v4d{0.0, 0.0, 0.0, 0.0};

  TallStep<TI, TB, kRows, kThreads> regs;
  if (kb < ke) {
    tall_load(regs, A, kb, ke, d, ld);
    tall_store(regs, ke - kb, L[0]);
  }
  __syncthreads();
  int buf = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += kRows) {
    const bool more = k0 + kRows < ke;
    if (more) tall_load(regs, A, k0 + kRows, ke, d, ld);
    __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of the products)
    // operand of lane l for rows k .. k + 3: row k + l / 16
    const tall_lds_t<TI>* base = L[buf] + (4 * kg + g) * stride + c;
    double oa[2], ob[2][4];
    auto read = [&](int u, int s, int slot) __attribute__((always_inline)) {
      const tall_lds_t<TI>* row = base + s * (4 * KG * stride);
      oa[slot] = (double)row[16 * ui[u]];
#pragma unroll
      for (int b = 0; b < 4; ++b) ob[slot][b] = (double)row[64 * uj[u] + 16 * b];
    };
    constexpr int S = kRows / 4 / KG;  // 4-row groups of this wave
    read(0, 0, 0);
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int cur = (s * U + u) & 1;
        if (u + 1 < U)
          read(u + 1, s, cur ^ 1);
        else if (s + 1 < S)
          read(0, s + 1, cur ^ 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[u][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(oa[cur], ob[cur][b], acc[u][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the other buffer was last read before the previous barrier
    if (more) tall_store(regs, ke - k0 - kRows, L[buf ^ 1]);
    __syncthreads();
    buf ^= 1;
  }

  if constexpr (KG > 1) {
    // the row groups' sums, added in order through LDS
    static_assert(sizeof(L) >= sizeof(double) * 64 * UG * U * 4, "one block of a unit a pass");
    double* X = reinterpret_cast<double*>(&L[0][0]);
#pragma unroll 1
    for (int from = 1; from < KG; ++from) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        __syncthreads();
        if (kg == from) {
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) X[((ug * U + u) * 4 + v) * 64 + lane] = acc[u][b][v];
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[u][b][v] += X[((ug * U + u) * 4 + v) * 64 + lane];
        }
      }
    }
    if (kg != 0) return;
  }
  double* out = partial + (int64_t)blockIdx.x * ((int64_t)d * (d + 1) / 2);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (!live[u]) continue;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * ui[u] + g + 4 * v, j = 64 * uj[u] + 16 * b + c;
        if (i <= j && j < d) out[packed(i, j, d)] = acc[u][b][v];
      }
  }
}

// B from the packed partial triangles: 64 elements of a row a workgroup, the
// partials in four interleaved groups added in a fixed order.
__global__ __launch_bounds__(256) void gram_tall_reduce_kernel(int d, int parts, const double* __restrict__ partial,
                                                               double* __restrict__ B) {
  __shared__ double s[4][64];
  const int i = blockIdx.y, j = blockIdx.x * 64 + (threadIdx.x & 63), z0 = threadIdx.x >> 6;
  if (blockIdx.x * 64 + 63 < (unsigned)i) return;
  const int64_t tri = (int64_t)d * (d + 1) / 2;
  const bool in = j >= i && j < d;
  const double* p = partial + (in ? packed(i, j, d) : 0);
  double a = 0.0;
#pragma unroll 8
  for (int z = z0; z < parts; z += 4) a += p[z * tri];
  s[z0][threadIdx.x & 63] = a;
  __syncthreads();
  if (z0 != 0 || !in) return;
  const double t = ((s[0][threadIdx.x] + s[1][threadIdx.x]) + s[2][threadIdx.x]) + s[3][threadIdx.x];
  B[(int64_t)i * d + j] = t;
  B[(int64_t)j * d + i] = t;
}

template <typename TI>
void launch(const TI* A, int64_t n, int d, int64_t ld, int parts, double* partial, hipStream_t s) {
  int64_t chunk = (n + parts - 1) / parts;
  chunk = (chunk + 3) / 4 * 4;
  // units: 4, 12, 24, 40 for one to four column blocks
  if (d <= 64)
    gram_tall_kernel<TI, 1, 2, 4><<<parts, kThreads, 0, s>>>(A, n, d, ld, chunk, partial);
  else if (d <= 128)
    gram_tall_kernel<TI, 2, 3, 2><<<parts, kThreads, 0, s>>>(A, n, d, ld, chunk, partial);
  else if (d <= 192)
    gram_tall_kernel<TI, 3, 3, 1><<<parts, kThreads, 0, s>>>(A, n, d, ld, chunk, partial);
  else
    gram_tall_kernel<TI, 4, 5, 1><<<parts, kThreads, 0, s>>>(A, n, d, ld, chunk, partial);
}

}  // namespace

// Partial triangles (workgroups) of the tall form within the room of
// `splits` full d x d partials, or 0 where the tiled form is the better one.
// The tall form keeps one workgroup a CU busy, at three to four times the
// tiled form's rate on FP32 and BF16, and gets about 2 splits of them (a triangle is half a
// square), so it needs a third of the CUs to win: 96 workgroups, which n of
// about 50 000 gives (exact scores at 65536 x 63 FP32, 127 workgroups: 184 us
// against 428; 100003 x 200 FP64: 1.05 ms against 1.21).
// FP64 A is not widened, so there the tiled form does better once the triangle
// is large against its fixed cost, a wider reduction: with fewer than 160
// workgroups it is taken beyond 192 columns, and beyond 128 for more than 2^16
// rows (rank of a 101- to 127-workgroup sketch, tall and tiled: 24000 x 200 303
// and 279 us, 400000 x 256 1546 and 947; 40000 x 160 232 and 246, 400000 x 160 787
// and 715).
// A's rows are read as 16-byte pieces, so its base and pitch have to be whole
// ones: the interface asks that of A, but not of a sketch handed to
// lev_rank_estimate, which may start 8 bytes off (the tiled form reads
// elements).
int gram_tall_partials(const void* A, int64_t n, int64_t d, int64_t ld, int64_t elt, int splits) {
  if (d > 256 || splits < 2 || (ld * elt) % 16 != 0 || reinterpret_cast<uintptr_t>(A) % 16 != 0) return 0;
  const int64_t room = (int64_t)splits * 2 * d / (d + 1);
  const int64_t parts = std::min<int64_t>(256, room);
  if (parts < 96 || n < 64 * parts) return 0;
  // FP64 with fewer than 160 workgroups: see above
  if (elt == 8 && parts < 160 && (d > 192 || (d > 128 && n > 65536))) return 0;
  return (int)parts;
}

hipError_t launch_gram_tall(int dtype, const void* A, int64_t n, int64_t d, int64_t ld, int parts, double* partial,
                            double* B, hipStream_t s) {
  switch (dtype) {
    case 0: launch(static_cast<const double*>(A), n, (int)d, ld, parts, partial, s); break;
    case 1: launch(static_cast<const float*>(A), n, (int)d, ld, parts, partial, s); break;
    case 2: launch(static_cast<const __hip_bfloat16*>(A), n, (int)d, ld, parts, partial, s); break;
    default: return hipErrorInvalidValue;
  }
  gram_tall_reduce_kernel<<<dim3((unsigned)((d + 63) / 64), (unsigned)d), 256, 0, s>>>((int)d, parts, partial, B);
  return hipGetLastError();
}

}  // namespace lev
