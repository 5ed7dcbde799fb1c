// Pass 2 for CSR input: theta~_i = || A[i, :] Z_full ||^2 (Algorithm 8, last
// step, on the selected columns; Z_full holds Z's rows at the selected
// columns' ids and zeros elsewhere).
//
// A sparse row times a dense d x k matrix has no dense tile for the matrix
// cores (a 16-row block of a 3%-dense A fills one 16x4 MFMA operand to a few
// percent), so this pass runs on the vector ALUs: every nonzero a_ij adds
// a_ij * Z_full[j, :] to the row's k-vector, one output column per lane.
// Z_full (padded to 64 columns) lives in LDS, shared by the 16 waves of a
// workgroup; each step gathers one 256-byte row of it, so the pass is bound
// by LDS bandwidth (about 256 B/clk per CU on gfx950) unless A's bytes are
// the larger cost.  Each wave streams a contiguous range of rows: the
// nonzeros of the range are read 64 at a time with coalesced loads and
// staged in a 64-entry LDS list (column offset into Z, value) that all lanes
// read by broadcast; row boundaries come from row_ptr and are uniform across
// the wave, so the step loop has no per-lane branches.  At a row boundary the
// squared k-vector is summed across the wave (DPP) into the row's lane of a
// result register, stored once per 64 rows.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "lev_internal.h"

namespace lev {
namespace {

constexpr int kCsrWaves = 16;
constexpr int kCsrThreads = 64 * kCsrWaves;
constexpr int kZStride = 64;  // Z_full row stride in elements (k <= 64)
constexpr int kRowsPerTask = 64, kMinRowsPerTask = 8, kTasksPerWave = 2;

template <typename T>
__device__ __forceinline__ float to_f32(T x);
template <>
__device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <>
__device__ __forceinline__ float to_f32<__hip_bfloat16>(__hip_bfloat16 x) {
  const uint16_t bits = *reinterpret_cast<const uint16_t*>(&x);
  return __uint_as_float((uint32_t)bits << 16);
}

// Sum over the 64 lanes (row shifts within 16-lane rows, then row
// broadcasts; lane 63 ends with the total), returned to every lane.
// (with every row on, a lane whose source is outside its row reads 0 either
// way; bound_ctrl says so, so no zeroed copy of the old value is made)
template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_sum_step(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWMASK, 0xF, ROWMASK == 0xF));
}
__device__ __forceinline__ float wave_sum(float v) {
  v = dpp_sum_step<0x111, 0xF>(v);
  v = dpp_sum_step<0x112, 0xF>(v);
  v = dpp_sum_step<0x114, 0xF>(v);
  v = dpp_sum_step<0x118, 0xF>(v);
  v = dpp_sum_step<0x142, 0xA>(v);
  v = dpp_sum_step<0x143, 0xC>(v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_sum_step(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWMASK, 0xF, ROWMASK == 0xF);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWMASK, 0xF, ROWMASK == 0xF);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_sum_step<0x111, 0xF>(v);
  v = dpp_sum_step<0x112, 0xF>(v);
  v = dpp_sum_step<0x114, 0xF>(v);
  v = dpp_sum_step<0x118, 0xF>(v);
  v = dpp_sum_step<0x142, 0xA>(v);
  v = dpp_sum_step<0x143, 0xC>(v);
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ int64_t readlane64(int64_t x, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <typename ZT>
struct StageEntry {
  int off;   // element offset of Z_full's row in LDS (column id * kZStride)
  ZT val;
};

// G consecutive steps t .. t + G - 1 of the staged list: the G entry reads,
// then the G Z-row reads, then the products (alternating accumulators).
template <int G, typename ZT>
__device__ __forceinline__ void steps(const StageEntry<ZT>* my, const ZT* Z, int t, int lane, ZT& y, ZT& y2) {
  StageEntry<ZT> e[G];
  ZT z[G];
#pragma unroll
  for (int u = 0; u < G; ++u) e[u] = my[t + u];
#pragma unroll
  for (int u = 0; u < G; ++u) z[u] = Z[e[u].off + lane];
#pragma unroll
  for (int u = 0; u < G; u += 2) {
    y = fma(e[u].val, z[u], y);
    y2 = fma(e[u + 1].val, z[u + 1], y2);
  }
}

// T: storage type of A's values; ZT: type of Z_full and of the arithmetic
// (float for FP32/BF16 values, double for FP64 values).  ZLDS: Z_full staged
// in LDS (else read from global memory, for d * 64 * sizeof(ZT) beyond LDS).
template <typename T, typename ZT, bool ZLDS>
__global__ __launch_bounds__(kCsrThreads) void rownorm_csr_kernel(const T* __restrict__ vals,
                                                                  const int64_t* __restrict__ row_ptr,
                                                                  const int32_t* __restrict__ col_idx,
                                                                  int64_t n, int64_t d, int64_t nnz,
                                                                  const ZT* __restrict__ Zg,
                                                                  ZT* __restrict__ theta, ColTile ct,
                                                                  int rows_per_task) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (col_tile_dead(ct)) return;
  StageEntry<ZT>* stage = reinterpret_cast<StageEntry<ZT>*>(smem);  // [kCsrWaves][64]
  ZT* Zs = reinterpret_cast<ZT*>(smem + sizeof(StageEntry<ZT>) * 64 * kCsrWaves);
  const ZT* Z = ZLDS ? Zs : Zg;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (ZLDS) {
    const int64_t total = d * kZStride;
    for (int64_t e = threadIdx.x; e < total; e += kCsrThreads) Zs[e] = Zg[e];
    __syncthreads();
  }
  StageEntry<ZT>* my = stage + wave * 64;

  const int64_t ntask = (n + rows_per_task - 1) / rows_per_task;
  for (int64_t task = (int64_t)blockIdx.x * kCsrWaves + wave; task < ntask;
       task += (int64_t)gridDim.x * kCsrWaves) {
    const int64_t r0 = task * rows_per_task;  // at most 64 rows
    const int64_t r1 = min(n, r0 + rows_per_task);
    // lane j holds row_ptr[r0 + j] (j <= r1 - r0; lane 64 would be r1 = r0 + 64)
    // Offsets are clamped to [0, nnz] and row ends to [pos, N1], so a
    // malformed row_ptr yields wrong rows but no stray access or endless loop.
    const int64_t rp = (r0 + lane <= r1) ? min(max(row_ptr[r0 + lane], (int64_t)0), nnz) : 0;
    const int64_t N0 = readlane64(rp, 0);
    const int64_t N1 = max(N0, min(max(row_ptr[r1], (int64_t)0), nnz));
    int64_t pos = N0;
    auto row_end = [&](int64_t row) -> int64_t {  // row_ptr[row + 1], row in [r0, r1)
      const int j = (int)(row + 1 - r0);
      return j < 64 ? min(max(readlane64(rp, j), pos), N1) : N1;
    };

    ZT out = 0;  // lane j: theta of row r0 + j
    ZT y = 0, y2 = 0;  // two accumulators: the unrolled steps alternate
    int64_t row = r0;
    int64_t rend = row_end(row);
    auto flush_rows = [&]() {
      while (row < r1 && rend == pos) {
        const ZT yy = y + y2;
        const ZT t = wave_sum(yy * yy);
        out = (lane == (int)(row - r0)) ? t : out;
        y = 0;
        y2 = 0;
        ++row;
        if (row < r1) rend = row_end(row);
      }
    };
    flush_rows();
    // the column ids and values of the next 64 nonzeros are loaded while the
    // current 64 are multiplied (one global round trip per chunk is no
    // longer on the wave's critical path)
    auto load_chunk = [&](int64_t cs, int32_t& c, T& v) {
      const int64_t p = cs + lane;
      const int64_t q = p < N1 ? p : (N1 > 0 ? N1 - 1 : 0);  // in bounds whenever nnz > 0
      c = p < N1 ? col_idx[q] : -1;
      v = p < N1 ? vals[q] : T{};
    };
    int32_t nc = -1;
    T nv{};
    if (N0 < N1) load_chunk(N0, nc, nv);
    for (int64_t c0 = N0; c0 < N1; c0 += 64) {
      const int32_t c = nc;
      const T cv = nv;
      if (c0 + 64 < N1) load_chunk(c0 + 64, nc, nv);
      StageEntry<ZT> e;
      e.off = 0;
      e.val = 0;
      if ((uint32_t)c < (uint32_t)d) {
        e.off = c * kZStride;
        if constexpr (sizeof(ZT) == 8) {
          e.val = (ZT)cv;
        } else {
          e.val = to_f32<T>(cv);
        }
      }
      my[lane] = e;
      __builtin_amdgcn_wave_barrier();
      const int64_t cend = min(c0 + 64, N1);
      while (pos < cend && row < r1) {
        const int stop = (int)(min(rend, cend) - c0);
        int t = (int)(pos - c0);
        // eight steps at a time: all sixteen LDS reads are issued before the
        // first product, so their latencies overlap; a segment's last steps
        // go in groups of 4, 2 and 1 (at most three dependent LDS round
        // trips instead of seven, and no step padded: with Z_full filling
        // LDS the pass runs four waves per SIMD and is bound by LDS issue
        // as much as by latency)
        for (; t + 8 <= stop; t += 8) steps<8>(my, Z, t, lane, y, y2);
        if (t + 4 <= stop) {
          steps<4>(my, Z, t, lane, y, y2);
          t += 4;
        }
        if (t + 2 <= stop) {
          steps<2>(my, Z, t, lane, y, y2);
          t += 2;
        }
        if (t < stop) {
          const StageEntry<ZT> e1 = my[t];
          y = fma(e1.val, Z[e1.off + lane], y);
        }
        pos = c0 + stop;
        flush_rows();
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (r0 + lane < r1) theta[r0 + lane] = ct.acc ? theta[r0 + lane] + out : out;
  }
}

// ---- FP32 Z: rows shared out to 16-lane groups --------------------------------
// A wave takes 64 consecutive rows.  Lane l of group g (16 lanes) owns
// columns 4 (l % 16) .. + 3 of the k <= 64 output columns, and a group walks
// one row's nonzeros 16 at a time: each lane loads one (column id, value),
// then for each of the 16 entries the group reads the 16 bytes of Z_full's row
// it needs (ds_read_b128: the group reads the whole 256-byte row, conflict-
// free) and does four FMAs; the address and the products take the entry from
// its lane by themselves (DPP row_newbcast on the add and the FMAs, no move
// and no LDS).  A row of at most one nonzero a_ij needs no k-vector:
// theta = a_ij^2 ||Z_full[j,:]||^2, from the squared row norms of Z_full
// kept in LDS beside it, one row a lane.  The other light rows (2 .. 63
// nonzeros) go four at a time, one per group.  The four groups move in step, so a wave pays for the longest of
// its four rows: the light rows of the 64 are first ordered by length class
// (1, 2, 3-4, 5-8, ..., 33-63; counted with ballots, moved with a forward
// lane permutation), which puts rows of similar length side by side (with
// power-law row lengths, a third of the group steps did useful work in row
// order).  Heavy rows are split over the four groups, entry c0 + 4 i + g
// of a 64-entry piece going to lane i of group g, so a row's last partial
// stretch costs a quarter of its length, and the groups' partial k-vectors
// are added at the end.
// Z_full sits in LDS unpadded, 256 bytes a row: a group's 16-lane read is
// one whole row (measured on gfx950: a 68-float stride cost two bank-
// conflict cycles per LDS instruction, 64 none).  The squares of a row's k-vector
// are summed over the group with four DPP steps; the group's last lane
// stores theta.
//
// Bound by vector issue (82 % of the cycles at 2^23 x 512 with 16 nonzeros a
// row: 1575 of a task's 2850 instructions are the additions and FMAs of the
// entries, the rest the ordering, loads and sums of rows, 40 % of which have
// one nonzero).  There: 904 us; 1165 when an entry was moved before it was
// used, each LDS read waited for the one before it, and the sixteen steps over
// the light rows were unrolled past the instruction cache.
constexpr int kGZStride = 64;
constexpr int kHeavy = 64;
constexpr uint32_t kSpanMask = 0xFFFFFF, kSpan = 0xFFFF00;  // a light row starts at most this far into its task

__device__ __forceinline__ float group_sum16(float v) {
  // prefix within each 16-lane row; lane 15 of the row ends with the total
  v = dpp_sum_step<0x111, 0xF>(v);
  v = dpp_sum_step<0x112, 0xF>(v);
  v = dpp_sum_step<0x114, 0xF>(v);
  v = dpp_sum_step<0x118, 0xF>(v);
  return v;
}

// The four LDS reads of entries U0 .. U0 + 3: each lane's 16 bytes of the row
// of Z_full whose byte offset lane U of the group holds (the add takes it from
// there; s_nop covers a vector write of off just before).
template <int U0>
__device__ __forceinline__ void group_read4(const float* __restrict__ Zs, uint32_t off, uint32_t gl16, float4 (&z)[4]) {
  uint32_t o[4];
  asm("s_nop 1\n\t"
      "v_add_u32_dpp %0, %4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %1, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_u32_dpp %3, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
      : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3])
      : "v"(off), "v"(gl16), "n"(U0), "n"(U0 + 1), "n"(U0 + 2), "n"(U0 + 3));
#pragma unroll
  for (int u = 0; u < 4; ++u)
    z[u] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(Zs) + o[u]);
}

// y += the entries' products, in order; the values come from their lanes.
template <int U0>
__device__ __forceinline__ void group_fma4(float val, const float4 (&z)[4], float (&y)[4]) {
  asm("s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %4, %5 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %6 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %7 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %8 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %9 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %10 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %11 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %12 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %13 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %14 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %15 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %16 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %17 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %18 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %19 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %20 row_newbcast:%24 row_mask:0xf bank_mask:0xf"
      : "+&v"(y[0]), "+&v"(y[1]), "+&v"(y[2]), "+&v"(y[3])
      : "v"(val), "v"(z[0].x), "v"(z[0].y), "v"(z[0].z), "v"(z[0].w), "v"(z[1].x), "v"(z[1].y), "v"(z[1].z),
        "v"(z[1].w), "v"(z[2].x), "v"(z[2].y), "v"(z[2].z), "v"(z[2].w), "v"(z[3].x), "v"(z[3].y), "v"(z[3].z),
        "v"(z[3].w), "n"(U0), "n"(U0 + 1), "n"(U0 + 2), "n"(U0 + 3));
}

// y += the group's first `steps` (wave-uniform; rounded up to fours, at most
// 16) staged entries (byte offset of Z_full's row, value); masked entries
// carry offset 0 and a zero value.  Four reads are in flight while the four
// before them are added.
__device__ __forceinline__ void group_chunk(const float* __restrict__ Zs, uint32_t off, float val, uint32_t gl16,
                                            float (&y)[4], int steps) {
  float4 a[4], b[4];
  group_read4<0>(Zs, off, gl16, a);
  if (steps <= 4) {
    group_fma4<0>(val, a, y);
    return;
  }
  group_read4<4>(Zs, off, gl16, b);
  group_fma4<0>(val, a, y);
  if (steps <= 8) {
    group_fma4<4>(val, b, y);
    return;
  }
  group_read4<8>(Zs, off, gl16, a);
  group_fma4<4>(val, b, y);
  if (steps <= 12) {
    group_fma4<8>(val, a, y);
    return;
  }
  group_read4<12>(Zs, off, gl16, b);
  group_fma4<8>(val, a, y);
  group_fma4<12>(val, b, y);
}

template <typename T>
__global__ __launch_bounds__(kCsrThreads) void rownorm_csr_grp_kernel(const T* __restrict__ vals,
                                                                      const int64_t* __restrict__ row_ptr,
                                                                      const int32_t* __restrict__ col_idx,
                                                                      int64_t n, int64_t d, int64_t nnz,
                                                                      const float* __restrict__ Zg,
                                                                      float* __restrict__ theta, ColTile ct) {
  extern __shared__ __align__(16) float Zs[];  // d rows of kGZStride floats, then d squared row norms
  if (col_tile_dead(ct)) return;
  float* zn = Zs + d * kGZStride;
  {
    const float4* Z4 = reinterpret_cast<const float4*>(Zg);
#pragma unroll 8
    for (int e = threadIdx.x; e < (int)d * 16; e += kCsrThreads) reinterpret_cast<float4*>(Zs)[e] = Z4[e];
    if (threadIdx.x < d) {
      float4 z[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) z[q] = Z4[threadIdx.x * 16 + q];
      float a = 0.f;
#pragma unroll
      for (int q = 0; q < 16; ++q) a = fmaf(z[q].w, z[q].w, fmaf(z[q].z, z[q].z, fmaf(z[q].y, z[q].y, fmaf(z[q].x, z[q].x, a))));
      zn[threadIdx.x] = a;
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, gl = lane & 15;
  const uint32_t gl16 = 16 * gl;
  const int64_t ntask = (n + 63) / 64;
  const int64_t tstep = (int64_t)gridDim.x * kCsrWaves;
  int64_t task = (int64_t)blockIdx.x * kCsrWaves + wave;
  // the next task's row starts load while the current task runs
  auto row_start = [&](int64_t tk) -> int64_t {
    const int64_t r = std::min<int64_t>(tk, ntask - 1) * 64 + lane;
    return min(max(row_ptr[std::min<int64_t>(r, n)], (int64_t)0), nnz);
  };
  int64_t rp_next = row_start(task);
  for (; task < ntask; task += tstep) {
    const int64_t r0 = task * 64;
    float* th = theta + r0;
    auto store = [&](uint32_t r, float sq) { th[r] = ct.acc ? th[r] + sq : sq; };
    const int nr = (int)min((int64_t)64, n - r0);
    // lane j: start of row r0 + j, made non-decreasing
    int64_t rp = rp_next;
    rp_next = row_start(task + tstep);
    // (the shuffles run on every lane: a lane masked off by a branch does not
    // supply its value to the others)
    const int64_t before = __shfl_up(rp, 1, 64);
    if (__ballot(lane > 0 && before > rp) != 0) {
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int64_t up = __shfl_up(rp, o, 64);
        if (lane >= o) rp = max(rp, up);
      }
    }
    int64_t last = min(max(row_ptr[r0 + nr], (int64_t)0), nnz);
    last = max(last, __shfl(rp, 63, 64));
    if (lane >= nr) rp = last;  // rows past the task's end are empty
    const int64_t down = __shfl_down(rp, 1, 64);
    const int64_t rnext = lane < 63 ? down : last;
    const int len = lane < nr ? (int)(rnext - rp) : 0;
    const bool light = lane < nr && len < kHeavy;
    uint64_t heavy = __ballot(lane < nr && len >= kHeavy);

    // The heavy rows' pieces, 64 entries each, one after the other: entry
    // c0 + 4 i + g to lane i of group g.  A piece loads while the one before
    // it is added (the first before the light rows); every load is
    // unconditional, a lane past the row's end takes the piece's first entry.
    int hj = 0, hc0 = 0, hlen = 0;  // row, first entry and length of the loaded piece (uniform)
    int32_t hcol = 0;
    T hval{};
    auto heavy_load = [&](int j, int c0) {
      hj = j;
      hc0 = c0;
      hlen = __builtin_amdgcn_readlane(len, j);
      const int64_t s0 = ((int64_t)__builtin_amdgcn_readlane((int)(rp >> 32), j) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)rp, j);
      const uint32_t e = 4 * gl + g;
      const uint32_t at = (int)e < hlen - c0 ? e : 0;
      hcol = (col_idx + s0 + c0)[at];
      hval = (vals + s0 + c0)[at];
    };
    if (heavy != 0) heavy_load(__builtin_ctzll(heavy), 0);

    // rows of at most one nonzero, one a lane (an empty row's theta is 0)
    int32_t c1 = 0;
    T v1{};
    if (nnz > 0) {
      const int64_t at = min(rp, nnz - 1);
      c1 = col_idx[at];
      v1 = vals[at];
    }
    // the other light rows by length class; sorted position q holds a row's
    // start (from the task's first), its length and its number; the rows of
    // at most one nonzero (class 0), then the heavy rows and lanes past the
    // task's end sort outside positions n01 .. nlight - 1
    const int cls = light ? (len <= 1 ? 0 : 32 - __builtin_clz((unsigned)(len - 1))) : 7;
    int pos = 0, base = 0, nlight = 0, n01 = 0, n16 = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint64_t m = __ballot(cls == c);
      const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (cls == c) pos = base + below;
      base += __popcll(m);
      if (c == 0) n01 = base;
      if (c == 4) n16 = base;
      if (c == 6) nlight = base;
    }
    const int64_t first = ((int64_t)__builtin_amdgcn_readfirstlane((int)(rp >> 32)) << 32) |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)rp);
    // (64 rows of at most d entries span far less; a malformed row_ptr stays in bounds)
    const int rel = (int)min(rp - first, (int64_t)kSpan);
    const int rel_s = __builtin_amdgcn_ds_permute(4 * pos, rel);
    const int row_s = __builtin_amdgcn_ds_permute(4 * pos, (light ? len : 0) | (lane << 8));
    // the longest of positions q .. q + 3 (past the wave it wraps to rows of
    // class 0, no longer than these)
    int longest = row_s & 0xFF;
    longest = max(longest, __shfl(longest, (lane + 1) & 63, 64));
    longest = max(longest, __shfl(longest, (lane + 2) & 63, 64));
    if (light && len <= 1) {
      float sq = 0.f;
      if (len == 1 && (uint32_t)c1 < (uint32_t)d) {
        const float vv = to_f32<T>(v1);
        sq = vv * vv * zn[c1];
      }
      store(lane, sq);
    }

    // light rows of 2 .. 63 nonzeros: group g takes sorted positions
    // n01 + 4 q + g; the first 16 nonzeros (32 once rows are longer) of the
    // rows two steps ahead load while a step runs; a position at or past
    // nlight stands for an empty row (its lanes load the task's first entry)
    const int32_t* cb = col_idx + first;
    const T* vb = vals + first;
    struct Quad {
      int32_t c[2];
      T v[2];
      uint32_t rel;
      int row;  // length (0: no row), number << 8
    };
    auto quad_load = [&](Quad& x, int q, auto pieces) {
      const int jj = n01 + 4 * q + g;
      const int rj = __shfl(rel_s, jj & 63, 64), wj = __shfl(row_s, jj & 63, 64);  // on every lane, then masked
      x.rel = jj < nlight ? (uint32_t)rj & kSpanMask : 0u;
      x.row = jj < nlight ? wj : 0;
      const int ll = x.row & 0xFF;
#pragma unroll
      for (int h = 0; h < decltype(pieces)::value; ++h) {
        const int t = 16 * h + gl;
        const uint32_t at = x.rel + (t < ll ? t : 0);
        x.c[h] = cb[at];
        x.v[h] = vb[at];
      }
      asm volatile("" ::: "memory");  // keeps the loads here
    };
    auto staged = [&](int32_t c, T v, bool ok, uint32_t& off, float& val) {
      const bool in = ok && (uint32_t)c < (uint32_t)d;
      off = in ? (uint32_t)c * (kGZStride * 4) : 0u;
      val = in ? to_f32<T>(v) : 0.f;
    };
    auto quad_run = [&](const Quad& x, int q, auto pieces) {
      const int mx = __builtin_amdgcn_readlane(longest, n01 + 4 * q);  // of the four groups' rows
      const int ll = x.row & 0xFF;
      float y[4] = {0.f, 0.f, 0.f, 0.f};
      uint32_t off;
      float val;
      staged(x.c[0], x.v[0], gl < ll, off, val);
      group_chunk(Zs, off, val, gl16, y, mx);
      if constexpr (decltype(pieces)::value == 2) {
        staged(x.c[1], x.v[1], 16 + gl < ll, off, val);
        group_chunk(Zs, off, val, gl16, y, mx - 16);
        for (int c0 = 32; c0 < mx; c0 += 16) {
          const int t = c0 + gl;
          const uint32_t at = x.rel + (t < ll ? t : 0);
          staged(cb[at], vb[at], t < ll, off, val);
          group_chunk(Zs, off, val, gl16, y, mx - c0);
        }
      }
      const float sq = group_sum16(y[0] * y[0] + y[1] * y[1] + y[2] * y[2] + y[3] * y[3]);
      if (ll > 0 && gl == 15) store((uint32_t)x.row >> 8, sq);
    };
    auto quads = [&](int q0, int q1, auto pieces) {
      if (q0 >= q1) return;
      Quad x0, x1, x2;
      quad_load(x0, q0, pieces);
      quad_load(x1, q0 + 1, pieces);
      for (int q = q0;; q += 3) {
        quad_load(x2, q + 2, pieces);
        quad_run(x0, q, pieces);
        if (q + 1 >= q1) break;
        quad_load(x0, q + 3, pieces);
        quad_run(x1, q + 1, pieces);
        if (q + 2 >= q1) break;
        quad_load(x1, q + 4, pieces);
        quad_run(x2, q + 2, pieces);
        if (q + 3 >= q1) break;
      }
    };
    // classes 1 .. 4 are at most 16 long: whole steps of them, then the rest
    const int nq = (nlight - n01 + 3) / 4, nshort = n16 == nlight ? nq : (n16 - n01) / 4;
    quads(0, nshort, std::integral_constant<int, 1>());
    quads(nshort, nq, std::integral_constant<int, 2>());

    // heavy rows: the groups' partial k-vectors are added at the end
    float y[4] = {0.f, 0.f, 0.f, 0.f};
    while (heavy != 0) {
      uint32_t off;
      float val;
      const int j = hj, c0 = hc0, lj = hlen;
      staged(hcol, hval, 4 * gl + g < lj - c0, off, val);
      const bool done = c0 + 64 >= lj;
      if (done) heavy &= heavy - 1;
      // the next piece: of this row or of the next (after the last one, the
      // first again, not used)
      heavy_load(done && heavy != 0 ? __builtin_ctzll(heavy) : j, done ? 0 : c0 + 64);
      asm volatile("" ::: "memory");
      group_chunk(Zs, off, val, gl16, y, min(16, (lj - c0 + 3) / 4));
      if (done) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          y[q] += __shfl_xor(y[q], 16, 64);
          y[q] += __shfl_xor(y[q], 32, 64);
        }
        const float sq = group_sum16(y[0] * y[0] + y[1] * y[1] + y[2] * y[2] + y[3] * y[3]);
        if (lane == 15) store(j, sq);
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] = 0.f;
      }
    }
  }
}

template <typename T, typename ZT>
hipError_t launch_typed(const void* vals, const int64_t* row_ptr, const int32_t* col_idx, int64_t n, int64_t d,
                        int64_t nnz, const void* Zpack, void* theta, const ColTile& ct, hipStream_t s) {
  int dev = 0, num_cu = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  err = hipDeviceGetAttribute(&num_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (err != hipSuccess) return err;
  const size_t stage_bytes = sizeof(StageEntry<ZT>) * 64 * kCsrWaves;
  const size_t z_bytes = (size_t)d * kZStride * sizeof(ZT);
  constexpr size_t kMaxLds = 144 * 1024;  // leave room below the 160 KB of a CU
  const T* v = static_cast<const T*>(vals);
  const ZT* Z = static_cast<const ZT*>(Zpack);
  ZT* th = static_cast<ZT*>(theta);
  if constexpr (sizeof(ZT) == 4) {
    const size_t gz = (size_t)d * (kGZStride + 1) * sizeof(float);
    if (gz <= 152 * 1024) {
      auto kern = rownorm_csr_grp_kernel<T>;
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)gz);
      if (e != hipSuccess) return e;
      const int64_t want = ((n + 63) / 64 + kCsrWaves - 1) / kCsrWaves;
      const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, (int64_t)num_cu));
      kern<<<grid, kCsrThreads, gz, s>>>(v, row_ptr, col_idx, n, d, nnz, Z, th, ct);
      return hipGetLastError();
    }
  }
  const bool zlds = stage_bytes + z_bytes <= kMaxLds;
  const size_t lds = zlds ? stage_bytes + z_bytes : stage_bytes;
  // one workgroup per CU holds the LDS copy of Z_full; a second fits when it is small
  const int64_t groups = (int64_t)num_cu * (2 * lds <= kMaxLds ? 2 : 1);
  // A wave works through a task's rows one after the other, so a task's own
  // length bounds the pass until every wave has two: tasks of 64 rows are
  // halved down to 8 till then (16 nonzeros a row, 64 rows and this rule:
  // 325770 x 50 FP64 108 and 72 us, 222824 x 323 FP64 151 and 132, 400001 x
  // 700 FP32 177 and 156; 1900001 x 200 keeps 64 rows, 615)
  int rows = kRowsPerTask;
  while (rows > kMinRowsPerTask && (n + rows - 1) / rows < kTasksPerWave * groups * kCsrWaves) rows /= 2;
  const int64_t want = ((n + rows - 1) / rows + kCsrWaves - 1) / kCsrWaves;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, groups));
  if (zlds) {
    auto kern = rownorm_csr_kernel<T, ZT, true>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kern<<<grid, kCsrThreads, lds, s>>>(v, row_ptr, col_idx, n, d, nnz, Z, th, ct, rows);
  } else {
    rownorm_csr_kernel<T, ZT, false><<<grid, kCsrThreads, lds, s>>>(v, row_ptr, col_idx, n, d, nnz, Z, th, ct, rows);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_rownorm_csr(int dtype, const void* vals, const int64_t* row_ptr, const int32_t* col_idx,
                              int64_t n, int64_t d, int64_t nnz, int64_t k, const void* Zpack,
                              const int64_t* live, void* theta, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int variant = dtype == 0 ? 6 : 5;
  // one pass per column tile of 64 (see launch_rownorm_dense)
  for (int64_t t = 0; t < z_tiles(k); ++t) {
    ColTile ct;
    ct.c0 = t * kZTile;
    ct.acc = t > 0;
    ct.live = t > 0 ? live : nullptr;
    const void* zt = static_cast<const char*>(Zpack) + pack_z_tile_offset(variant, d, k, t);
    hipError_t e = hipErrorInvalidValue;
    switch (dtype) {
      case 0: e = launch_typed<double, double>(vals, row_ptr, col_idx, n, d, nnz, zt, theta, ct, s); break;
      case 1: e = launch_typed<float, float>(vals, row_ptr, col_idx, n, d, nnz, zt, theta, ct, s); break;
      case 2: e = launch_typed<__hip_bfloat16, float>(vals, row_ptr, col_idx, n, d, nnz, zt, theta, ct, s); break;
      default: break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lev
