// Staging of a tall row-major A through LDS, for the kernels that contract
// over its rows on the FP64 matrix cores: a step is ROWS rows of 64 TB
// columns, loaded by the whole workgroup as 16-byte pieces (held in registers
// while the step before is worked on) and stored with rows padded by 16
// elements, which puts the four rows of an MFMA operand read on different
// banks.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lev {

constexpr int tall_stride(int tb) { return 64 * tb + 16; }

// What LDS holds of an element: BF16 is widened to FP32 when staged, the rest
// to FP64 when read.
template <typename TI>
using tall_lds_t = std::conditional_t<std::is_same_v<TI, double>, double, float>;

template <typename TI, int TB, int ROWS, int THREADS>
struct TallStep {  // a thread's part of a step: 16-byte pieces of A
  static constexpr int kElts = 16 / (int)sizeof(TI);
  static constexpr int kPieces = (ROWS * 64 * TB / kElts + THREADS - 1) / THREADS;
  uint4 v[kPieces];
};

template <typename TI, int TB, int ROWS, int THREADS>
__device__ __forceinline__ void tall_load(TallStep<TI, TB, ROWS, THREADS>& r, const TI* __restrict__ A, int64_t k0,
                                          int64_t ke, int d, int64_t ld) {
  using R = TallStep<TI, TB, ROWS, THREADS>;
  constexpr int per = 64 * TB / R::kElts;  // pieces per row
#pragma unroll
  for (int q = 0; q < R::kPieces; ++q) {
    const int e = threadIdx.x + THREADS * q;
    const int c = (e % per) * R::kElts;
    const int64_t row = k0 + e / per;
    // No branch and no select on what is loaded, so that nothing waits for it
    // here: a piece past the rows or columns reads the step's first.  Rows are
    // 16-byte multiples, so a piece that starts below d ends below ld; what it
    // holds past d reaches only outputs past d, which are not stored.
    const int64_t at = (row < ke ? row : k0) * ld + (c < d ? c : 0);
    r.v[q] = *reinterpret_cast<const uint4*>(A + at);
  }
}

// rows: how many rows of the step there are (the rest is stored as zeros).
template <typename TI, int TB, int ROWS, int THREADS>
__device__ __forceinline__ void tall_store(const TallStep<TI, TB, ROWS, THREADS>& r, int64_t rows,
                                           tall_lds_t<TI>* __restrict__ L) {
  using R = TallStep<TI, TB, ROWS, THREADS>;
  constexpr int per = 64 * TB / R::kElts, stride = tall_stride(TB);
#pragma unroll
  for (int q = 0; q < R::kPieces; ++q) {
    const int e = threadIdx.x + THREADS * q;
    if (R::kPieces * THREADS > ROWS * per && e >= ROWS * per) continue;
    const uint4 x = e / per < rows ? r.v[q] : uint4{0, 0, 0, 0};
    tall_lds_t<TI>* dst = L + (e / per) * stride + (e % per) * R::kElts;
    if constexpr (std::is_same_v<TI, __hip_bfloat16>) {
      const uint32_t w[4] = {x.x, x.y, x.z, x.w};
      float f[8];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        f[2 * h] = __uint_as_float(w[h] << 16);
        f[2 * h + 1] = __uint_as_float(w[h] & 0xffff0000u);
      }
      reinterpret_cast<float4*>(dst)[0] = make_float4(f[0], f[1], f[2], f[3]);
      reinterpret_cast<float4*>(dst)[1] = make_float4(f[4], f[5], f[6], f[7]);
    } else {
      *reinterpret_cast<uint4*>(dst) = x;
    }
  }
}

}  // namespace lev
