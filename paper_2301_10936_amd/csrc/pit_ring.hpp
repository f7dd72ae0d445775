// What the kernels with a ring in LDS per wave share (pit_gemm_ring.hip, pit_gemm_m_ring.hip; gfx950): the layout of a K-major
// operand's slab for transposing reads, and of a wave's partial tile where the waves meet.
#pragma once
#include "pit_gemm_dev.hpp"

namespace pit {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <bool BF>
__device__ __forceinline__ f32x4_t mfma16r(const u32x4_t& a, const u32x4_t& b, const f32x4_t& c) {
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

// One operand's slab in LDS: 32 rows ("slots") of T columns
template <int T> struct SlabLayout {
  static_assert(T == 32 || T == 64, "columns of a tile");
  static constexpr int BYTES = 32 * T * 2, LOADS = BYTES / 1024;
  static constexpr int LPR = T / 8, RPI = 64 / LPR;        // lanes per row, rows per load instruction
  // swizzle of the 32-byte chunks of a row
  static __device__ __forceinline__ int f(int slot) { return T == 64 ? ((slot >> 1) & 1) | (((slot >> 3) & 1) << 1) : (slot >> 3) & 1; }
};

// Partial tiles in LDS: vector (row m, columns 4 c .. 4 c + 3) of a tile of TB columns and 16 FA rows.  Block (c / 4, m / 16), 256
// bytes per c % 4 in it, 16 bytes at a place that differs both for the 16 rows of a block and for the vectors of a row, so that
// neither the writes (a lane holds row lane % 16, vector lane / 16 of a block) nor the reads (lanes along a row) meet on a bank.
template <int TB, int FA>
__device__ __forceinline__ uint32_t partial_place(int m, int c) {
  const int x = (m & 15) ^ (c & 15) ^ (TB == 32 ? (m & 1) << 3 : 0);
  return (uint32_t)(((c >> 2) * FA + (m >> 4)) * 1024 + (c & 3) * 256 + x * 16);
}

}  // namespace
}  // namespace pit
