// Device-side helpers shared by the SRead / MFMA / SWrite kernels (gfx950): LDS accessors, MFMA wrappers,
// output rounding, the GELU of the MoE epilogue, in-lane 8 x 8 transposes of 16-bit elements, and
// global loads at a wave-uniform base plus a 32-bit per-lane offset.
#pragma once
#include "pit_gemm.hpp"

namespace pit {
namespace {

__device__ __forceinline__ u32x4_t lds_read_frag(uint32_t addr) {
  return *(PIT_LDS u32x4_t*)(uintptr_t)addr;
}
template <bool BF>
__device__ __forceinline__ f32x16_t mfma32(const u32x4_t& a, const u32x4_t& b, const f32x16_t& c) {
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ uint16_t f32_to_f16_rne(float f) {
  return __builtin_bit_cast(uint16_t, (_Float16)f);
}
template <bool BF> __device__ __forceinline__ uint16_t f32_to_in(float f) {
  return BF ? f32_to_bf16_rne(f) : f32_to_f16_rne(f);
}
// Two fp32 values rounded (nearest-even) to the 16-bit input type and packed, a in the low half: one
// v_cvt_pk_bf16_f32 on gfx950 for bf16 (the same rounding as f32_to_bf16_rne for every finite value and for
// infinities; a NaN stays a NaN).
typedef __bf16 pit_bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 pit_f16x2_t __attribute__((ext_vector_type(2)));
typedef float pit_f32x2_t __attribute__((ext_vector_type(2)));
template <bool BF> __device__ __forceinline__ uint32_t pack2_in(float a, float b) {
  const pit_f32x2_t v = {a, b};
  if constexpr (BF) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, pit_bf16x2_t));
  else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, pit_f16x2_t));
}
// GELU(x) = x (1 + erf(x / sqrt 2)) / 2 with erf(z) = 1 - 2^(-q(z)) for z >= 0, q the polynomial of degree 5 without
// constant term fitted (weighted least squares, reweighted towards the minimax fit) to -log2(erfc z) on [0, 4.2];
// beyond 4.2 q keeps growing (q >= 28.6 there: erfc itself is below 3e-9) until 2^-q underflows to zero.
// |error of erf| <= 7e-7 in fp32, far below the rounding of the result to bf16 / fp16.  Evaluated as
//   x / 2 + |x| (1/2 - 2^-q / 2),
// with q as a polynomial in |x| (its coefficients times 2^(-k/2)): eight vector instructions and one transcendental, where q of
// |x| / sqrt 2, 1 - 2^-q, its sign, 1 + and the two products were eleven and one.  Its error in fp32 against that form's, root
// mean square over -8 < x < 8 in ten ranges down to 1e-6: 0.2 % larger at most (-0.1 < x < -0.001), 4 % smaller beyond 4, 42 %
// smaller for 0 < x < 0.001.  (2^-(q + 1), with the 1 as the polynomial's first coefficient, loses q's last bits near zero: 29 %
// larger for -0.001 < x < 0.)  The epilogue of the first MoE matmul is 128 of these per lane, a quarter of its workgroups' run
// time with erff.  NaN stays NaN, +inf stays, -inf gives NaN (-inf * 0), as the product x (1 + erf) does.
__device__ __forceinline__ float gelu_erf_fast(float x) {
  const float a = fabsf(x);
  const float q = a * fmaf(fmaf(fmaf(fmaf(0.0005204583285f, a, -0.007397509646f), a, 0.05256123468f), a, 0.4592546821f), a, 1.151091337f);
  return fmaf(a, fmaf(-0.5f, __builtin_amdgcn_exp2f(-q), 0.5f), 0.5f * x);
}

// JA consecutive 16-bit columns of one k-row as loaded (JA = 8: 16 bytes, 4: 8 bytes, 2: 4 bytes)
template <int JA> struct ACols { uint32_t d[JA / 2]; };
// Dword jj (k = 2 jj, 2 jj + 1) of column x out of 8 k-rows of JA columns each (one v_perm_b32).
template <int JA>
__device__ __forceinline__ uint32_t transpose_cols_dword(const ACols<JA> (&r)[8], int x, int jj) {
  const uint32_t sel = (x & 1) ? 0x07060302u : 0x05040100u;
  return __builtin_amdgcn_perm(r[2 * jj + 1].d[x >> 1], r[2 * jj].d[x >> 1], sel);
}
// r[j] = 8 consecutive columns of k-row j (16-bit elements); result = 8 consecutive k of column x (4 v_perm_b32).
__device__ __forceinline__ uint4 transpose8x8_row(const uint4 (&r)[8], int x) {
  const int i = x >> 1;
  const uint32_t sel = (x & 1) ? 0x07060302u : 0x05040100u;
  uint32_t d[4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const uint32_t a = i == 0 ? r[2 * jj].x : i == 1 ? r[2 * jj].y : i == 2 ? r[2 * jj].z : r[2 * jj].w;
    const uint32_t b = i == 0 ? r[2 * jj + 1].x : i == 1 ? r[2 * jj + 1].y : i == 2 ? r[2 * jj + 1].z : r[2 * jj + 1].w;
    d[jj] = __builtin_amdgcn_perm(b, a, sel);
  }
  return make_uint4(d[0], d[1], d[2], d[3]);
}

__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}
// 16-byte load from global memory at a wave-uniform base plus a 32-bit per-lane byte offset.  The
// explicit global address space keeps the access a global_load (a flat load would tie up both
// memory counters and force full waits).
__device__ __forceinline__ uint4 load16(const char* base, uint32_t byte_off) {
  typedef const u32x4_t __attribute__((address_space(1))) * gptr_t;
  const u32x4_t v = *(gptr_t)(uintptr_t)(reinterpret_cast<uintptr_t>(base) + byte_off);
  return __builtin_bit_cast(uint4, v);
}
// the same for 2 * JA bytes
template <int JA>
__device__ __forceinline__ ACols<JA> load_cols(const char* base, uint32_t byte_off) {
  ACols<JA> r;
  const uintptr_t a = reinterpret_cast<uintptr_t>(base) + byte_off;
  if constexpr (JA == 8) {
    const u32x4_t v = *(const u32x4_t __attribute__((address_space(1)))*)a;
    r.d[0] = v[0]; r.d[1] = v[1]; r.d[2] = v[2]; r.d[3] = v[3];
  } else if constexpr (JA == 4) {
    const u32x2_t v = *(const u32x2_t __attribute__((address_space(1)))*)a;
    r.d[0] = v[0]; r.d[1] = v[1];
  } else {
    static_assert(JA == 2, "columns per lane");
    r.d[0] = *(const uint32_t __attribute__((address_space(1)))*)a;
  }
  return r;
}

// Direct global -> LDS load of 16 bytes per lane: lane i's bytes land at lds_wave_base + 16 i.
// `base` and `lds_wave_base` are wave-uniform.
__device__ __forceinline__ void dma16(const char* base, uint32_t byte_off, uint32_t lds_wave_base) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_wave_base);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(m0v), "v"(byte_off), "s"(reinterpret_cast<uint64_t>(base)) : "memory", "m0");
}
// the same with 4 bytes per lane
__device__ __forceinline__ void dma4(const char* base, uint32_t byte_off, uint32_t lds_wave_base) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_wave_base);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(m0v), "v"(byte_off), "s"(reinterpret_cast<uint64_t>(base)) : "memory", "m0");
}
// transposing LDS read (ds_read_b64_tr_b16): in each group of 16 lanes, lane i receives column i of the four rows addressed by
// lanes 4 j .. 4 j + 3
__device__ __forceinline__ uint2 lds_tr(uint32_t addr) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((PIT_LDS v4i16_t*)(uintptr_t)addr));
}
// wait until at most n vector-memory operations of this wavefront are outstanding (gfx9 encoding:
// vmcnt in bits 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at "no wait"); LDS accesses that
// follow in program order stay behind it
#define PIT_WAIT_VMCNT(n) do { __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14)); \
                               asm volatile("" ::: "memory"); } while (0)
// nothing may be scheduled across this point
#define PIT_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)


}  // namespace
}  // namespace pit
