// pit_sread_gemm: the SRead -> dense MFMA tile -> SWrite kernels (paper Section 3.1, sparse kernel
// template) for gfx950 with k as the PIT-axis, and the host-side validation and launch of all GEMM modes.  bf16 or f16 inputs, fp32 accumulation.
// There is one kernel per PIT-axis of MatMul (paper Table 1):
//
//   k_gather_k_direct  GATHER_K: A is K-major (At[k][m]); the tile's k-list comes from the index and
//             names the rows of At and of B to multiply.  Operands go global -> registers directly
//             and are transposed inside each lane; the waves of a workgroup split the k-list and
//             reduce their partial tiles through LDS at the end (details above the kernel).
//             Tiles of 128, 64 or 32 rows x 128 columns (at most the height of the micro-tile).
//   k_gather_k_ring (pit_gemm_ring.hip)  the same product with few tiles: up to 64 x 64, eight waves, rings in LDS.
//   k_slab_strip, k_slab_strip_tall (pit_slab.hip)  GATHER_M with several k-slabs per row (1 x mt micro-tiles of a
//             row-major A): a strip of C stays in LDS while the listed rows of every slab are added to it.
//   k_gather_m_lds (pit_gemm_m.hip)  GATHER_M with whole-row micro-tiles (padded batches, MoE): the
//             tile's row numbers come from the index once, operands are staged through LDS.
//
// SWrite.  GATHER_K writes the rows of its m-tile in place.
#include "pit_gemm.hpp"
#include "pit_gemm_dev.hpp"
#include <type_traits>
#include <algorithm>
#include <climits>

namespace pit {
namespace {

// ------------------------------------------------------------------------------------------------
// GATHER_K, register-direct: no LDS and no barrier inside the k loop.
//
// Both operands of GATHER_K are K-major (rows of At and of B), and an MFMA operand register holds
// 8 consecutive k of ONE column.  A lane that loads 16 bytes (8 columns) from each of 8 listed
// rows owns an 8 k x 8 column block, and transposing that block inside the lane (v_perm_b32, no
// cross-lane traffic) yields 8 operand registers, one per column.  With v_mfma_f32_16x16x32 (lane
// l: column l % 16, k-block l / 16) 16 lanes x 8 columns cover 128 columns, so a wavefront's 8
// loads of At give it the A operands of all 128 tile rows for 32 k, its 8 loads of B the B
// operands of all 128 tile columns, and 8 x 8 MFMAs consume them: MFMA (ja, jb) works on the
// strided row set {8r + ja} and column set {8c + jb}.  Each operand byte travels global -> register
// exactly once per workgroup and never through LDS.
// The four wavefronts split the tile's k-list in slabs of 32 entries (wave w takes slabs w, w+4, ..),
// each accumulating a full 128 x 128 partial tile in 256 accumulator registers; at the end the
// partial tiles are reduce-scattered through LDS (4 rounds of 48 KiB) and every wave stores a
// quarter of the tile, 512 contiguous bytes per row.  With more tiles than compute units a workgroup
// loops over tiles.
// The k loop is branch-free: list positions past the end are clamped to the last entry on load, the
// last slab of each wave is processed apart with the clamped rows zeroed.
// ------------------------------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// acc += A * B with v_mfma_f32_16x16x32.  Written as inline assembly so that the accumulator is
// updated IN PLACE in an accumulation register: with all 256 of them live the register allocator
// otherwise gives the result a different register than the input and shuffles accumulators
// through vector registers between MFMAs.  The assembly is opaque to the compiler's hazard
// handling: callers must leave 64 other MFMAs (or PIT_MFMA_DRAIN) between an update of an
// accumulator and its next use.
template <bool BF>
__device__ __forceinline__ void mfma16_acc(const uint4& a, const uint4& b, f32x4_t& c) {
  const u32x4_t av = __builtin_bit_cast(u32x4_t, a), bv = __builtin_bit_cast(u32x4_t, b);
  if constexpr (BF) asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(av), "v"(bv));
  else              asm("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(av), "v"(bv));
}
// acc = z z + 0 (z = zeros), in place as well and under the same rules
__device__ __forceinline__ void mfma16_zero(const u32x4_t& z, f32x4_t& c) {
  asm("v_mfma_f32_16x16x32_bf16 %0, %1, %1, 0" : "+a"(c) : "v"(z));
}
// wait until the matrix pipe has written every accumulator (a 4-pass MFMA needs at most 10 idle
// issue slots before another kind of instruction may read its result)
#define PIT_MFMA_DRAIN() do { PIT_SCHED_FENCE(); asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); PIT_SCHED_FENCE(); } while (0)

constexpr int RED_SLOT_BYTES = 16 * 64 * 16;        // 16 accumulator quads x 64 lanes x 16 B
constexpr int RED_BUF_BYTES = 4 * RED_SLOT_BYTES;   // one slot per sending wave

// LDS accesses of the wave's lanes before this point are done before those after it (the hardware keeps a wave's LDS
// accesses in order; this keeps the compiler from exchanging accesses of different lanes that no single lane sees meet)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// Round P of the reduction: the partial sums of tile rows {8r + ja : ja in {2P, 2P + 1}} go to wave
// P.  P is a compile-time constant so that every accumulator index is static.
template <int P>
__device__ __forceinline__ void red_send(const f32x4_t (&acc)[8][8], PIT_LDS char* buf, int wv, int lane) {
  PIT_LDS char* slot = buf + wv * RED_SLOT_BYTES + lane * 16;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) *(PIT_LDS f32x4_t*)(slot + (a * 8 + jb) * 1024) = acc[2 * P + a][jb];
}
// Wave P adds the three other waves' partial sums to its own.
template <int P>
__device__ __forceinline__ void red_recv(f32x4_t (&acc)[8][8], PIT_LDS char* buf, int lane) {
  // (all 16 reads of one sender are issued before the first addition: one LDS latency per sender
  // instead of one per read)
#pragma unroll
  for (int o = 1; o < 4; ++o) {
    PIT_LDS char* slot = buf + ((P + o) & 3) * RED_SLOT_BYTES + lane * 16;
    f32x4_t part[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) part[i] = *(PIT_LDS f32x4_t*)(slot + i * 1024);
    PIT_SCHED_FENCE();
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[2 * P + (i >> 3)][i & 7] += part[i];
    PIT_SCHED_FENCE();
  }
}
// Two-wave workgroups: half H of the tile = the row groups ja in {H * JA / 2 .. (H + 1) * JA / 2 - 1}
// (JA = row groups of the tile = tile rows / 16).
template <int JA> constexpr int red_half_bytes() { return 4 * JA * 64 * 16; }
template <int JA, int H>
__device__ __forceinline__ void red_send_half(const f32x4_t (&acc)[JA][8], PIT_LDS char* slot) {
#pragma unroll
  for (int i = 0; i < 4 * JA; ++i) *(PIT_LDS f32x4_t*)(slot + i * 1024) = acc[(JA / 2) * H + (i >> 3)][i & 7];
}
template <int JA, int H>
__device__ __forceinline__ void red_recv_half(f32x4_t (&acc)[JA][8], PIT_LDS char* slot) {
  constexpr int CH = 4 * JA < 16 ? 4 * JA : 16;     // reads issued together, ahead of their additions
#pragma unroll
  for (int a = 0; a < 4 * JA / CH; ++a) {
    f32x4_t part[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) part[i] = *(PIT_LDS f32x4_t*)(slot + (a * CH + i) * 1024);
    PIT_SCHED_FENCE();
#pragma unroll
    for (int i = 0; i < CH; ++i) acc[(JA / 2) * H + ((a * CH + i) >> 3)][(a * CH + i) & 7] += part[i];
    PIT_SCHED_FENCE();
  }
}
// Store the row groups ja in [J0, J0 + NJ) of the tile: rows JA * (4 * (lane / 16) + e) + ja; a lane holds 8
// consecutive columns of such a row (one per jb): 16 lanes write 256 contiguous bytes of 16-bit results.  Of fp32
// results a lane's 32 bytes are two stores, i.e. two instructions that each leave every second 16 bytes of a row to
// the other.  Where workgroups store tile after tile (at most two waves per tile) these half-filled lines are what the
// memory sees, so there the rows go through 4 KiB of LDS of the wave (STAGED) and an instruction stores two whole rows:
// 4096^3, live in runs of 32 at 10 %: 128-row tiles 55.5 -> 47.7 us, 64 rows 49.4 -> 39.9, 32 rows 47.5 -> 42.5 (without
// any store 41, 34, 37); 2944 x 3001 x 3072, full lists, 79.4 -> 75.4.  With four waves per tile, one or two tiles per
// compute unit, the way through LDS costs what it gains (2048 x 8192 x 2048: 58.4 and 58.9).
constexpr int STAGE_OUT_BYTES = 4096;              // two rows sets (four rows x 512 bytes each), used in turn
// PART: with has_part another partial tile of the lane (quad (ja, jb) at part + 1024 (8 ja + jb)) is added first.
template <bool BF, int CT, int JA, int J0, int NJ, bool STAGED = false, bool PART = false>
__device__ __forceinline__ void red_store(f32x4_t (&acc)[JA][8], const GemmArgs& g, int m_base, int n0, int lane, PIT_LDS char* stage = nullptr,
                                          bool has_part = false, PIT_LDS char* part = nullptr) {
  const int q = lane & 15, kb = lane >> 4;
#pragma unroll
  for (int a = 0; a < NJ; ++a) {
    const int ja = J0 + a;
    if constexpr (PART) {
      if (has_part) {
#pragma unroll
        for (int jb = 0; jb < 8; ++jb) acc[ja][jb] += *(PIT_LDS f32x4_t*)(part + (8 * ja + jb) * 1024 + lane * 16);
      }
      PIT_SCHED_FENCE();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t row = m_base + JA * (4 * kb + e) + ja;
      const int col = n0 + 8 * q;
      if constexpr (CT == 0 && STAGED) {
        PIT_LDS char* s = stage + ((a * 4 + e) & 1) * (STAGE_OUT_BYTES / 2);   // row kb of the four at 512 kb
        *(PIT_LDS f32x4_t*)(s + lane * 32) = f32x4_t{acc[ja][0][e], acc[ja][1][e], acc[ja][2][e], acc[ja][3][e]};
        *(PIT_LDS f32x4_t*)(s + lane * 32 + 16) = f32x4_t{acc[ja][4][e], acc[ja][5][e], acc[ja][6][e], acc[ja][7][e]};
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4_t v = *(PIT_LDS f32x4_t*)(s + i * 1024 + lane * 16);
          const int64_t r = m_base + JA * (4 * (2 * i + (lane >> 5)) + e) + ja;
          __builtin_nontemporal_store(v, reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(g.C) + r * g.ldc + n0 + 4 * (lane & 31)));
        }
        wave_lds_fence();
      } else if constexpr (CT == 0) {
        // (streaming stores: the result is not read again by this kernel and should not displace the
        // operand panels from L2)
        typedef float f4_t __attribute__((ext_vector_type(4)));
        f4_t* d = reinterpret_cast<f4_t*>(reinterpret_cast<float*>(g.C) + row * g.ldc + col);
        __builtin_nontemporal_store(f4_t{acc[ja][0][e], acc[ja][1][e], acc[ja][2][e], acc[ja][3][e]}, d);
        __builtin_nontemporal_store(f4_t{acc[ja][4][e], acc[ja][5][e], acc[ja][6][e], acc[ja][7][e]}, d + 1);
      } else {
        uint32_t w[4];
#pragma unroll
        for (int x = 0; x < 4; ++x)
          w[x] = pack2_in<BF>(acc[ja][2 * x][e], acc[ja][2 * x + 1][e]);
        __builtin_nontemporal_store(u32x4_t{w[0], w[1], w[2], w[3]},
                                    reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(g.C) + row * g.ldc + col));
      }
    }
  }
}

// Four waves on a low tile: vector ((ja * 4 + e) * 2 + h) of a wave's slot = columns 4 h .. 4 h + 3 of the
// rows JA * (4 * (lane / 16) + e) + ja.
template <int JA>
__device__ __forceinline__ void red_send_all(const f32x4_t (&acc)[JA][8], PIT_LDS char* slot) {
#pragma unroll
  for (int ja = 0; ja < JA; ++ja)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *(PIT_LDS f32x4_t*)(slot + ((ja * 4 + e) * 2 + h) * 1024) = f32x4_t{acc[ja][4 * h][e], acc[ja][4 * h + 1][e], acc[ja][4 * h + 2][e], acc[ja][4 * h + 3][e]};
}
template <bool BF, int CT, int NW, int JA>
__device__ __forceinline__ void red_sum_store(PIT_LDS char* red, const GemmArgs& g, int m_base, int n0, int wv, int lane) {
  constexpr int U = 4 * JA / NW;                    // row sets (ja, e) of a wave
  const int q = lane & 15, kb = lane >> 4;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int unit = wv * U + u;
    f32x4_t part[NW][2];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int h = 0; h < 2; ++h) part[w][h] = *(PIT_LDS f32x4_t*)(red + w * (JA * 8 * 1024) + (unit * 2 + h) * 1024);
    f32x4_t s[2] = {part[0][0], part[0][1]};
#pragma unroll
    for (int w = 1; w < NW; ++w) { s[0] += part[w][0]; s[1] += part[w][1]; }
    const int64_t row = m_base + JA * (4 * kb + (unit & 3)) + (unit >> 2);
    const int col = n0 + 8 * q;
    if constexpr (CT == 0) {
      f32x4_t* d = reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(g.C) + row * g.ldc + col);
      __builtin_nontemporal_store(s[0], d);
      __builtin_nontemporal_store(s[1], d + 1);
    } else {
      __builtin_nontemporal_store(u32x4_t{pack2_in<BF>(s[0][0], s[0][1]), pack2_in<BF>(s[0][2], s[0][3]), pack2_in<BF>(s[1][0], s[1][1]), pack2_in<BF>(s[1][2], s[1][3])},
                                  reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(g.C) + row * g.ldc + col));
    }
  }
}

// what a wave needs to know about one tile
struct DirectTile {
  int row, n0, list_len, n_w;      // tile row, first column, length of the k-list, this wave's slabs
  const char* list;                // the k-list
  uint32_t a_col, b_col;           // this lane's byte offsets into a row of At and of B
};

// NW = waves per workgroup that split the k-list: 4 (one 128-row tile fills a compute unit), 2 (two
// workgroups, i.e. two tiles, share a compute unit at the same register cost, and the set-up, drain,
// reduction and stores of one tile run under the MFMA loop of the other) or 1 (no reduction between waves).
// One wave sums the first half of its slabs, puts that partial tile away in LDS, sums the other half and adds the two:
// chains of additions as long as those of two waves.  (One chain over all slabs has up to 1.4 times their rounding error:
// 4096^3, half live, 32-row tiles 1.05e-7 of the result, 7.8e-8 with two chains and with two waves.)
// JA = row groups of the tile: the tile is 16 * JA rows high (128, 64 or 32), a lane loads JA consecutive m of
// each listed row of At (16, 8 or 4 bytes) and a slab takes JA x 8 MFMAs.  Lower tiles follow a finer sparsity
// pattern (the micro-tile height of the index; fewer all-zero micro-tiles are multiplied) or spread a small
// product over more compute units, and pay for it with more traffic of B per row of C.  The rule that chooses is at
// launch_gather_k.
template <bool BF, int CT, int NW, int JA>
__global__ void __launch_bounds__(64 * NW, JA == 2 ? 2 : 1)
k_gather_k_direct(const GemmArgs g, const int tm_tiles) {
  static_assert((JA == 8 && (NW == 2 || NW == 4)) || (JA == 4 && (NW == 1 || NW == 2 || NW == 4)) ||
                (JA == 2 && (NW == 1 || NW == 2 || NW == 4)), "tile heights and waves");
  constexpr int SK = 32;   // list entries per slab = k extent of one MFMA
  constexpr int TMJ = 16 * JA;   // tile rows
  constexpr int RED_HALF_BYTES = red_half_bytes<JA>();
  constexpr int RED_ALL_BYTES = 2 * RED_HALF_BYTES;   // one wave's whole partial tile
  constexpr bool RED_QUARTERS = NW == 4 && JA == 8;
  __shared__ __attribute__((aligned(16)))
  char s_red[NW == 1 ? RED_ALL_BYTES : RED_QUARTERS ? 2 * RED_BUF_BYTES : NW == 2 ? 2 * RED_HALF_BYTES : NW * RED_ALL_BYTES];
  __shared__ __attribute__((aligned(16))) char s_out[CT == 0 && NW <= 2 ? NW * STAGE_OUT_BYTES : 16];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  PIT_LDS char* stage = (PIT_LDS char*)s_out + (CT == 0 && NW <= 2 ? wv * STAGE_OUT_BYTES : 0);
  const int q = lane & 15, kb = lane >> 4;
  const char* a_src = uniform_ptr(g.A);
  const char* b_src = uniform_ptr(g.B);
  const uint32_t pitch_a = (uint32_t)(g.lda * 2), pitch_b = (uint32_t)(g.ldb * 2);

  // The grid is one-dimensional and may hold fewer workgroups than there are tiles: a workgroup then
  // works through tiles lin = blockIdx.x, blockIdx.x + gridDim.x, ... (gridDim.x is a multiple of 8
  // in that case, so all of them belong to the same XCD).
  const int tn = g.N / TN, total = tn * tm_tiles;
  // Consecutive workgroup ids go to different XCDs (8, each with its own L2): renumber so that each
  // XCD works on a contiguous run of tiles, ordered in bands of 4 tile columns x all tile rows.  What an XCD
  // fetches into its L2 per step of k is then 4 x 128 columns of B and the listed share of its rows of At; bands of
  // 4 tile rows x all columns fetch (almost) the union of 4 lists of B over all columns instead, and that traffic, not
  // the MFMAs, bounded sparse products (4096^3, live in runs of 32 tokens with probability 0.1: 32-row tiles 79.8 us
  // there, 48.5 here; 64 rows 69.2, 53.6; 128 rows 61.6, 55.4; full lists: the same).  Bands of 2 columns are 5 % better
  // for 32-row tiles at that density and 7 % worse at 50 %, bands of 8 columns 17 % and 6 % worse;
  // where tiles are few along m (8 x 32 tiles, 1024 x 16384 x 4096 half listed) rows are better by 1 %.
  const bool dense = g.idx == nullptr;
  const bool wide = tn > 2 * tm_tiles;
  // 1, 2 or 4 tiles share one list (the tile may be lower than the micro-tile)
  const int sub_shift = JA == 8 ? 0 : __builtin_ctz((unsigned)g.slab / (unsigned)TMJ);
  auto tile_of = [&](int lin) -> DirectTile {
    const int x = lin & 7, qq = total >> 3, rr = total & 7;
    const int lp = x * qq + min(x, rr) + (lin >> 3);
    DirectTile t;
    constexpr int G = 4;
    const int across = wide ? tn : tm_tiles, along = wide ? tm_tiles : tn;   // a band: G of `along` x all of `across`
    const int band = lp / (G * across), within = lp - band * (G * across), n = min(G, along - band * G);
    const int thin = band * G + within % n, len = within / n;
    t.row = wide ? thin : len;
    t.n0 = (wide ? len : thin) * TN;
    // dense mode (no index): every tile's list is 0, 1, .., K - 1 and is never read from memory
    const int seg = t.row >> sub_shift;
    const int list_begin = dense ? 0 : g.seg_ptr[seg];
    t.list_len = dense ? g.K : g.seg_ptr[seg + 1] - list_begin;
    const int nslab = (t.list_len + SK - 1) / SK;
    t.n_w = nslab > wv ? (nslab - wv + NW - 1) / NW : 0;   // this wave's slabs: wv, wv + NW, ...
    t.list = uniform_ptr(g.idx + list_begin);
    t.a_col = (uint32_t)(t.row * TMJ + JA * q) * 2u;
    t.b_col = (uint32_t)(t.n0 + 8 * q) * 2u;
    return t;
  };

  // lane l of a slab's list load holds entry (l % 32) of the slab
  auto load_list = [&](const DirectTile& T, int t) -> int {
    const int pos = min(SK * (wv + NW * t) + (lane & 31), T.list_len - 1);
    if (dense) return pos;
    typedef const int __attribute__((address_space(1))) * gint_t;
    return *(gint_t)(uintptr_t)(reinterpret_cast<uintptr_t>(T.list) + (uint32_t)pos * 4u);
  };
  // rows k(8 kb + i), i = 0..7, of At and of B
  auto issue = [&](const DirectTile& T, int kraw, ACols<JA> (&ra)[8], uint4 (&rb)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t k = (uint32_t)__builtin_amdgcn_ds_bpermute((8 * kb + i) * 4, kraw);
      ra[i] = load_cols<JA>(a_src, __umul24(k, pitch_a) + T.a_col);
      rb[i] = load16(b_src, __umul24(k, pitch_b) + T.b_col);
    }
  };

  f32x4_t acc[JA][8];
#pragma unroll
  for (int i = 0; i < JA; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // A wave on its own puts the sums of the first half of its slabs away in LDS.  The accumulators are then set to zero by
  // the matrix pipe: written by vector instructions, in a branch inside the loop, they come out in other registers, and
  // the kernel spills.
  auto half_done = [&](const DirectTile& T, int done) {
    if constexpr (NW == 1) {
      if (done == T.n_w >> 1) {
        u32x4_t z = {0u, 0u, 0u, 0u};
        asm volatile("" : "+v"(z));
        PIT_MFMA_DRAIN();
#pragma unroll
        for (int i = 0; i < JA; ++i)
#pragma unroll
          for (int j = 0; j < 8; ++j) *(PIT_LDS f32x4_t*)((PIT_LDS char*)s_red + (8 * i + j) * 1024 + lane * 16) = acc[i][j];
        PIT_SCHED_FENCE();
#pragma unroll
        for (int i = 0; i < JA; ++i)
#pragma unroll
          for (int j = 0; j < 8; ++j) mfma16_zero(z, acc[i][j]);
        PIT_SCHED_FENCE();
      }
    }
  };

  // JA x 8 MFMAs on one slab (64 for the 128-row tile, which the description below is written for).  All B operands are transposed first; the A operand of column group
  // ja + 1 is transposed (4 v_perm_b32) in the shadow of the first MFMAs of group ja.  The order is
  // pinned: an MFMA must not read a register in the issue slot right after a vector instruction
  // wrote it, and the inline-assembly MFMAs are invisible to the compiler's hazard handling, so
  // every operand is produced at least four MFMAs (or the explicit s_nop) before its first use.
  // ISSUE: the loads of the slab two ahead (list entries in kraw) are issued from inside the MFMA
  // sequence as soon as their registers are free: the B rows during column groups 0..3 (rb is dead
  // once the B operands are transposed), the A rows during group 7 (ra is dead once the last A
  // operand is transposed).  Spreading them keeps 16 to 24 loads of a wave in flight; with 32 in
  // flight at once the load path of a CU runs at less than half its rate (measured).  (Lower tiles: the B
  // rows during the second half of every column group but the last, the A rows during the last group.)
  auto process_impl = [&](const DirectTile& T, ACols<JA> (&ra)[8], uint4 (&rb)[8], int kraw, auto issue_tag) {
    constexpr bool ISSUE = decltype(issue_tag)::value;
    uint4 bfr[8];
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) bfr[jb] = transpose8x8_row(rb, jb);
    uint32_t af[4], afn[4] = {0, 0, 0, 0};
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) af[jj] = transpose_cols_dword<JA>(ra, 0, jj);
    uint32_t kk[8];
    if constexpr (ISSUE) {
#pragma unroll
      for (int i = 0; i < 8; ++i) kk[i] = (uint32_t)__builtin_amdgcn_ds_bpermute((8 * kb + i) * 4, kraw);
    }
    PIT_SCHED_FENCE();
    asm volatile("s_nop 7");
    PIT_SCHED_FENCE();
#pragma unroll
    for (int ja = 0; ja < JA; ++ja) {
#pragma unroll
      for (int jb = 0; jb < 8; ++jb) {
        mfma16_acc<BF>(make_uint4(af[0], af[1], af[2], af[3]), bfr[jb], acc[ja][jb]);
        if (ja < JA - 1 && jb < 4) afn[jb] = transpose_cols_dword<JA>(ra, ja + 1, jb);
        if constexpr (ISSUE) {
          if constexpr (JA >= 4) {
            if (ja < 4 && (jb == 4 || jb == 6)) {
              const int i = ja * 2 + ((jb - 4) >> 1);
              rb[i] = load16(b_src, __umul24(kk[i], pitch_b) + T.b_col);
            }
          } else {
            if (jb >= 4) {   // JA == 2: 8 loads in the second halves of the two column groups
              const int i = ja * 4 + (jb - 4);
              rb[i] = load16(b_src, __umul24(kk[i], pitch_b) + T.b_col);
            }
          }
          // (the A rows of the next-but-one slab may only replace ra once the last A operand of this
          // slab has been taken out of it: during the last column group)
          if (ja == JA - 1) ra[jb] = load_cols<JA>(a_src, __umul24(kk[jb], pitch_a) + T.a_col);
        }
        PIT_SCHED_FENCE();
      }
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) af[jj] = afn[jj];
    }
  };
  auto process = [&](const DirectTile& T, ACols<JA> (&ra)[8], uint4 (&rb)[8]) { process_impl(T, ra, rb, 0, std::false_type{}); };
  auto process_issue = [&](const DirectTile& T, ACols<JA> (&ra)[8], uint4 (&rb)[8], int kraw) { process_impl(T, ra, rb, kraw, std::true_type{}); };
  // local slab t with the rows of positions past the end of the list zeroed
  auto process_last = [&](const DirectTile& T, int t, ACols<JA> (&ra)[8], uint4 (&rb)[8]) {
    const int p0 = SK * (wv + NW * t) + 8 * kb;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (p0 + i >= T.list_len) {
#pragma unroll
        for (int d = 0; d < JA / 2; ++d) ra[i].d[d] = 0u;
        rb[i] = make_uint4(0, 0, 0, 0);
      }
    process(T, ra, rb);
  };

  // With several tiles per workgroup the next tile's description and the list entries of its first
  // two slabs are fetched ahead of the current tile's reduction, so that only the row loads remain
  // between two tiles.
  ACols<JA> ra0[8], ra1[8];
  uint4 rb0[8], rb1[8];
  PIT_LDS char* red = (PIT_LDS char*)s_red;
  int lin = blockIdx.x;
  DirectTile T = tile_of(lin);
  int k0 = 0, k1 = 0;
  if (T.n_w > 0) { k0 = load_list(T, 0); k1 = load_list(T, 1); }
  for (;;) {
    if (T.n_w > 0) {
      // (the fences keep the list loads of slabs 2 and 3 ahead of the second slab's data loads: the
      // memory counter retires in order, so a list load issued last would make the loop wait for all)
      PIT_SCHED_FENCE();
      issue(T, k0, ra0, rb0); k0 = load_list(T, 2); PIT_SCHED_FENCE();
      issue(T, k1, ra1, rb1); k1 = load_list(T, 3); PIT_SCHED_FENCE();
      int t = 0;
      for (; t + 2 < T.n_w; t += 2) {
        process_issue(T, ra0, rb0, k0); k0 = load_list(T, t + 4); PIT_SCHED_FENCE();
        half_done(T, t + 1);
        process_issue(T, ra1, rb1, k1); k1 = load_list(T, t + 5); PIT_SCHED_FENCE();
        half_done(T, t + 2);
      }
      if (T.n_w - t == 2) {
        process(T, ra0, rb0);
        half_done(T, t + 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) { ra0[i] = ra1[i]; rb0[i] = rb1[i]; }
        ++t;
      }
      process_last(T, t, ra0, rb0);
      PIT_MFMA_DRAIN();
    }
    const int lin_next = lin + (int)gridDim.x;
    const bool more = lin_next < total;
    DirectTile Tn = T;
    if (more) {
      Tn = tile_of(lin_next);
      if (Tn.n_w > 0) { k0 = load_list(Tn, 0); k1 = load_list(Tn, 1); }
    }
    PIT_SCHED_FENCE();

    const int m_base = T.row * TMJ;
    if constexpr (NW == 1) {
      red_store<BF, CT, JA, 0, JA, true, true>(acc, g, m_base, T.n0, lane, stage, T.n_w > 1, red);
    } else if constexpr (!RED_QUARTERS && NW > 2) {
      // Every wave leaves its whole partial tile in LDS as the vectors of four columns that are stored later; each then
      // adds up, in the order of the waves, and stores an NW-th of the tile.
      __syncthreads();
      red_send_all<JA>(acc, red + wv * RED_ALL_BYTES + lane * 16);
      __syncthreads();
      red_sum_store<BF, CT, NW, JA>(red + lane * 16, g, m_base, T.n0, wv, lane);
    } else if constexpr (NW == 4) {
      // Reduction across the four waves, one quarter of the tile rows per round, double-buffered in
      // LDS: round P's partial sums are written before barrier P and read by wave P after it, while the
      // other waves already write round P + 1 into the other buffer.
      if (wv != 0) red_send<0>(acc, red, wv, lane);
      __syncthreads();
      if (wv == 0) { red_recv<0>(acc, red, lane); red_store<BF, CT, 8, 0, 2>(acc, g, m_base, T.n0, lane); }
      if (wv != 1) red_send<1>(acc, red + RED_BUF_BYTES, wv, lane);
      __syncthreads();
      if (wv == 1) { red_recv<1>(acc, red + RED_BUF_BYTES, lane); red_store<BF, CT, 8, 2, 2>(acc, g, m_base, T.n0, lane); }
      if (wv != 2) red_send<2>(acc, red, wv, lane);
      __syncthreads();
      if (wv == 2) { red_recv<2>(acc, red, lane); red_store<BF, CT, 8, 4, 2>(acc, g, m_base, T.n0, lane); }
      if (wv != 3) red_send<3>(acc, red + RED_BUF_BYTES, wv, lane);
      __syncthreads();
      if (wv == 3) { red_recv<3>(acc, red + RED_BUF_BYTES, lane); red_store<BF, CT, 8, 6, 2>(acc, g, m_base, T.n0, lane); }
    } else {
      // The two waves trade the halves of their partial tiles that the other one owns (wave 0: the
      // row groups ja < 4).  The first barrier keeps a wave from overwriting what the other still
      // reads for the previous tile.
      __syncthreads();
      if (wv == 0) red_send_half<JA, 1>(acc, red + lane * 16);
      else         red_send_half<JA, 0>(acc, red + RED_HALF_BYTES + lane * 16);
      __syncthreads();
      if (wv == 0) {
        red_recv_half<JA, 0>(acc, red + RED_HALF_BYTES + lane * 16);
        red_store<BF, CT, JA, 0, JA / 2, true>(acc, g, m_base, T.n0, lane, stage);
      } else {
        red_recv_half<JA, 1>(acc, red + lane * 16);
        red_store<BF, CT, JA, JA / 2, JA / 2, true>(acc, g, m_base, T.n0, lane, stage);
      }
    }
    if (!more) break;
    PIT_SCHED_FENCE();
    lin = lin_next;
    T = Tn;
#pragma unroll
    for (int i = 0; i < JA; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
}

__global__ void __launch_bounds__(256) k_zero_rows(void* C, int64_t ld_bytes, int M, int64_t row_bytes) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  char* p = reinterpret_cast<char*>(C) + (int64_t)row * ld_bytes;
  for (int64_t b = (int64_t)(threadIdx.x & 63) * 16; b < row_bytes; b += 64 * 16)
    *reinterpret_cast<uint4*>(p + b) = make_uint4(0, 0, 0, 0);
}



}  // namespace

template <bool BF, int CT, int NW, int JA>
static int launch_gather_k_tile(const GemmArgs& g, int resident, hipStream_t st) {
  const int64_t tm = g.M / (16 * JA), total = tm * (g.N / TN);
  // with more tiles than `resident` per compute unit the workgroups loop
  const unsigned wgs = (unsigned)std::min<int64_t>(total, (int64_t)resident * compute_units());
  hipLaunchKernelGGL((k_gather_k_direct<BF, CT, NW, JA>), dim3(wgs), dim3(64 * NW), 0, st, g, (int)tm);
  PIT_LAUNCH_CHECK();
  return PIT_OK;
}

// Tile height and waves per tile by the number of tiles the product has at each height (128 columns wide; cus compute
// units).  A tile may be lower than the micro-tile: the tiles of a micro-tile row share its list.
//   few tiles: k_gather_k_ring (the rule is at ring_tile); what is left of the next two lines is products it does not take.
//   32-row tiles <= cus (lists of micro-tiles of 32 rows): those, four waves each.  The taller tile leaves compute units
//     idle, or alone with the latency of one long tile; with two waves 512 x 4096 x 512 was 31.6 for 22.0 us.
//   64-row tiles <= cus: those, four waves each: 2048 x 2048 x 1024 19.4 / 14.8 (at 512 tiles of 64 rows, 2048 x 4096 x
//     2048, 128-row tiles are better: 32.6 / 43.6).
//   otherwise the micro-tile's own height.  128 rows: four waves up to two tiles per compute unit, two beyond.  Lower
//     tiles: two waves, and from eight tiles per compute unit on one wave, without a reduction (4096^3, two waves / one:
//     32 rows at 10 % 48.5 / 47.3, at 50 % 171 / 147; 64 rows at 10 % 53.6 / 49.5, at 50 % 88.6 / 89.0; with four tiles
//     per compute unit and lists of 200 entries, 32 rows, 10.1 / 11.2; measured with one chain of additions: the second
//     adds 0 - 0.5 us to the 32-row, 0.6 - 1.5 to the 64-row products; the most seen: 64 rows, 4096^3, live in
//     runs of 32 at 10 %, 42.6 -> 46.4).
template <bool BF, int CT>
static int launch_gather_k(const GemmArgs& g, int tm_tiles, hipStream_t st) {
  const int64_t cus = compute_units(), tn = g.N / TN;
  const RingTile ring = ring_tile(g);
  if (ring != RING_NONE) return launch_gather_k_ring(BF, CT, g, ring, st);
  if (g.M / 32 * tn <= cus) return launch_gather_k_tile<BF, CT, 4, 2>(g, 2, st);
  if (g.slab >= 64 && g.M / 64 * tn <= cus) return launch_gather_k_tile<BF, CT, 4, 4>(g, 1, st);
  const int64_t total = tm_tiles * tn;
  if (g.slab == 32) return total >= 8 * cus ? launch_gather_k_tile<BF, CT, 1, 2>(g, 8, st) : launch_gather_k_tile<BF, CT, 2, 2>(g, 4, st);
  if (g.slab == 64) return total >= 8 * cus ? launch_gather_k_tile<BF, CT, 1, 4>(g, 4, st) : launch_gather_k_tile<BF, CT, 2, 4>(g, 2, st);
  return total >= 2 * cus ? launch_gather_k_tile<BF, CT, 2, 8>(g, 2, st) : launch_gather_k_tile<BF, CT, 4, 8>(g, 1, st);
}

// GATHER_K: tm_tiles = number of row tiles = segments of the index
static int launch_sread_gemm_k(bool bf, int c_is_in_type, const GemmArgs& g, int tm_tiles, hipStream_t st) {
  if (tm_tiles <= 0 || g.N <= 0) return PIT_OK;
  // the kernel addresses each operand with 32-bit byte offsets from a uniform base and multiplies row
  // numbers by the row pitch in 24 bits
  if (g.lda * 2 >= (1ll << 24) || g.ldb * 2 >= (1ll << 24) || (int64_t)g.K >= (1ll << 24)) return PIT_ESHAPE;
  if ((int64_t)g.K * g.lda * 2 >= (1ll << 32) || (int64_t)g.K * g.ldb * 2 >= (1ll << 32)) return PIT_ESHAPE;
  if (bf) return c_is_in_type ? launch_gather_k<true, 1>(g, tm_tiles, st) : launch_gather_k<true, 0>(g, tm_tiles, st);
  return c_is_in_type ? launch_gather_k<false, 1>(g, tm_tiles, st) : launch_gather_k<false, 0>(g, tm_tiles, st);
}

int launch_zero_rows(void* C, int64_t ld_bytes, int M, int64_t row_bytes, hipStream_t st) {
  if (M <= 0 || row_bytes <= 0) return PIT_OK;
  hipLaunchKernelGGL(k_zero_rows, dim3((unsigned)ceil_div(M, 4)), dim3(256), 0, st, C, ld_bytes, M, row_bytes);
  PIT_LAUNCH_CHECK();
  return PIT_OK;
}

}  // namespace pit

using namespace pit;

extern "C" int pit_sread_gemm(int mode, const void* d_A, int64_t lda, const void* d_B, int64_t ldb,
                              void* d_C, int64_t ldc, int M, int N, int K, int in_dt, int c_dt,
                              const pit_index* ix, int mt, int zero_uncovered, pit_stream stream) {
  if (mode != PIT_GEMM_GATHER_M && mode != PIT_GEMM_GATHER_K && mode != PIT_GEMM_DENSE_K) return PIT_EINVAL;
  if (mode != PIT_GEMM_DENSE_K && (!ix || !ix->seg_ptr)) return PIT_EINVAL;
  if (in_dt != PIT_BF16 && in_dt != PIT_F16) return PIT_EINVAL;
  if (c_dt != PIT_F32 && c_dt != in_dt) return PIT_EINVAL;
  if (M < 0 || N < 0 || K < 0 || mt <= 0) return PIT_ESHAPE;
  if (N % TN) return PIT_ESHAPE;
  const int c_esize = c_dt == PIT_F32 ? 4 : 2;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (M == 0 || N == 0) return PIT_OK;
  if (!d_C || !aligned(d_C, 16) || ldc < N || (ldc * c_esize) % 16) return PIT_EINVAL;
  if (K > 0) {
    if (!d_A || !d_B || (mode != PIT_GEMM_DENSE_K && !ix->idx)) return PIT_EINVAL;
    if (!aligned(d_A, 16) || !aligned(d_B, 16) || lda % 8 || ldb % 8 || ldb < N) return PIT_EINVAL;
  }

  GemmArgs g = {};
  g.A = d_A; g.lda = lda; g.B = d_B; g.ldb = ldb; g.b_seg_stride = 0;
  g.C = d_C; g.ldc = ldc; g.gate = nullptr;
  g.M = M; g.N = N; g.K = K;
  if (mode == PIT_GEMM_DENSE_K) {
    // the dense kernel of Algorithm 1's fallback: the GATHER_K tile with identity addressing
    if ((mt != 128 && mt != 64 && mt != 32) || M % mt) return PIT_ESHAPE;
    if (K > 0 && lda < M) return PIT_EINVAL;
    g.seg_ptr = nullptr; g.idx = nullptr; g.nseg = M / mt; g.slab = mt;
    return launch_sread_gemm_k(in_dt == PIT_BF16, c_dt != PIT_F32, g, M / mt, st);
  }
  g.seg_ptr = ix->seg_ptr; g.idx = ix->idx; g.nseg = ix->nseg;

  if (mode == PIT_GEMM_GATHER_K) {
    if ((mt != 128 && mt != 64 && mt != 32) || M % mt) return PIT_ESHAPE;
    if (ix->nseg != M / mt) return PIT_ECAPACITY;
    if (K > 0 && lda < M) return PIT_EINVAL;
    g.slab = mt;       // GATHER_K: the micro-tile height of the index
    return launch_sread_gemm_k(in_dt == PIT_BF16, c_dt != PIT_F32, g, ix->nseg, st);
  }

  // GATHER_M
  if (K == 0) {  // empty product: C is zero wherever the call is asked to define it
    if (zero_uncovered || ix->nseg > 1) {
      return launch_zero_rows(d_C, ldc * c_esize, M, (int64_t)N * c_esize, st);
    }
    return PIT_OK;
  }
  if (mt % 32 || K % mt) return PIT_ESHAPE;
  if (ix->nseg != K / mt) return PIT_ECAPACITY;
  if (lda < K) return PIT_EINVAL;
  g.slab = mt; g.a_gather = 1; g.c_scatter = 1; g.slab_per_seg = 1;
  if (ix->nseg == 1) {
    // (rows the list does not name are cleared inside the product's launch, by its workgroups without a tile)
    g.zero_rest = zero_uncovered ? 1 : 0;
    return launch_gather_m(in_dt == PIT_BF16, EPI_STORE, c_dt != PIT_F32, g, M, st);
  }
  if (c_dt != PIT_F32) return PIT_EINVAL;
  // several k-slabs per row: C-stationary strips (every element of C is written, nothing to clear)
  if (g.lda * 2 >= (1ll << 24) || g.ldb * 2 >= (1ll << 24) || (int64_t)M >= (1ll << 24) || (int64_t)K >= (1ll << 24)) return PIT_ESHAPE;
  if ((int64_t)M * g.lda * 2 >= (1ll << 32) || (int64_t)K * g.ldb * 2 >= (1ll << 32)) return PIT_ESHAPE;
  return launch_slab_strip(in_dt == PIT_BF16, g, st);
}

// ------------------------------------------------------------------------------------------------
// Algorithm 1 end to end: select among the GATHER_K tile heights and the dense kernel, then run the winner.
// ------------------------------------------------------------------------------------------------
namespace pit {
namespace {
struct SelectWs { size_t seg_ptr_off, idx_off, build_off, total; };
// sized for the finest micro-tile (32): the most segments and the most entries
SelectWs select_layout(int M, int K) {
  SelectWs w;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += (bytes + 255) & ~(size_t)255; return at; };
  const size_t nseg = (size_t)(M > 0 ? M : 0) / 32 + 1;
  w.seg_ptr_off = take((nseg + 1) * 4);
  w.idx_off = take((nseg * (size_t)(K > 0 ? K : 1)) * 4);
  size_t b = 0;
  for (int mt : {32, 64, 128}) b = std::max(b, pit_build_index_workspace(K, M - M % mt, 1, mt, 0, 0));
  w.build_off = take(b + 64);
  w.total = o;
  return w;
}
}  // namespace
}  // namespace pit

extern "C" size_t pit_select_and_run_gemm_workspace(int M, int K) {
  if (M < 0 || K < 0) return 0;
  return select_layout(M, K).total;
}

extern "C" int pit_select_and_run_gemm(const pit_kernel_candidate* cand, int ncand, const int64_t* num_tiles,
                                       const int64_t* grid_tiles, int nsamples,
                                       const void* d_At, int64_t lda, const void* d_B, int64_t ldb,
                                       void* d_C, int64_t ldc, int M, int N, int K, int in_dt, int c_dt,
                                       void* d_ws, size_t ws_bytes, int* chosen, pit_stream stream) {
  if (!cand || ncand <= 0) return PIT_EINVAL;
  for (int j = 0; j < ncand; ++j) {
    const int mt = cand[j].mt_cols;
    if (cand[j].mt_rows != 1 || (mt != 32 && mt != 64 && mt != 128)) return PIT_ESHAPE;
  }
  int best = 0;
  const int rc = pit_select_kernel(cand, ncand, num_tiles, grid_tiles, nsamples, nullptr, &best);
  if (rc != PIT_OK) return rc;
  if (chosen) *chosen = best;
  const int mt = cand[best].mt_cols;
  if (M < 0 || N < 0 || K < 0) return PIT_ESHAPE;
  if (M % mt) return PIT_ESHAPE;
  if (cand[best].dense)
    return pit_sread_gemm(PIT_GEMM_DENSE_K, d_At, lda, d_B, ldb, d_C, ldc, M, N, K, in_dt, c_dt, nullptr, mt, 0, stream);
  const SelectWs L = select_layout(M, K);
  if (!d_ws || !aligned(d_ws, 256)) return PIT_EINVAL;
  if (ws_bytes < L.total) return PIT_ECAPACITY;
  char* ws = reinterpret_cast<char*>(d_ws);
  pit_index ix;
  ix.seg_ptr = reinterpret_cast<int32_t*>(ws + L.seg_ptr_off);
  ix.idx = reinterpret_cast<int32_t*>(ws + L.idx_off);
  ix.bits = nullptr;
  ix.nseg = M / mt;
  ix.cap = (int32_t)std::min<int64_t>((int64_t)(M / mt) * K, INT32_MAX);
  if ((int64_t)(M / mt) * K > INT32_MAX) return PIT_ESHAPE;
  const int rb = pit_build_index(d_At, in_dt, K, M, lda, 1, mt, 0, &ix, ws + L.build_off, L.total - L.build_off, stream);
  if (rb != PIT_OK) return rb;
  return pit_sread_gemm(PIT_GEMM_GATHER_K, d_At, lda, d_B, ldb, d_C, ldc, M, N, K, in_dt, c_dt, &ix, mt, 0, stream);
}
