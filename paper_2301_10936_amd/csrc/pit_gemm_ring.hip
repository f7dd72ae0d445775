// GATHER_K for products with few tiles (pit_gemm.hip has the kernel for the others), gfx950.  bf16 or f16 inputs, fp32
// accumulation.
//
// A product of few rows and columns and a long k leaves most compute units idle at 128 columns a tile, and those that work
// alone with the latency of four waves (512 x 5195 x 512: 64 tiles, 29 us; here 128 tiles, 12.9).  Here a tile is 32 x 32, 32 x 64
// or 64 x 64, and NW waves of one workgroup split its k-list (slabs of 32 entries, wave w takes w, w + NW, ..), each with a ring
// of NST slabs of its own in LDS: no barrier before the partial tiles meet.  With eight waves a compute unit has 64 - 128 KB
// on their way.  Bound: 2 - 3 us of launch, first loads, reduction and stores, then the rate at which a compute unit is
// given operands, 64 x 64: 55 bytes per clock (512 x 5195 x 512, 10 us for the 1.3 MB of a tile), rows of 64 bytes half of it.
//   SRead   both operands are K-major (rows of At and of B).  They travel global -> LDS directly, 16 bytes per lane: an
//           instruction brings 8 or 16 listed rows of 128 or 64 bytes, and the lane's source address expresses both the gather
//           (which row) and the bank swizzle (which 32 bytes of it).  A row of T columns lies in LDS as 2 T bytes, its
//           32-byte chunk c at c ^ f(row): f keeps the 16 rows that one transposing read touches on all banks.
//   list    the entries travel to LDS by the same kind of load, 64 at a time (two slabs of the wave), NST slabs ahead of
//           their use; no load of the loop has a register for a destination, so all waits are the explicit ones here.
//   MFMA    v_mfma_f32_16x16x32, operands read with ds_read_b64_tr_b16 (8 consecutive slots of the slab of one column); the
//           blocks are computed transposed, so that a lane holds four consecutive columns of a row of C.
//   SWrite  every wave leaves its partial tile in LDS (over the rings); the partial tiles are added in the order of the
//           waves and stored, 16 lanes filling 256 contiguous bytes of an fp32 row.
#include "pit_gemm.hpp"
#include "pit_ring.hpp"

namespace pit {
namespace {

template <bool BF, int CT, int TA, int TB, int NW, int NST, bool DENSE>
__global__ void __launch_bounds__(64 * NW, NW / 4)
k_gather_k_ring(const GemmArgs g, const int tm_tiles) {
  static_assert(NST % 2 == 0 && NST <= 4, "stages of a wave's ring: the list comes for two slabs at a time");
  using LA = SlabLayout<TA>;
  using LB = SlabLayout<TB>;
  constexpr int SK = 32, NA = LA::LOADS, NB = LB::LOADS, LOADS = NA + NB, STAGE = LA::BYTES + LB::BYTES;
  constexpr int FA = TA / 16, FB = TB / 16;                // 16-column operand blocks
  constexpr int RING = NW * NST * STAGE, PART = TA * TB * 4;
  constexpr int CHUNKS = 4;                                // list chunks (two slabs each) of a wave
  __shared__ __attribute__((aligned(1024))) char smem[RING > NW * PART ? RING : NW * PART];
  __shared__ __attribute__((aligned(256))) int s_list[DENSE ? 1 : NW * CHUNKS * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  // tiles in the order of k_gather_k_direct: a contiguous run per XCD, in bands of 4 tile columns x all tile rows.  8 where there
  // are two workgroups per compute unit, as wide as that kernel's bands: each band reads A again, and an operand that the launch before
  // wrote does not come from this XCD's L2.  The producer and 3328 x 768 x 384: 18.9 us by that kernel, 20.9 in bands of 4, 19.2 of 8;
  // 64 products of 264 - 512 tiles behind the producer 0.99 of its time in bands of 4, the slowest 1.17, and 0.97 of 8 (1.03).  With one workgroup per
  // compute unit 4 is better for 32 x 64 (the index and 512 x 11160 x 512: 1.24 times as long in bands of 8) and the same for 64 x 64.
  const int tn = g.N / TB, total = tn * tm_tiles;
  const bool wide = tn > 2 * tm_tiles;
  int row, n0;
  {
    const int lin = blockIdx.x, x = lin & 7, rr = total & 7;
    const int lp = x * (total >> 3) + min(x, rr) + (lin >> 3);
    constexpr int G = NW == 4 ? 8 : 4;
    const int across = wide ? tn : tm_tiles, along = wide ? tm_tiles : tn;
    const int band = lp / (G * across), within = lp - band * (G * across), n = min(G, along - band * G);
    const int thin = band * G + within % n, len = within / n;
    row = wide ? thin : len;
    n0 = (wide ? len : thin) * TB;
  }
  const int seg = row / (g.slab / TA);                     // the tiles of a micro-tile row share its list
  const int list_begin = DENSE ? 0 : g.seg_ptr[seg];
  const int list_len = __builtin_amdgcn_readfirstlane(DENSE ? g.K : g.seg_ptr[seg + 1] - list_begin);
  const int nslab = (list_len + SK - 1) / SK;
  const int n_w = nslab > wv ? (nslab - wv + NW - 1) / NW : 0;
  const char* a_src = uniform_ptr(g.A);
  const char* b_src = uniform_ptr(g.B);
  const char* list = uniform_ptr(DENSE ? nullptr : g.idx + list_begin);
  const uint32_t pitch_a = (uint32_t)(g.lda * 2), pitch_b = (uint32_t)(g.ldb * 2);

  const uint32_t lds0 = (uint32_t)(uintptr_t)(PIT_LDS char*)smem, ring = lds0 + (uint32_t)(wv * NST * STAGE);
  const uint32_t list0 = (uint32_t)(uintptr_t)(PIT_LDS int*)s_list + (uint32_t)(DENSE ? 0 : wv * CHUNKS * 256);

  // lane constants of the loads: byte offset into a row of At / B
  uint32_t a_col[NA], b_col[NB];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int p = lane % LA::LPR, s = LA::RPI * j + lane / LA::LPR;
    a_col[j] = (uint32_t)(row * TA * 2 + (((p >> 1) ^ LA::f(s)) * 32) + (p & 1) * 16);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int p = lane % LB::LPR, s = LB::RPI * j + lane / LB::LPR;
    b_col[j] = (uint32_t)(n0 * 2 + (((p >> 1) ^ LB::f(s)) * 32) + (p & 1) * 16);
  }
  // position of slot 0 of the wave's slab t in the list
  auto pos_of = [&](int t) { return SK * (wv + NW * t); };
  // entries of the wave's slabs t and t + 1 (t even) -> chunk (t / 2) % CHUNKS; positions past the end: the last entry
  auto issue_list = [&](int t) {
    if constexpr (!DENSE) {
      const int pos = min(pos_of(t + (lane >> 5)) + (lane & 31), list_len - 1);
      dma4(list, (uint32_t)pos * 4u, list0 + (uint32_t)(((t >> 1) & (CHUNKS - 1)) * 256));
    }
  };
  auto entry = [&](int t, int slot) -> uint32_t {
    if constexpr (DENSE) return (uint32_t)min(pos_of(t) + slot, list_len - 1);
    else return *(PIT_LDS uint32_t*)(uintptr_t)(list0 + (uint32_t)(((t >> 1) & (CHUNKS - 1)) * 256 + (t & 1) * 128 + slot * 4));
  };
  struct Rows { uint32_t a[NA], b[NB]; };
  auto rows_of = [&](int t, Rows& r) {                     // source offsets of the lane's pieces of slab t
#pragma unroll
    for (int j = 0; j < NA; ++j) r.a[j] = entry(t, LA::RPI * j + lane / LA::LPR);
#pragma unroll
    for (int j = 0; j < NB; ++j) r.b[j] = TA == TB ? r.a[j] : entry(t, LB::RPI * j + lane / LB::LPR);
#pragma unroll
    for (int j = 0; j < NB; ++j) r.b[j] = __umul24(r.b[j], pitch_b) + b_col[j];
#pragma unroll
    for (int j = 0; j < NA; ++j) r.a[j] = __umul24(r.a[j], pitch_a) + a_col[j];
  };
  auto issue = [&](const Rows& r, int u) {                 // -> stage u
    const uint32_t at = ring + (uint32_t)(u * STAGE);
#pragma unroll
    for (int j = 0; j < NA; ++j) dma16(a_src, r.a[j], at + (uint32_t)(j * 1024));
#pragma unroll
    for (int j = 0; j < NB; ++j) dma16(b_src, r.b[j], at + (uint32_t)(LA::BYTES + j * 1024));
  };

  // operand reads: lane -> column lane % 16 of a block, slots 8 (lane / 16) .. + 7.  In a transposing read lanes 4 j .. 4 j + 3 of
  // a group of 16 address slot 8 (lane / 16) + j (+ 4), 8 bytes each of the block's 32.
  const int s_rd = 8 * (lane >> 4) + ((lane >> 2) & 3);
  uint32_t a_rd[FA], b_rd[FB];
#pragma unroll
  for (int c = 0; c < FA; ++c) a_rd[c] = ring + (uint32_t)(s_rd * TA * 2 + ((c ^ LA::f(s_rd)) * 32) + (lane & 3) * 8);
#pragma unroll
  for (int c = 0; c < FB; ++c) b_rd[c] = ring + (uint32_t)(LA::BYTES + s_rd * TB * 2 + ((c ^ LB::f(s_rd)) * 32) + (lane & 3) * 8);
  struct Frags { u32x4_t a[FA], b[FB]; };
  auto read_frags = [&](int u, Frags& fr) {
    const uint32_t so = (uint32_t)(u * STAGE);
#pragma unroll
    for (int c = 0; c < FA; ++c) {
      const uint2 lo = lds_tr(a_rd[c] + so), hi = lds_tr(a_rd[c] + so + 4 * TA * 2);
      fr.a[c] = u32x4_t{lo.x, lo.y, hi.x, hi.y};
    }
#pragma unroll
    for (int c = 0; c < FB; ++c) {
      const uint2 lo = lds_tr(b_rd[c] + so), hi = lds_tr(b_rd[c] + so + 4 * TB * 2);
      fr.b[c] = u32x4_t{lo.x, lo.y, hi.x, hi.y};
    }
  };
  f32x4_t acc[FB][FA];
#pragma unroll
  for (int i = 0; i < FB; ++i)
#pragma unroll
    for (int j = 0; j < FA; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto mfmas = [&](const Frags& fr) {
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int j = 0; j < FA; ++j) acc[i][j] = mfma16r<BF>(fr.b[i], fr.a[j], acc[i][j]);
  };

  if (n_w > 0) {
    // In every iteration t the loads are issued in the order: list chunk of slabs t + 2 NST and t + 2 NST + 1 (t even), slab
    // t + NST.  So when slab t has landed, the entries of slab t + NST have, and younger than slab t are the loads of
    // NST - 1 slabs and the list chunks of the even ones of NST - 1 iterations.  The same order before the loop.
#pragma unroll
    for (int u = 0; u < NST; u += 2) issue_list(u);
    PIT_WAIT_VMCNT(0);
#pragma unroll
    for (int u = 0; u < NST; ++u) {
      if ((u & 1) == 0) issue_list(u + NST);
      if (u < n_w) { Rows r; rows_of(u, r); issue(r, u); }
    }
    int t = 0;
    for (; t + 2 * NST <= n_w; t += NST) {
#pragma unroll
      for (int u = 0; u < NST; ++u) {
        constexpr int lists_even = DENSE ? 0 : (NST - 2) / 2, lists_odd = DENSE ? 0 : NST / 2;
        if ((u & 1) == 0) PIT_WAIT_VMCNT((NST - 1) * LOADS + lists_even);
        else              PIT_WAIT_VMCNT((NST - 1) * LOADS + lists_odd);
        Frags fr;
        Rows r;
        rows_of(t + u + NST, r);
        read_frags(u, fr);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read
        if ((u & 1) == 0) issue_list(t + u + 2 * NST);
        issue(r, u);
        mfmas(fr);
      }
    }
    for (int s = t; s < n_w; ++s) {                        // t is a multiple of NST
      const int u = s - t < NST ? s - t : s - t - NST;
      // (list chunks not counted: a little stricter than needed)
      const int younger = min(NST - 1, n_w - 1 - s);
      if (NST > 3 && younger == 3) PIT_WAIT_VMCNT(3 * LOADS);
      else if (NST > 2 && younger == 2) PIT_WAIT_VMCNT(2 * LOADS);
      else if (younger == 1) PIT_WAIT_VMCNT(LOADS);
      else PIT_WAIT_VMCNT(0);
      Frags fr;
      read_frags(u, fr);
      if (s + NST < n_w) {
        Rows r;
        rows_of(s + NST, r);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(r, u);
      }
      const int left = list_len - pos_of(s);
      if (left < SK) {                                     // the list's last slab: slots past the end are zero in both operands
        const int valid = max(0, min(8, left - 8 * (lane >> 4)));
        u32x4_t m;
#pragma unroll
        for (int d = 0; d < 4; ++d) m[d] = valid >= 2 * d + 2 ? 0xffffffffu : valid == 2 * d + 1 ? 0x0000ffffu : 0u;
#pragma unroll
        for (int c = 0; c < FA; ++c) fr.a[c] &= m;
#pragma unroll
        for (int c = 0; c < FB; ++c) fr.b[c] &= m;
      }
      mfmas(fr);
    }
    PIT_WAIT_VMCNT(0);                                     // (list chunks past the last slab: nothing may land in LDS after this)
  }

  // ---------------------------------------------------------------- reduction and SWrite
  auto place = [](int m, int c) { return partial_place<TB, FA>(m, c); };
  __syncthreads();
#pragma unroll
  for (int i = 0; i < FB; ++i)
#pragma unroll
    for (int j = 0; j < FA; ++j)
      *(PIT_LDS f32x4_t*)(uintptr_t)(lds0 + (uint32_t)(wv * PART) + place(16 * j + (lane & 15), 4 * i + (lane >> 4))) = acc[i][j];
  __syncthreads();
  constexpr int VPR = TB / 4;
#pragma unroll
  for (int v = tid; v < TA * VPR; v += 64 * NW) {
    const int m = v / VPR, c = v % VPR;
    const uint32_t at = lds0 + place(m, c);
    f32x4_t part[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) part[w] = *(PIT_LDS f32x4_t*)(uintptr_t)(at + (uint32_t)(w * PART));
    f32x4_t s = part[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += part[w];
    const int64_t o = (int64_t)(row * TA + m) * g.ldc + n0 + 4 * c;
    if constexpr (CT == 0) __builtin_nontemporal_store(s, reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(g.C) + o));
    else __builtin_nontemporal_store(u32x2_t{pack2_in<BF>(s[0], s[1]), pack2_in<BF>(s[2], s[3])},
                                     reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(g.C) + o));
  }
}

template <bool BF, int CT, int TA, int TB, int NW>
int launch_ring(const GemmArgs& g, hipStream_t st) {
  const int64_t tm = g.M / TA, total = tm * (g.N / TB);      // (at most 2 cus: ring_tile)
  constexpr int NST = 2;                                   // (four for 32 x 32: the same)
  if (g.idx == nullptr) hipLaunchKernelGGL((k_gather_k_ring<BF, CT, TA, TB, NW, NST, true>), dim3((unsigned)total), dim3(64 * NW), 0, st, g, (int)tm);
  else                  hipLaunchKernelGGL((k_gather_k_ring<BF, CT, TA, TB, NW, NST, false>), dim3((unsigned)total), dim3(64 * NW), 0, st, g, (int)tm);
  PIT_LAUNCH_CHECK();
  return PIT_OK;
}
template <bool BF, int CT>
int launch_ring_bf(const GemmArgs& g, int tile, hipStream_t st) {
  switch (tile) {
    case RING_32x32: return launch_ring<BF, CT, 32, 32, 8>(g, st);
    case RING_32x64: return launch_ring<BF, CT, 32, 64, 8>(g, st);
    case RING_64x64: return launch_ring<BF, CT, 64, 64, 8>(g, st);
    case RING_64x64_SHORT: return launch_ring<BF, CT, 64, 64, 4>(g, st);
    default: return PIT_EINVAL;
  }
}

}  // namespace

// Which tile, by how many of each the product has (cus compute units; times of the product alone, us, of k_gather_k_direct
// and of the tiles 32 x 32, 32 x 64 and 64 x 64, eight waves each).  One workgroup per compute unit: the smallest tile
// that gives no more of them -- a smaller tile splits the operands over more compute units and reads more of them in all, and with
// rows of 64 bytes (32 columns) a load instruction brings half as much per clock, hence 3/4.
//   32 x 32 up to 3/4 cus    128 x 1837 x 128  9.1 / 4.6, 5.7, 7.5;  256 x 512 x 256  4.8 / 3.1, 3.7, 4.7;
//     384 x 5448 x 256 (96 tiles) 17.7 / 8.0, 11.9, 12.5;  128 x 6942 x 2048 (256) 28.3 / 19.8, 21.2, 23.8; 512 x 2706 x 512
//     (256) 12.0 / 8.2, 7.3, 9.5
//   32 x 64 up to cus        512 x 5195 x 512 (128) 29.1 / 13.8, 12.9, 15.6;  384 x 4788 x 1280 (240) 24.8 / 26.7, 18.1, 19.9;
//     480 x 10676 x 1152 (270) 44.5 / 78.6, 59.5
//   64 x 64 up to cus        512 x 2936 x 1152 (144) 16.8 / 20.1, 17.7, 11.1;  3584 x 6104 x 256 (224) 29.0 / 55.4, 35.8, 22.7;
//     1024 x 8192 x 1024 (256) 34.4 / 74.9, 47.6, 28.9;  512 x 5070 x 2688 (336) 29.4 / 66.7, 45.2, 35.2
//   64 x 64, four waves and two workgroups per compute unit, up to 2 cus where k is short (a tile's start and end then weigh as
//     much as its slabs): 896 x 328 x 2048 (448) 7.7 / 6.1, 3328 x 836 x 512 (416) 9.2 / 8.0, 832 x 1468 x 2432 (494) 12.5 / 13.2;
//     up to cus, eight waves / four: 448 x 1162 x 1664 6.9 / 6.6, 640 x 311 x 896 4.2 / 4.1, 512 x 2629 x 1408 10.6 / 11.1.
// 130 products of 128 - 4096 x 257 - 12000 x 128 - 4096 with at most 700 tiles of 64 x 64, full and sparse lists: 0.75 of
// k_gather_k_direct's time in the geometric mean (the fastest of them every time: 0.74), none slower by more than 1 %.
RingTile ring_tile(const GemmArgs& g) {
  const int64_t cus = compute_units(), t32x64 = (int64_t)(g.M / 32) * (g.N / 64), t64 = t32x64 / 2;
  if (8 * t32x64 <= 3 * cus) return RING_32x32;
  if (t32x64 <= cus) return RING_32x64;
  if (g.slab >= 64 && g.K <= 1024 && t64 <= 2 * cus) return RING_64x64_SHORT;
  if (g.slab >= 64 && t64 <= cus) return RING_64x64;
  return RING_NONE;
}

int launch_gather_k_ring(bool bf, int c_is_in_type, const GemmArgs& g, RingTile tile, hipStream_t st) {
  if (bf) return c_is_in_type ? launch_ring_bf<true, 1>(g, tile, st) : launch_ring_bf<true, 0>(g, tile, st);
  return c_is_in_type ? launch_ring_bf<false, 1>(g, tile, st) : launch_ring_bf<false, 0>(g, tile, st);
}

}  // namespace pit
