// GATHER_M for products with few tiles, and for segments of few rows with a B of their own (pit_gemm_m.hip has the kernel for
// the others), gfx950.  bf16 or f16 inputs, fp32 accumulation.
//
// k_gather_m_lds walks all of k with one workgroup barrier per 32: 0.3 us a step and 6 us around it, however few rows there are.
// Here a tile is TR x TC with 16 to 64 rows and 32 or 64 columns, and the four or eight waves of a workgroup split k (steps of 32,
// wave w takes w, w + NW, ..), each with a ring of two steps of its own in LDS; the partial tiles meet at the end.  Bound: 3 - 4 us of
// launch, first loads (the tile, its row numbers, the operands one after the other), reduction and stores; then what a compute
// unit is given per clock (few tiles), or the memory's rate for the weights (a mixture of experts).
//   SRead   A rows (K-minor) and B rows (K-major) travel global -> LDS directly.  A: 16 listed rows x 64 bytes per instruction,
//           the 16-byte chunk c of row r at c ^ ((r >> 2) & 3), operands read with ds_read_b128.  B: as in k_gather_k_ring,
//           operands read with the transposing LDS read.
//   SWrite  partial tiles added in the order of the waves (with a B per segment of eight chains along k); rows go where the index says, 16 lanes filling 256 contiguous bytes of
//           an fp32 row.  The rows that a list does not name are cleared by the workgroups without a tile, when asked for.
//   SLABS   micro-tiles along k: the tile's rows are those of C; which of them a slab lists comes as bits in LDS
//           (build_slab_masks, while the first operands travel), and the A operands of the others are set to zero in registers; a wave
//           that meets many steps without a listed row leaves those out.
// Product alone, k_gather_m_lds / here, us: 186 rows (140 listed) x 1408 x 384 14.6 / 4.0, 732 (308) x 1920 x 1792 19.0 / 7.8, 2911 x
// 1408 x 512 14.2 / 7.8.  Whole mixture-of-experts calls, us, before (segments of few rows went to a kernel with the weights in
// registers) / here: 1 token, 896 x 1792, 8 experts 11.6 / 8.0; 515, 640 x 1920, 8 31.6 / 21.5; 48, 768 x 3072, 64, bound by the memory, 56.2 / 55.2.
// Tried: four steps per ring (fewer workgroups per compute unit: up to 1.7 times the time), three with 16 x 64 and eight waves (the same).
#include "pit_ring.hpp"
#include "pit_gather_m.hpp"
#include "pit_slab_masks.hpp"
#include <algorithm>
#include <cmath>

namespace pit {
namespace {

// where the rows of the tiles come from: one list; a list per segment, each with a B of its own; the expert ids of up to 64 tokens;
// all rows, with a list per k-slab of those that count
enum { ONE, SEGMENTS, ROUTE, SLABS };

template <bool BF, int EPI, int CT, int TR, int TC, int NW, int MODE>
__global__ void __launch_bounds__(64 * NW, 2)
k_gather_m_ring(const GemmArgs g) {
  using LB = SlabLayout<TC>;
  constexpr int KS = 32, NST = 2;
  constexpr int A_BYTES = TR * KS * 2, NA = A_BYTES / 1024, NB = LB::LOADS, LOADS = NA + NB, STAGE = A_BYTES + LB::BYTES;
  constexpr int FA = TR / 16, FB = TC / 16;
  // A B per segment: eight chains of additions whatever the number of waves, chain c with the steps c, c + 8, .. (four waves have
  // two each).  Four chains round a sum of 2048 - 4096 products 1.08 - 1.19 times as much.
  constexpr int CH = (MODE == SEGMENTS || MODE == ROUTE) && NW == 4 ? 2 : 1;
  static_assert(CH == 1 || NST == 2, "a step's stage and chain");
  static_assert(MODE != ROUTE || TR < 64, "lane 63 holds no row's token");
  constexpr int RING = NW * NST * STAGE, PART = TR * TC * 4;
  __shared__ __attribute__((aligned(1024))) char smem[RING > NW * PART ? RING : NW * PART];
  constexpr int MW = (TR + 31) / 32;                       // SLABS: words of the rows listed for a slab
  __shared__ uint32_t s_mask[MODE == SLABS ? SLABS_MAX * MW : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(PIT_LDS char*)smem, ring = lds0 + (uint32_t)(wv * NST * STAGE);

  // The tile.  Which rows exist is known only here; the grid holds the worst case.  Every XCD (own L2) takes a contiguous run
  // of the tiles that exist.
  const int tn = g.N / TC;
  const int lin = blockIdx.x, xcd = lin & 7, slot = lin >> 3;
  int n0, begin = 0, cnt, seg = 0;
  int rows = 0;                                            // ROUTE: lane r holds the token of the tile's row r
  if constexpr (MODE == SLABS) {
    const int rt = (g.M + TR - 1) / TR, total = rt * tn;
    const int lp = xcd * (total >> 3) + min(xcd, total & 7) + slot;
    const bool down = rt <= tn;
    const int outer = lp / (down ? rt : tn), inner = lp - outer * (down ? rt : tn);
    n0 = (down ? outer : inner) * TC;
    begin = (down ? inner : outer) * TR;
    cnt = min(TR, g.M - begin);
  } else if constexpr (MODE == ONE) {
    const int begin0 = g.seg_ptr[0], cnt0 = g.seg_ptr[1] - begin0;
    const int rt = (cnt0 + TR - 1) / TR, total = rt * tn;
    const int share = (total >> 3) + (xcd < (total & 7) ? 1 : 0);
    if (slot >= share) {
      if (g.zero_rest) {                                   // the workgroups without a tile: an equal share of the rows of C each
        const int grid = (int)gridDim.x, idle = grid - total;
        // number of this one among them: those of the XCDs before its own first
        const int d = xcd * ((grid >> 3) - (total >> 3)) + min(xcd, grid & 7) - min(xcd, total & 7) + slot - share;
        const int per = (g.M + idle - 1) / idle;
        const int rb = min(g.M, d * per), re = min(g.M, rb + per);
        if (rb < re) zero_unlisted_rows<CT ? 2 : 4, NW>(g, rb, re, wv, lane);
      }
      return;
    }
    const int lp = xcd * (total >> 3) + min(xcd, total & 7) + slot;
    const bool down = rt <= tn;                            // along the shorter side first: fewer panels of both per XCD
    const int outer = lp / (down ? rt : tn), inner = lp - outer * (down ? rt : tn);
    const int r0 = (down ? inner : outer) * TR;
    n0 = (down ? outer : inner) * TC;
    begin = begin0 + r0;
    cnt = min(TR, cnt0 - r0);
  } else if constexpr (MODE == ROUTE) {
    // A wave holds all expert ids, one per lane; ballots over their bits give every lane the lanes with its expert, the first lane
    // of each expert stands for it, and ballots over their numbers of row tiles say which expert a tile belongs to (experts in
    // the order of their first token).
    const int e = lane < g.M ? g.route[lane] : -1;
    const bool valid = e >= 0 && e < g.nseg;
    const unsigned long long all = __ballot(valid);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
    for (int bit = 0; (g.nseg - 1) >> bit; ++bit) {        // (keep the lanes whose bit is this lane's)
      const uint32_t on = 0u - (((uint32_t)e >> bit) & 1u);
      const unsigned long long b = __ballot(on != 0u);
      lo &= ~((uint32_t)b ^ on);
      hi &= ~((uint32_t)(b >> 32) ^ on);
    }
    const int size = __builtin_popcount(lo) + __builtin_popcount(hi);
    const int rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
    const int nt = valid && rank == 0 ? (size + TR - 1) / TR : 0;
    int ahead = 0, rt = 0;                                 // row tiles of the experts before this lane's; of all
#pragma unroll
    for (int n = 1; n <= 64 / TR; ++n) {
      const unsigned long long b = __ballot(nt >= n);
      ahead = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, ahead));
      rt += __builtin_popcountll(b);
    }
    if (g.route_rest && lin < tn) {                        // tokens without an expert: counted, their rows of C cleared
      unsigned long long bad = __ballot(lane < g.M && !valid);
      if (lin == 0 && tid == 0 && g.status != nullptr) *g.status = __builtin_popcountll(bad);
      for (int i = 0; bad != 0ull; ++i, bad &= bad - 1ull)
        if ((i & (NW - 1)) == wv) {
          char* p = reinterpret_cast<char*>(g.C) + ((int64_t)__builtin_ctzll(bad) * g.ldc + lin * TC) * (CT ? 2 : 4);
          if (lane < TC * (CT ? 2 : 4) / 16) *reinterpret_cast<u32x4_t*>(p + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
        }
    }
    const int total = rt * tn, share = (total >> 3) + (xcd < (total & 7) ? 1 : 0);
    if (slot >= share) return;
    const int lp = xcd * (total >> 3) + min(xcd, total & 7) + slot;
    const int l = __builtin_ctzll(__ballot(lp >= ahead * tn && lp < (ahead + nt) * tn));   // (one lane: lp < total)
    const int mine_nt = __builtin_amdgcn_readlane(nt, l), within = lp - __builtin_amdgcn_readlane(ahead, l) * tn, col = within / mine_nt;
    n0 = col * TC;
    const int first = (within - col * mine_nt) * TR;       // rank of the tile's first row
    seg = __builtin_amdgcn_readlane(e, l);
    const bool mine = valid && e == seg;
    cnt = min(TR, __builtin_amdgcn_readlane(size, l) - first);
    const int r = rank - first;
    rows = __builtin_amdgcn_ds_permute((mine && r >= 0 && r < TR ? r : 63) * 4, lane);   // (lane 63 is no row's)
  } else {
    // Tiles in the order of the segments, and of a segment along its shorter side first: the row tiles of a few-row segment share its
    // columns of B through one L2.  A lane counts the row tiles of `per`
    // consecutive segments; where that is more than one, those of the tile's lane are looked at again, one per lane.
    const int per = (g.nseg + 63) >> 6;
    auto scan = [&](int nt) -> int {                       // inclusive
      int inc = nt;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(inc, d);
        if (lane >= d) inc += t;
      }
      return inc;
    };
    int beg = g.seg_ptr[min(lane * per, g.nseg)], end = beg, nt = 0;
    for (int i = 1; i <= per; ++i) {
      const int nx = g.seg_ptr[min(lane * per + i, g.nseg)];
      nt += (nx - end + TR - 1) / TR;
      end = nx;
    }
    int inc = scan(nt);
    const int rt = __shfl(inc, 63), total = rt * tn, share = (total >> 3) + (xcd < (total & 7) ? 1 : 0);
    if (slot >= share) return;
    int lp = xcd * (total >> 3) + min(xcd, total & 7) + slot;
    int l = __builtin_ctzll(__ballot(inc * tn > lp));      // (lp < total)
    seg = l;
    if (per > 1) {
      const int s_end = min((l + 1) * per, g.nseg);
      lp -= (__shfl(inc, l) - __shfl(nt, l)) * tn;
      seg = l * per;
      for (;; seg += 64) {
        const int s = min(seg + lane, s_end);
        beg = g.seg_ptr[s];
        end = g.seg_ptr[min(s + 1, s_end)];
        nt = (end - beg + TR - 1) / TR;
        inc = scan(nt);
        const int here = __shfl(inc, 63) * tn;
        if (lp < here || seg + 64 >= s_end) break;
        lp -= here;
      }
      l = __builtin_ctzll(__ballot(inc * tn > lp) | (1ull << 63));
      seg += l;
    }
    const int mine_nt = max(1, __shfl(nt, l)), within = lp - (__shfl(inc, l) - __shfl(nt, l)) * tn;
    const bool down = mine_nt <= tn;
    const int outer = within / (down ? mine_nt : tn), inner = within - outer * (down ? mine_nt : tn);
    const int in_seg = down ? inner : outer;
    n0 = (down ? outer : inner) * TC;
    seg = __builtin_amdgcn_readfirstlane(seg);
    begin = __shfl(beg, l) + in_seg * TR;
    cnt = min(TR, __shfl(end, l) - begin);
  }
  begin = __builtin_amdgcn_readfirstlane(begin);
  cnt = __builtin_amdgcn_readfirstlane(cnt);
  n0 = __builtin_amdgcn_readfirstlane(n0);

  const char* a_src = uniform_ptr(g.A);
  const char* b_src = uniform_ptr(reinterpret_cast<const char*>(g.B) + (int64_t)seg * g.b_seg_stride * 2);
  const uint32_t pitch_a = (uint32_t)(g.lda * 2), pitch_b = (uint32_t)(g.ldb * 2);
  const int nsteps = (MODE == SLABS ? g.K : g.slab) / KS;
  const int n_w = nsteps > wv ? (nsteps - wv + NW - 1) / NW : 0;
  uint32_t b_off[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int p = lane % LB::LPR, s = LB::RPI * j + lane / LB::LPR;
    b_off[j] = __umul24((uint32_t)s, pitch_b) + (uint32_t)(n0 * 2 + (((p >> 1) ^ LB::f(s)) * 32) + (p & 1) * 16);
  }
  auto issue_b = [&](int t, int u) {                              // step t of this wave -> stage u = t % NST
    const uint32_t at = ring + (uint32_t)(u * STAGE + A_BYTES), k = (uint32_t)(KS * (wv + NW * t)) * pitch_b;
#pragma unroll
    for (int j = 0; j < NB; ++j) dma16(b_src, b_off[j] + k, at + (uint32_t)(j * 1024));
  };
  // (B does not depend on the row numbers: it is requested ahead of them)
#pragma unroll
  for (int u = 0; u < NST; ++u)
    if (u < n_w) issue_b(u, u);
  uint32_t a_off[NA];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int r = 16 * j + (lane >> 2), p = begin + min(r, cnt - 1);       // rows past the end: the last one, never stored
    a_off[j] = __umul24((uint32_t)(MODE == ROUTE ? __shfl(rows, min(r, cnt - 1)) : MODE != SLABS && g.a_gather ? g.idx[p] : p), pitch_a) + (uint32_t)(((lane & 3) ^ ((r >> 2) & 3)) * 16);
  }
  auto issue_a = [&](int t, int u) {
    const uint32_t at = ring + (uint32_t)(u * STAGE), k = (uint32_t)(KS * (wv + NW * t)) * 2u;
#pragma unroll
    for (int j = 0; j < NA; ++j) dma16(a_src, a_off[j] + k, at + (uint32_t)(j * 1024));
  };

  const int s_rd = 8 * (lane >> 4) + ((lane >> 2) & 3), xa = (lane >> 2) & 3;
  const uint32_t a_rd = ring + (uint32_t)((lane & 15) * 64 + (((lane >> 4) ^ xa) << 4));
  uint32_t b_rd[FB];
#pragma unroll
  for (int c = 0; c < FB; ++c) b_rd[c] = ring + (uint32_t)(A_BYTES + s_rd * TC * 2 + ((c ^ LB::f(s_rd)) * 32) + (lane & 3) * 8);
  struct Frags { u32x4_t a[FA], b[FB]; };
  auto read_frags = [&](int u, Frags& fr) {
    const uint32_t so = (uint32_t)(u * STAGE);
#pragma unroll
    for (int c = 0; c < FA; ++c) fr.a[c] = lds_read_frag(a_rd + so + (uint32_t)(c * 1024));
#pragma unroll
    for (int c = 0; c < FB; ++c) {
      const uint2 lo = lds_tr(b_rd[c] + so), hi = lds_tr(b_rd[c] + so + 4 * TC * 2);
      fr.b[c] = u32x4_t{lo.x, lo.y, hi.x, hi.y};
    }
  };
  f32x4_t acc[CH][FB][FA];                                 // chain x of a wave: its steps x, x + CH, ..
#pragma unroll
  for (int x = 0; x < CH; ++x)
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int j = 0; j < FA; ++j) acc[x][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto mfmas = [&](const Frags& fr, f32x4_t (&to)[FB][FA]) {
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int j = 0; j < FA; ++j) to[i][j] = mfma16r<BF>(fr.b[i], fr.a[j], to[i][j]);
  };
  if (n_w > 0) {
#pragma unroll
    for (int u = 0; u < NST; ++u)
      if (u < n_w) issue_a(u, u);
  }
  // SLABS: which rows of the tile each slab lists, as bits (the first operands are on their way meanwhile)
  if constexpr (MODE == SLABS) {
    build_slab_masks<(TR < 32 ? 32 : TR), NW>(g, begin, s_mask, tid);
  }
  const uint32_t per_k = 0xffffffffu / (uint32_t)g.slab + 1u;      // k / slab by its reciprocal: exact below 2^32 / slab
  auto slab_of = [&](int t) { return (int)__umulhi((uint32_t)(KS * (wv + NW * t)), per_k); };
  auto listed = [&](int t, int c) -> bool {                // is this lane's row of block c listed for step t?
    return (s_mask[slab_of(t) * MW + (c >> 1)] >> ((c & 1) * 16 + (lane & 15))) & 1u;
  };
  auto mask_rows = [&](int t, Frags& fr) {
    if constexpr (MODE == SLABS) {
#pragma unroll
      for (int c = 0; c < FA; ++c) {
        fr.a[c] &= listed(t, c) ? 0xffffffffu : 0u;
      }
    }
  };
  if (n_w > 0) {
    // under way after the wait for a step: the loads of the next one (of step 1 ahead of step 0's wait its A loads: the B loads of
    // both were issued before)
    if (n_w > 1) PIT_WAIT_VMCNT(NA);
    else PIT_WAIT_VMCNT(0);
    Frags fr;
    int t = 0;
    if constexpr (MODE == SLABS) {
      // Steps whose slab lists no row of the tile would add zeros.  Where an eighth of them or more do, the wave takes the first two, which
      // are under way, and those that list a row (bits of `rest`; the lanes look at a step each).  Index and product, us, all steps / those,
      // 1 % kept: 1050 x 1952 x 1536, 1 x 32 27.3 / 22.5, 775 x 3584 x 768, 1 x 128 25.7 / 21.9.  A loop over such steps in every case takes longer
      // where few are left out: 1024^3, 1 x 32, 10 % kept 16.8 / 17.5.
      uint32_t any = 0u;
#pragma unroll
      for (int w = 0; w < MW; ++w) any |= lane < n_w ? s_mask[slab_of(lane) * MW + w] : 0u;
      uint64_t rest = __ballot(any != 0u) & ~3ull;
      if (n_w <= 64 && 8 * (__builtin_popcountll(rest) + 2) <= 7 * n_w) {
        auto next = [&]() -> int {                         // n_w: none
          if (rest == 0ull) return n_w;
          const int step = __builtin_ctzll(rest);
          rest &= rest - 1ull;
          return step;
        };
        int s[2] = {0, 1}, ahead[2] = {next(), next()};    // in the stages; the steps after those
        for (; ahead[1] < n_w; ahead[0] = next(), ahead[1] = next()) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            read_frags(u, fr);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_a(ahead[u], u);
            issue_b(ahead[u], u);
            mask_rows(s[u], fr);
            mfmas(fr, acc[0]);
            PIT_WAIT_VMCNT(LOADS);
            s[u] = ahead[u];
          }
        }
        const bool third = ahead[0] < n_w;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          if (u < 2 || third) {                            // (n_w >= 3 here)
            read_frags(u & 1, fr);
            if (u == 0 && third) {
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
              issue_a(ahead[0], 0);
              issue_b(ahead[0], 0);
            }
            mask_rows(u == 2 ? ahead[0] : s[u], fr);
            mfmas(fr, acc[0]);
            if (u == 0 && third) PIT_WAIT_VMCNT(LOADS);
            else PIT_WAIT_VMCNT(0);
          }
        }
        t = n_w;
      }
    }
    for (; t + 3 < n_w; t += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        read_frags(u, fr);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read
        issue_a(t + u + 2, u);
        issue_b(t + u + 2, u);
        mask_rows(t + u, fr);
        mfmas(fr, acc[u % CH]);
        PIT_WAIT_VMCNT(LOADS);
      }
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {                          // the last three steps at most
      if (t + u < n_w) {
        read_frags(u & 1, fr);
        if (u == 0 && t + 2 < n_w) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          issue_a(t + 2, 0);
          issue_b(t + 2, 0);
        }
        mask_rows(t + u, fr);
        mfmas(fr, acc[u % CH]);
        if (u == 0 && t + 2 < n_w) PIT_WAIT_VMCNT(LOADS);
        else PIT_WAIT_VMCNT(0);
      }
    }
    if constexpr (MODE == SLABS) {
      // An infinity or a NaN in B must not reach the rows that are not listed.  It reaches all rows of its column here (0 x inf is a
      // NaN), so sums that are all finite met none; otherwise the wave takes its steps again and keeps each one's results for the
      // rows that it lists.  The others keep what they had, which is what adding zeros gives: the same roundings both times, so
      // sums that meet no infinity have the same bits whether another one does or not.
      float big = 0.f;
#pragma unroll
      for (int i = 0; i < FB; ++i)
#pragma unroll
        for (int j = 0; j < FA; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) big = fmaf(acc[0][i][j][e], 0.f, big);    // 0 or a NaN
      if (__any(big != 0.f)) {
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
          for (int j = 0; j < FA; ++j) acc[0][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (t = 0; t < n_w; ++t) {
          issue_a(t, 0);
          issue_b(t, 0);
          PIT_WAIT_VMCNT(0);
          read_frags(0, fr);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
          for (int j = 0; j < FA; ++j) {
            const bool on = listed(t, j);
#pragma unroll
            for (int i = 0; i < FB; ++i) {
              const f32x4_t p = mfma16r<BF>(fr.b[i], fr.a[j], acc[0][i][j]);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[0][i][j][e] = on ? p[e] : acc[0][i][j][e];
            }
          }
        }
      }
    }
  }

  auto leave = [&](const f32x4_t (&from)[FB][FA], int slot) {          // a chain's partial tile -> LDS
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int j = 0; j < FA; ++j)
        *(PIT_LDS f32x4_t*)(uintptr_t)(lds0 + (uint32_t)(slot * PART) + partial_place<TC, FA>(16 * j + (lane & 15), 4 * i + (lane >> 4))) = from[i][j];
  };
  // a partial tile per chain, or, where they don't fit into the rings' place, per wave
  constexpr int TILES = CH * NW * PART <= RING ? CH : 1;
  if constexpr (TILES < CH) {
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int j = 0; j < FA; ++j) acc[0][i][j] += acc[1][i][j];
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < TILES; ++x) leave(acc[x], x * NW + wv);
  constexpr int VPR = TC / 4, VECS = TR * VPR, PER = (VECS + 64 * NW - 1) / (64 * NW);
  int crow[PER];
  float scale[PER];
#pragma unroll
  for (int v = 0; v < PER; ++v) {
    const int m = (tid + 64 * NW * v) / VPR;
    const int tok = MODE == ROUTE ? __shfl(rows, min(m, cnt - 1)) : 0;
    if constexpr (MODE == ROUTE) crow[v] = m < cnt ? tok : -1;
    else if constexpr (MODE == SLABS) crow[v] = m < cnt ? begin + m : -1;
    else crow[v] = m < cnt ? (g.c_scatter ? g.idx[begin + m] : begin + m) : -1;
    scale[v] = EPI == EPI_STORE && MODE != ONE && MODE != SLABS && g.gate && m < cnt ? g.gate[crow[v]] : 1.f;
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < PER; ++v) {
    const int x = tid + 64 * NW * v, m = x / VPR, c = x % VPR;
    if (crow[v] < 0 || x >= VECS) continue;
    const uint32_t at = lds0 + partial_place<TC, FA>(m, c);
    f32x4_t part[TILES * NW];
#pragma unroll
    for (int w = 0; w < TILES * NW; ++w) part[w] = *(PIT_LDS f32x4_t*)(uintptr_t)(at + (uint32_t)(w * PART));
    f32x4_t s = part[0];
#pragma unroll
    for (int w = 1; w < TILES * NW; ++w) s += part[w];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (EPI == EPI_GELU) s[e] = gelu_erf_fast(s[e]);
      if constexpr (EPI == EPI_STORE && MODE != ONE && MODE != SLABS) s[e] *= scale[v];
    }
    const int64_t o = (int64_t)crow[v] * g.ldc + n0 + 4 * c;
    if constexpr (CT == 0) *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(g.C) + o) = s;
    else *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(g.C) + o) = u32x2_t{pack2_in<BF>(s[0], s[1]), pack2_in<BF>(s[2], s[3])};
  }
}

template <bool BF, int EPI, int CT, int TR, int TC, int NW, int MODE>
int launch_tile(const GemmArgs& g, int64_t total_rows, hipStream_t st) {
  // (where unlisted rows are to be cleared, one workgroup more for every 64 rows of C: whatever the list holds, none without a tile
  // looks at more than a chunk of 64 rows.  With 8 more, a full list of 4070 rows: 13.2 us instead of 6.)
  const int64_t row_tiles = MODE != ONE && MODE != SLABS ? std::min<int64_t>(total_rows, total_rows / TR + g.nseg) : ceil_div(total_rows, TR);
  const int64_t wgs = row_tiles * (g.N / TC) + (g.zero_rest ? ceil_div(g.M, 64) : 0);
  hipLaunchKernelGGL((k_gather_m_ring<BF, EPI, CT, TR, TC, NW, MODE>), dim3((unsigned)wgs), dim3(64 * NW), 0, st, g);
  PIT_LAUNCH_CHECK();
  return PIT_OK;
}
template <bool BF, int EPI, int CT, int MODE>
int launch_mode(const GemmArgs& g, int64_t total_rows, RingMTile tile, hipStream_t st) {
  if constexpr (MODE == ONE || MODE == SLABS) {
    switch (tile) {
      case RINGM_32x32: return launch_tile<BF, EPI, CT, 32, 32, 8, MODE>(g, total_rows, st);
      case RINGM_32x64_8: return launch_tile<BF, EPI, CT, 32, 64, 8, MODE>(g, total_rows, st);
      case RINGM_64x64: return launch_tile<BF, EPI, CT, 64, 64, 4, MODE>(g, total_rows, st);
      case RINGM_64x64_8: return launch_tile<BF, EPI, CT, 64, 64, 8, MODE>(g, total_rows, st);
      default: return PIT_EINVAL;
    }
  } else {
    switch (tile) {
      case RINGM_16x32: return launch_tile<BF, EPI, CT, 16, 32, 8, MODE>(g, total_rows, st);
      case RINGM_16x64: return launch_tile<BF, EPI, CT, 16, 64, 4, MODE>(g, total_rows, st);
      case RINGM_16x64_8: return launch_tile<BF, EPI, CT, 16, 64, 8, MODE>(g, total_rows, st);
      case RINGM_32x64: return launch_tile<BF, EPI, CT, 32, 64, 4, MODE>(g, total_rows, st);
      case RINGM_64x64:                                    // (more than 150 rows per segment: never ROUTE)
        if constexpr (MODE == SEGMENTS) return launch_tile<BF, EPI, CT, 64, 64, 4, MODE>(g, total_rows, st);
        return PIT_EINVAL;
      default: return PIT_EINVAL;
    }
  }
}
template <bool BF, int MODE>
int launch_bf(int epi, int ct, const GemmArgs& g, int64_t rows, RingMTile tile, hipStream_t st) {
  if constexpr (MODE != ONE)
    if (epi == EPI_GELU) return ct ? launch_mode<BF, EPI_GELU, 1, MODE>(g, rows, tile, st) : PIT_EINVAL;
  if (epi != EPI_STORE) return PIT_EINVAL;
  return ct ? launch_mode<BF, EPI_STORE, 1, MODE>(g, rows, tile, st) : launch_mode<BF, EPI_STORE, 0, MODE>(g, rows, tile, st);
}
template <bool BF>
int launch_any(int epi, int ct, const GemmArgs& g, int64_t rows, RingMTile tile, hipStream_t st) {
  if (g.route != nullptr) return launch_bf<BF, ROUTE>(epi, ct, g, rows, tile, st);
  return g.b_seg_stride != 0 ? launch_bf<BF, SEGMENTS>(epi, ct, g, rows, tile, st) : launch_bf<BF, ONE>(epi, ct, g, rows, tile, st);
}

// number of segments that rows dealt at random would hit (the number that is hit is known on the device only)
double hit_segments(const GemmArgs& g, int64_t rows) { return g.nseg * (1.0 - std::pow(1.0 - 1.0 / g.nseg, (double)rows)); }

}  // namespace

// One B.  Tiles by how many of 64 x 64 there are if all rows are listed (how many are, the device knows): the smallest that gives
// a compute unit one workgroup at most, as in ring_tile, and four waves at 64 x 64 unless k is long, two workgroups per compute
// unit then.  Product alone, us, half of the rows listed: k_gather_m_lds / 32 x 32, 32 x 64, 64 x 64 with eight waves (four):
//   504 x 640 x 384 (48 tiles) 8.6 / 3.4, 4.0, 5.1;  1225 x 896 x 512 (160) 10.9 / 5.8, 4.7, 5.6;  384 x 896 x 2304 (216) 11.3 / -, -, 5.8 (5.9);
//   2205 x 384 x 640 (350) 7.5 / -, -, 6.2 (5.0);  944 x 1024 x 2048 (480) 12.8 / -, -, 7.9 (6.9);  1323 x 512 x 2176 (714) 10.4 / -, -, 11.7 (9.0);
//   all rows listed: 602 x 1280 x 640 (100) 14.4 / -, 5.0, 6.3;  1463 x 512 x 1024 (368) 8.4 / -, -, 8.7 (6.4);  1956 x 256 x 1024 (496) 8.0 / -, -, 9.9
//   (7.2);  962 x 640 x 2432 (608) 11.2 / -, -, 13.2 (10.5);  1003 x 256 x 2560 (640) 8.3 / -, -, 11.5 (8.6): the line is at 576.
//   Over 60 padded layers drawn over 1 - 48 sequences of 48 - 512, 256 - 2048 -> 256 - 4096, whole calls: 0.70, none slower.
//
// A B per segment.  hit = the segments with a row to be expected, per = rows of one of them, t16 = workgroups of 16 x 64 tiles to be
// expected, wide = rounds of k_gather_m_lds' 128 x 256 tiles (two per compute unit).  Whole calls, us, where the line is crossed:
//   t16 <= 0.4 cus   16 x 32, eight waves: 3 tokens, 1024 x 4096, 8 experts, second product by 16 x 64 / 16 x 32 15.5 / 14.0;  13, 640 x 1920, 128
//                    experts (130) 16.3 / 18.1
//   t16 <= cus       16 x 64, eight waves: 40 tokens, 768 x 2304, 32 experts (192) by four / eight 24.6 / 24.3
//   weights beyond 330 MB: both kernels run at the memory's rate, that one a little better with rows of 512 bytes (64 tokens on 64 experts
//                    of 1024 x 4096: 185 / 200)
//   per > 150        64 x 64 where k_gather_m_lds has a sixth of a round: 4612 tokens, 256 x 1024, 16 experts, second product 32.2 / 29.3 (0.10); 3371,
//                    768 x 2304, 8 55.7 / 60.4 (0.20)
//   the tiles read 500 MB or more from L2: 4096 tokens, 768 x 3072, 64 experts 157 / 195 (first product), 175 (second)
//   wide             per <= 16: up to 1.17 (482, 768 x 1536, 128: 118 / 108);  per <= 64: 0.94 (2595, 512 x 1024, 64: 51.1 / 46.7 and 2916, 512 x 1536, 64
//                    60.3 / 61.9 at 1.02);  per <= 150: 0.22 (4646, 384 x 1536, 32, first product 44.7 / 51.0 at 0.80, second 44.8 / 44.1)
//   16 rows a tile up to 12 per segment, else 32: 721, 640 x 1280, 128 (7) 84.1 by 32, 83.0 by 16; 459, 768 x 3072, 16 (29) 51.5, 54.4
// Over 120 calls of 1 - 8192 tokens and 120 of 3 - 200, 256 - 1024 wide, 8 - 128 experts: 0.83 and 0.81 of the time before, 4 slower by more than 2 % (1551 tokens, 512 x
// 1024, 128 experts 59.4 / 62.6; besides 152, 1024 x 4096, 8 36.3 / 37.5 and 24, 1024 x 2048, 128 25.7 / 26.9, which no tile here gives).  Each product of 190 such calls by every tile:
// the best one every time takes 0.985 of this rule.
RingMTile ring_m_tile(int epi, const GemmArgs& g, int64_t total_rows) {
  const double cus = compute_units(), rows = (double)total_rows;
  if (g.b_seg_stride == 0) {
    if (g.nseg != 1 || epi != EPI_STORE || g.gate != nullptr) return RINGM_NONE;
    const double t64 = (double)ceil_div(total_rows, 64) * (g.N / 64);
    if (4 * t64 <= cus) return RINGM_32x32;
    if (2 * t64 <= cus) return RINGM_32x64_8;
    if (g.K > 1024 && t64 <= cus) return RINGM_64x64_8;
    return 4 * t64 <= 9 * cus ? RINGM_64x64 : RINGM_NONE;
  }
  const double hit = hit_segments(g, total_rows), per = rows / hit, t16 = std::max(hit, 0.5 * hit + rows / 16) * (g.N / 64);
  if (t16 <= 0.4 * cus) return RINGM_16x32;
  if (t16 <= cus) return RINGM_16x64_8;
  if (g.nseg > 512 && total_rows <= g.nseg) return RINGM_16x64;    // (k_gather_m_lds visits all segments to find a tile's)
  if (hit * g.N * g.slab * 2.0 > 330e6) return RINGM_NONE;
  const double wide = (rows / 128 + hit) * (g.N / 256.0) / (2 * cus);
  if (per > 150) return wide <= 0.16 ? RINGM_64x64 : RINGM_NONE;
  const int R = per <= 12 ? 16 : 32;
  const bool few = std::min(rows, hit + (double)(total_rows / 16)) * (g.N / 64) <= 2 * cus && (g.N >= 512 || per <= 16) && hit * g.N * g.slab * 2.0 <= 200e6;
  if (!few && (rows / R + hit) * (g.N / 64) * (R + 64) * 2.0 * g.slab > 500e6) return RINGM_NONE;
  if (wide > (per <= 16 ? 1.17 : per <= 64 ? 0.94 : 0.22)) return RINGM_NONE;
  return R == 16 ? RINGM_16x64 : RINGM_32x64;
}

// Up to 64 tokens the index's launch (3 us) is saved, except where k_gather_m_lds takes a product or much is read (300 MB; the index of
// more than 512 experts is two launches and is always saved).
bool gather_m_routes(const GemmArgs& g) {
  if (g.M > 64 || g.b_seg_stride == 0 || ring_m_tile(EPI_STORE, g, g.M) == RINGM_NONE) return false;
  return g.nseg > 512 || hit_segments(g, g.M) * g.N * g.slab * 2.0 <= 300e6;
}

// Micro-tiles along k: all rows of a tile are multiplied, those that a slab does not list as zeros, where that takes less time than
// strips of C in LDS over the listed rows alone (pit_slab.hip): the strips' time is their chain of list searches and visits.  How
// many rows are listed the device knows.  Product alone, us, strips / 32 x 32, 32 x 64, 64 x 64 by four waves, by eight (rows listed in %):
//   327 x 3648 x 256, 1 x 64 (30 %, 24 tiles of 64 x 64) 24.5 / 12.0, 13.9, 17.2, 14.2;  930 x 2496 x 256, 1 x 64 (6 %, 60) 17.7 / 9.9, 9.9, 13.7, 11.9
//   538 x 1984 x 768, 1 x 64 (10 %, 108) 13.9 / 11.5, 9.4, 11.3, 11.0;  401 x 832 x 1408, 1 x 64 (46 %, 154) 11.8 / 14.7, 15.0, 8.9, 8.7
//   1024^3, 1 x 32 (10 %, 256) 12.2 / 17.5, 15.3, 9.4, 9.7;  1229 x 3072 x 512, 1 x 32 (8 %, 160) 29.4 / 31.5, 30.4, 22.0, 19.6
// (Those times are without the steps left out in the kernel.)  The line is at one workgroup of 64 x 64 per compute unit: beyond it the
// strips are ahead where few rows are listed (2097 x 1216 x 512, 1 x 64, 1 %, 264 tiles: 10.0 / 11.2 by four waves; 755 x 3456 x 1536, 1 x 128,
// 11 %, 288: 22.9 / 25.2), but for the 32-wide slabs that cost them most (1669 x 1984 x 640, 16 %, 270: 24.6 / 19.5; 321 x 1568 x 3456, 4 %, 324: 21.2 /
// 14.8; 2295 x 1504 x 768, 7 %, 432: 20.9 / 17.3; not with a long k: 488 x 4032 x 2816, 2 %, 352: 28.2 / 34.3).  Index and product of 100
// drawn calls, 300 - 4096 x 512 - 4096 x 256 - 4096, 1 - 50 % kept, against strips in all of them: 0.92, none more than 2 % slower; the slowest looked for, at 1 %
// and slabs of 128: 775 x 3584 x 768 20.0 / 21.8, 1529 x 512 x 384 12.9 / 13.4.
RingMTile ring_slab_tile(const GemmArgs& g) {
  const int64_t cus = compute_units(), t64 = ceil_div(g.M, 64) * (g.N / 64);
  if (g.nseg > SLABS_MAX || g.K > (1 << 16)) return RINGM_NONE;
  if (4 * t64 <= cus) return RINGM_32x32;
  if (2 * t64 <= cus) return RINGM_32x64_8;
  if (t64 <= cus) return g.K > 2048 ? RINGM_64x64_8 : RINGM_64x64;
  return g.slab == 32 && 4 * t64 <= 7 * cus && g.K <= 2048 ? RINGM_64x64 : RINGM_NONE;
}

int launch_slab_ring(bool bf, const GemmArgs& g, RingMTile tile, hipStream_t st) {
  return bf ? launch_mode<true, EPI_STORE, 0, SLABS>(g, g.M, tile, st) : launch_mode<false, EPI_STORE, 0, SLABS>(g, g.M, tile, st);
}

int launch_gather_m_ring(bool bf, int epi, int c_is_in_type, const GemmArgs& g, int64_t total_rows, RingMTile tile, hipStream_t st) {
  return bf ? launch_any<true>(epi, c_is_in_type, g, total_rows, tile, st) : launch_any<false>(epi, c_is_in_type, g, total_rows, tile, st);
}

}  // namespace pit
