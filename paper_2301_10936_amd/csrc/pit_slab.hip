// GATHER_M with several k-slabs per row (1 x mt micro-tiles of a row-major A): SRead -> MFMA -> SWrite with C in LDS
// (paper Section 3.1, sparse kernel template), for gfx950.  bf16 or f16 inputs, fp32 accumulation and results.
//   k_slab_strip       strips of 32 x 128 (four per workgroup, added at the end)
//   k_slab_strip_tall  the same for products that fill the chip with strips of 64 or 128 rows
//   (k_gather_m_ring, pit_gemm_m_ring.hip, takes products with few tiles: ring_slab_tile)
// Which one: the rule is at launch_slab_strip_bf.
#include "pit_gemm.hpp"
#include "pit_gemm_dev.hpp"

namespace pit {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------------
// GATHER_M with micro-tiles along k (several k-slabs per row: 1 x mt micro-tiles of a row-major A).
//
// The rows listed for slab s differ from those of slab s', so the partial products of the slabs
// have to meet in C.  Here C stays put: a workgroup owns a strip of R rows x W columns of C
// (R x W = 4096: 64 x 64, or 32 x 128) and walks ALL slabs; per slab it gathers the strip's listed
// rows (SRead along m inside the strip, in blocks of 16 rows), multiplies them with the slab's rows
// of B on v_mfma_f32_16x16x32, and adds the result to the strip held in LDS.  The four waves take
// the slabs round-robin, each with a strip of its own (no atomics, no races); at the end the four
// strips are added in a fixed order and the whole strip is stored, rows that nothing touched as
// zeros.  So the result does not depend on the order in which anything ran, and C needs no clearing
// beforehand.  B is read once per strip of rows, so its traffic falls with R; A is read once per
// strip of columns.
//   rows of a slab inside the strip: the slab's list is ascending, so they are one contiguous run
//   of it; a 64-ary search by the wave finds where the run starts, two 64-entry loads hold it.
//   A operand: 16 bytes (8 k) of a listed row per lane -- already the operand layout.
//   B operand: 8 k-rows x CW columns (CW = W / 16) per lane, transposed inside the lane.
//   strip in LDS: a lane moves the CW columns it holds of a row as 16-byte vectors and the 16
//   lanes of a row lie side by side; a spare row swallows the results of unused block rows.
// ------------------------------------------------------------------------------------------------
constexpr int SS_BATCH = 8;                          // slabs per wave whose row lookups are in flight together
static_assert(SS_BATCH == 8, "the lane layout of the list-bounds load assumes 8");
template <int CW> struct StripShape {
  static_assert(CW == 4 || CW == 8, "columns per lane");
  static constexpr int W = 16 * CW;                  // columns of C per workgroup
  static constexpr int R = 4096 / W;                 // rows of C per workgroup (at most 64: one lane per listed row)
  static constexpr int FLOATS = (R + 1) * W;         // one wave's strip, with the spare row
};

// CW 16-bit columns of one k-row, as loaded
template <int CW> struct BRow { uint32_t d[CW / 2]; };
template <int CW>
__device__ __forceinline__ BRow<CW> load_brow(const char* base, uint32_t byte_off) {
  BRow<CW> r;
  if constexpr (CW == 8) {
    const uint4 v = load16(base, byte_off);
    r.d[0] = v.x; r.d[1] = v.y; r.d[2] = v.z; r.d[3] = v.w;
  } else {
    typedef const u32x2_t __attribute__((address_space(1))) * gptr_t;
    const u32x2_t v = *(gptr_t)(uintptr_t)(reinterpret_cast<uintptr_t>(base) + byte_off);
    r.d[0] = v[0]; r.d[1] = v[1];
  }
  return r;
}
// 8 consecutive k of column x out of 8 k-rows (4 v_perm_b32)
template <int CW>
__device__ __forceinline__ uint4 bcolumn(const BRow<CW> (&r)[8], int x) {
  const uint32_t sel = (x & 1) ? 0x07060302u : 0x05040100u;
  uint32_t d[4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) d[jj] = __builtin_amdgcn_perm(r[2 * jj + 1].d[x >> 1], r[2 * jj].d[x >> 1], sel);
  return make_uint4(d[0], d[1], d[2], d[3]);
}

template <bool BF>
__device__ __forceinline__ f32x4_t mfma16(const uint4& a, const uint4& b, const f32x4_t& c) {
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

template <bool BF, int CW>
__global__ void __launch_bounds__(256, 2)
k_slab_strip(const GemmArgs g) {
  using SH = StripShape<CW>;
  constexpr int SS_RM = SH::R;
  __shared__ __attribute__((aligned(16))) float s_c[4][SH::FLOATS];
  __shared__ __attribute__((aligned(16))) int s_rows[4][SS_BATCH][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 15, kb = lane >> 4;
  const int n0 = blockIdx.x * SH::W;
  const int r0 = blockIdx.y * SS_RM;
  float* strip = s_c[wv];
  for (int i = lane * 4; i < SH::FLOATS; i += 256) *reinterpret_cast<f32x4_t*>(strip + i) = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const char* a_src = uniform_ptr(g.A);
  const char* b_src = uniform_ptr(g.B);
  const uint32_t pitch_a = (uint32_t)(g.lda * 2), pitch_b = (uint32_t)(g.ldb * 2);
  const uint32_t b_lane = __umul24((uint32_t)(8 * kb), pitch_b) + (uint32_t)(n0 + CW * q) * 2u;
  const int ksteps = g.slab / 32;                   // items per block of a slab
  const int nsl = g.nseg > wv ? (g.nseg - wv + 3) >> 2 : 0;   // this wave's slabs: wv, wv + 4, ...

  for (int j0 = 0; j0 < nsl; j0 += SS_BATCH) {
    // ---- which rows of the strip does each slab of the batch list?  rowsel[j]: lane i < cnt[j]
    //      holds the i-th of them (ascending)
    int rowsel[SS_BATCH], cnt[SS_BATCH];
    int lo[SS_BATCH], hi[SS_BATCH], end[SS_BATCH];
    // one vector load brings the batch's list bounds: lane j the start of slab j's list, lane 8 + j its end
    // (slabs past the last: slab 0 stands in, so that nothing branches)
    const int pv = g.seg_ptr[(j0 + (lane & 7) < nsl ? wv + 4 * (j0 + (lane & 7)) : 0) + ((lane >> 3) & 1)];
#pragma unroll
    for (int j = 0; j < SS_BATCH; ++j) {
      const bool valid = j0 + j < nsl;                         // slabs past the end: empty
      lo[j] = valid ? __builtin_amdgcn_readlane(pv, j) : 0;
      end[j] = valid ? __builtin_amdgcn_readlane(pv, SS_BATCH + j) : 0;
      hi[j] = end[j];
    }
    // 64-ary search for p* = the first position whose entry is >= r0.  Invariant: lo <= p* <= hi, every
    // entry before lo is below r0, the entry at hi (if hi < end) is not.  All slabs of the batch advance
    // together, one round trip to memory per round.
    for (;;) {
      bool any_wide = false;
#pragma unroll
      for (int j = 0; j < SS_BATCH; ++j) any_wide |= hi[j] - lo[j] > 64;
      if (!any_wide) break;
      // every slab of the batch takes the round (it leaves a narrow range correct and no wider), so the code
      // is free of branches and the eight loads are in flight together; entry 0 exists because some list is wide
      int smp[SS_BATCH], step[SS_BATCH];
#pragma unroll
      for (int j = 0; j < SS_BATCH; ++j) {
        step[j] = (hi[j] - lo[j] + 63) / 64;
        const int pos = lo[j] + lane * step[j];
        const int v = g.idx[max(min(pos, hi[j] - 1), 0)];
        smp[j] = pos < hi[j] ? v : 0x7fffffff;
      }
#pragma unroll
      for (int j = 0; j < SS_BATCH; ++j) {
        const int c = __popcll(__ballot(smp[j] < r0));        // samples below the strip: a prefix
        const int hi_new = (c < 64 && lo[j] + c * step[j] < hi[j]) ? lo[j] + c * step[j] : hi[j];
        hi[j] = c == 0 ? lo[j] : hi_new;
        lo[j] = c == 0 ? lo[j] : lo[j] + (c - 1) * step[j] + 1;
      }
    }
    // the run of entries inside [r0, r0 + R) starts at most 64 positions after lo and is at most R <= 64 long
    int e0[SS_BATCH], e1[SS_BATCH];
#pragma unroll
    for (int j = 0; j < SS_BATCH; ++j) {
      const int p0 = lo[j] + lane, p1 = lo[j] + 64 + lane;
      e0[j] = p0 < end[j] ? g.idx[p0] : 0x7fffffff;
      e1[j] = p1 < end[j] ? g.idx[p1] : 0x7fffffff;
    }
#pragma unroll
    for (int j = 0; j < SS_BATCH; ++j) {
      const bool in0 = e0[j] >= r0 && e0[j] < r0 + SS_RM, in1 = e1[j] >= r0 && e1[j] < r0 + SS_RM;
      const unsigned long long b0 = __ballot(in0), b1 = __ballot(in1);
      const unsigned long long below = (1ull << lane) - 1ull;
      const int rank0 = __popcll(b0 & below), rank1 = __popcll(b0) + __popcll(b1 & below);
      // forward permutes: an in-range entry goes to the lane of its rank; the other lanes send a zero to a
      // lane that no entry of the same permute goes to (lane 63, which only a full first vector reaches, and
      // then every lane has an entry; for the second vector lane 0 when the ranks reach 63: the first vector
      // then holds rank 0, or the second is full)
      cnt[j] = __popcll(b0) + __popcll(b1);
      const int idle1 = cnt[j] == 64 ? 0 : 63;
      int got = 0;
      {
        const int a = __builtin_amdgcn_ds_permute((in0 ? rank0 : 63) * 4, in0 ? e0[j] + 1 : 0);
        const int b = __builtin_amdgcn_ds_permute((in1 ? rank1 : idle1) * 4, in1 ? e1[j] + 1 : 0);
        got = a | b;
      }
      rowsel[j] = got - 1;                              // -1 where no entry arrived
    }

    // ---- hand the row lists to the item loop through LDS (so that a slab can be picked at run time)
    uint32_t live = 0;
#pragma unroll
    for (int j = 0; j < SS_BATCH; ++j) {
      s_rows[wv][j][lane] = rowsel[j];
      live |= cnt[j] > 0 ? 1u << j : 0u;
    }
    if (live == 0) continue;

    // ---- one item = one 32-k step of one block (16 listed rows) of one live slab; the loads of item
    //      t + 1 are in flight while item t is computed.  (A later block of a slab reads the slab's
    //      rows of B again, from the L1 that the first block has just filled.)
    struct Item { uint32_t k0, a; int c[4]; int j, b, nblk, ks; };
    struct Regs { uint4 ra; BRow<CW> rb[8]; };
    auto setup = [&](int j, int b, Item& T) {
      const int* rs = s_rows[wv][j];
      const int first = rs[0];                                  // live slab: lane 0 holds a listed row
      const int r_a = rs[16 * b + q];
      T.j = j; T.b = b; T.ks = 0;
      T.nblk = (__popcll(__ballot(rs[lane] >= 0)) + 15) >> 4;   // blocks of 16 listed rows
      T.k0 = (uint32_t)((wv + 4 * (j0 + j)) * g.slab);
      T.a = __umul24((uint32_t)(r_a < 0 ? first : r_a), pitch_a) + 16u * (uint32_t)kb;   // unused block rows re-read a listed row
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int x = rs[16 * b + 4 * kb + e];
        // float offset of (row, q) in the strip; unused rows: the spare row
        T.c[e] = (((x < 0 ? SS_RM : x - r0) * (CW / 4)) * 16 + q) * 4;
      }
    };
    auto loads = [&](const Item& T, Regs& R) {
      const uint32_t k = T.k0 + 32u * (uint32_t)T.ks;
      R.ra = load16(a_src, T.a + 2u * k);
#pragma unroll
      for (int i = 0; i < 8; ++i) R.rb[i] = load_brow<CW>(b_src, b_lane + __umul24(k + (uint32_t)i, pitch_b));
    };
    f32x4_t acc[CW];
    // strip element (row, column CW q + x) lives at ((row * (CW / 4) + x / 4) * 16 + q) * 4 + x % 4: a lane
    // moves its columns of a row as 16-byte vectors, 16 lanes of a row side by side
    auto process = [&](const Item& T, const Regs& R) {
      if (T.ks == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < CW / 4; ++h) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(strip + T.c[e] + 64 * h);
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[4 * h + x][e] = v[x];
          }
      }
#pragma unroll
      for (int x = 0; x < CW; ++x) acc[x] = mfma16<BF>(R.ra, bcolumn<CW>(R.rb, x), acc[x]);
      if (T.ks == ksteps - 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < CW / 4; ++h)
            *reinterpret_cast<f32x4_t*>(strip + T.c[e] + 64 * h) =
                f32x4_t{acc[4 * h][e], acc[4 * h + 1][e], acc[4 * h + 2][e], acc[4 * h + 3][e]};
      }
    };
    // the item after T: the block's next k-step, else the slab's next block, else the next live slab.
    // After the last item the same item is named again: its loads are issued once more and dropped, so
    // that the loop holds no conditional load and every wait counts exactly the loads of the item after.
    auto copy_item = [&](const Item& T, Item& N) {
      N.k0 = T.k0; N.a = T.a; N.j = T.j; N.b = T.b; N.nblk = T.nblk; N.ks = T.ks;
#pragma unroll
      for (int e = 0; e < 4; ++e) N.c[e] = T.c[e];
    };
    auto advance = [&](const Item& T, Item& N) -> bool {
      if (T.ks + 1 < ksteps) { copy_item(T, N); N.ks = T.ks + 1; return true; }
      if (T.b + 1 < T.nblk) { setup(T.j, T.b + 1, N); return true; }
      if (live != 0) {
        const int j = __builtin_ctz(live);
        live &= live - 1;
        setup(j, 0, N);
        return true;
      }
      copy_item(T, N);
      return false;
    };
    Item T0, T1;
    Regs Ra, Rb;
    {
      const int j = __builtin_ctz(live);
      live &= live - 1;
      setup(j, 0, T0);
    }
    loads(T0, Ra);
    for (;;) {
      bool more = advance(T0, T1);
      loads(T1, Rb);
      process(T0, Ra);
      if (!more) break;
      more = advance(T1, T0);
      loads(T0, Ra);
      process(T1, Rb);
      if (!more) break;
    }
  }
  __syncthreads();
  // the four strips in a fixed order; thread (row, q) stores CW consecutive columns
  for (int i = tid; i < SS_RM * 16; i += 256) {
    const int row = i >> 4, qq = i & 15;
    if (r0 + row >= g.M) continue;
    float* d = reinterpret_cast<float*>(g.C) + (int64_t)(r0 + row) * g.ldc + n0 + CW * qq;
#pragma unroll
    for (int h = 0; h < CW / 4; ++h) {
      const int o = ((row * (CW / 4) + h) * 16 + qq) * 4;
      const f32x4_t v = ((*reinterpret_cast<const f32x4_t*>(&s_c[0][o]) + *reinterpret_cast<const f32x4_t*>(&s_c[1][o])) +
                         *reinterpret_cast<const f32x4_t*>(&s_c[2][o])) + *reinterpret_cast<const f32x4_t*>(&s_c[3][o]);
      *reinterpret_cast<float4*>(d + 4 * h) = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// The same product with tall strips, for products large enough to give every compute unit one.
//
// k_slab_strip reads B once per 32 rows of C and multiplies blocks of 16 rows of which, at 10 % density, three are
// real; its four waves each hold a strip, so strips cannot grow.  Here a workgroup owns R x 128 of C in LDS (fp32) and
// a wavefront owns 64 of the columns: rows are only ever touched by one wave (no atomics, no barrier
// between slabs, a fixed order of additions), and the strip is R = 128 rows high: B is read a quarter as often and the
// blocks of 16 rows are nearly full.  With SG = 2 two pairs of waves take every other slab into strips of
// their own that are added at the end.  Rows that nothing touched are stored as zeros.
// Rounding: a visit's products are summed from zero and then added to the strip, one rounding of the running sum per
// visit where the matrix unit makes one per eight products.  With 64 k per visit that makes one chain of additions more
// exact than k_slab_strip's four, with 32 k two chains (error against 64 bits, 4096^3, four chains / here: 1 x 64 at
// 10 % and 50 % 7.7e-8 / 6.8e-8 and 1.36e-7 / 1.15e-7; 1 x 32 7.3e-8 / 6.6e-8 and 1.34e-7 / 1.15e-7; one chain at 1 x 32:
// 7.7e-8 and 1.52e-7).  Hence SG = 2 with R = 128 as well where KS = 1.
//   list of a strip: lower bounds of its first row and of the row after it in every slab's ascending list,
//   searched 8-ary with one slab per lane (64 slabs at once: two waves, four round trips to memory for
//   lists of thousands); the rows are kept as bytes in LDS.
//   A operand: 16 bytes (8 k) of a listed row per lane -- already the operand layout.
//   B operand: 8 k-rows x 4 columns per lane (8-byte loads; 16 lanes side by side fill a 128-byte line of a
//   k-row), transposed inside the lane: MFMA x of a block works on the columns {4 q + x}.
//   strip in LDS: [wave][row][64 columns]; a lane moves its four columns of a row as 16 bytes and the 16 lanes
//   of a row lie side by side (no bank conflicts).  A spare row swallows the results of a block's unused rows.
// Bound by the vector L1 (rocprofv3, 4096^3, 1 x 64, 10 % kept): a visit takes 1900 clocks, in which a wave issues 105 vector,
// 14 LDS and 20 load instructions (430, 140 and 200 clocks of issue); a load of B is 20 accesses for 512 bytes, the L1
// serves 0.74 accesses per clock, its address unit is busy 69 % of the time, the matrix pipe 7 %.  One wave per SIMD:
// the strips fill the LDS.  4096^3, 1 x 64 micro-tiles, 10 % kept: 231 -> 111 us (50 %: 363 -> 267, 1 %: 112 -> 76; 1 x 32,
// 10 %: 339 -> 156; the launch without its slab loop: 18 us).
// Tried: waves of 32 columns, eight per CU (twice the load instructions: 121 us), R = 256 with four waves per CU (114),
// four chains in 64-row strips, one workgroup of eight waves per CU (205: B is read twice as often).
// ------------------------------------------------------------------------------------------------
constexpr int ST_W = 128;                            // columns of C per workgroup (2 waves x 64)
constexpr int ST_BATCH = 64;                         // slabs whose row lists are in LDS together (one lane each)

// KS = steps of 32 k taken per visit of a row (a slab's k extent is a multiple of 32 KS)
template <bool BF, int KS, int R, int SG>
__global__ void __launch_bounds__(128 * SG, 2)
k_slab_strip_tall(const GemmArgs g) {
  static_assert(R >= 32 && R <= 256 && R % 32 == 0, "rows of a strip are kept as bytes");
  static_assert(SG == 1 || SG == 2, "groups of two waves");
  constexpr int CW = 4, WC = 16 * CW;               // columns of a lane, of a wave
  constexpr int GW = ST_W / WC;                     // waves of a group
  constexpr int NW = GW * SG;
  __shared__ __attribute__((aligned(16))) float s_c[NW][(R + 1) * WC];
  __shared__ __attribute__((aligned(16))) uint8_t s_list[ST_BATCH][R];
  __shared__ int s_bound[2][ST_BATCH];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wv % GW, grp = wv / GW;
  const int q = lane & 15, kb = lane >> 4;
  int n0, r0;
  {
    // Consecutive workgroup ids go to different XCDs (8, own L2 each): renumber so that each takes a contiguous run of the
    // strips, the runs equal but for one strip, in bands of 4 tile columns x all rows.  (4 column groups x 2 row groups of
    // XCDs, us / here: 16 or 32 tile columns the same; 17, 3456 x 2048 x 2176, 58.9 / 35.3; 5, 11000 x 1024 x 640, 43.8 / 25.2;
    // 1, 60000 x 1024 x 128, 86.4 / 25.9: XCDs without work.)
    const int tn = g.N / ST_W, tm = (g.M + R - 1) / R, total = tn * tm;
    const int x = blockIdx.x & 7, lp = x * (total >> 3) + min(x, total & 7) + ((int)blockIdx.x >> 3);
    const int band = lp / (4 * tm), within = lp - band * (4 * tm), n = min(4, tn - 4 * band);
    n0 = (4 * band + within % n) * ST_W;
    r0 = within / n * R;
  }
  const int rows = min(R, g.M - r0);
  float* strip = s_c[wv];

  const uint32_t pitch_a = (uint32_t)(g.lda * 2), pitch_b = (uint32_t)(g.ldb * 2);
  const int cps = g.slab / (32 * KS);               // visits per slab
  // Both operands come through buffer loads: the lane's 32-bit offset stays in one register, the k position is a scalar
  // offset.  A lane of A without a listed row asks for an offset outside the buffer: it reads zero and moves nothing.
  constexpr uint32_t NO_ROW = 0xf0000000u;          // (rows of a strip lie within 2^31 bytes)
  const uint32_t b_lane = __umul24((uint32_t)(8 * kb), pitch_b) + (uint32_t)(n0 + WC * wc + CW * q) * 2u;
  const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(uniform_ptr(g.B)), 0, 0xffffffffu, 0x00020000);
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(uniform_ptr(reinterpret_cast<const char*>(g.A) + (int64_t)r0 * g.lda * 2)), 0,
      (uint32_t)(rows - 1) * pitch_a + (uint32_t)g.K * 2u, 0x00020000);

  for (int s0 = 0; s0 < g.nseg; s0 += ST_BATCH) {
    // ---- where the strip's rows lie in the lists of the batch's slabs: wave 0 looks for the first entry >= r0, wave
    //      1 for the first entry >= r0 + R, one slab per lane.  Invariant: lo <= p* <= hi, entries before lo are below the
    //      target, entries from hi on are not; a round leaves at most an eighth of a range.
    if (s0 != 0) __syncthreads();                   // the previous batch's lists have been read
    if (wv < 2) {
      const int s = min(s0 + lane, g.nseg - 1);
      const int target = wv == 0 ? r0 : r0 + R;
      int lo = g.seg_ptr[s], hi = g.seg_ptr[s + 1];
      while (__ballot(lo < hi) != 0ull) {
        const int step = (hi - lo + 7) >> 3;
        int v[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) v[k] = g.idx[max(min(lo + (k + 1) * step, hi) - 1, 0)];
        int below = 0;                              // probes below the target: a prefix of the valid ones
#pragma unroll
        for (int k = 0; k < 7; ++k) below += (lo + (k + 1) * step <= hi && v[k] < target) ? 1 : 0;
        const int nhi = below < 7 ? lo + (below + 1) * step - 1 : hi;   // (there is no eighth probe)
        lo += below * step;
        hi = max(lo, min(hi, nhi));
      }
      s_bound[wv][lane] = lo;
    }
    // (the strip is private to its wave; cleared while the searches travel)
    if (s0 == 0)
      for (int i = lane * 4; i < (R + 1) * WC; i += 256) *reinterpret_cast<f32x4_t*>(strip + i) = f32x4_t{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    // lane j: number of rows that slab j of the batch lists inside the strip
    const int begv = s_bound[0][lane];
    const int cntv = s0 + lane < g.nseg ? max(0, min(rows, s_bound[1][lane] - begv)) : 0;
    // the rows themselves, as bytes: wave w fills the lists of slabs w, w + NW, ..., eight at a time
#pragma unroll 1
    for (int j0 = 0; j0 < ST_BATCH / NW; j0 += 8) {
      int v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int slab = wv + NW * (j0 + j), beg = __builtin_amdgcn_readlane(begv, slab), n = __builtin_amdgcn_readlane(cntv, slab);
        v[j] = g.idx[max(beg + min(lane, n - 1), 0)];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int slab = wv + NW * (j0 + j), beg = __builtin_amdgcn_readlane(begv, slab), n = __builtin_amdgcn_readlane(cntv, slab);
        // (clamped: an index that breaks its own rules must not lead outside the strip)
        if (lane < n) s_list[slab][lane] = (uint8_t)max(0, min(v[j] - r0, rows - 1));
        if constexpr (R > 64)
          for (int i = lane + 64; i < n; i += 64) s_list[slab][i] = (uint8_t)max(0, min(g.idx[beg + i] - r0, rows - 1));
      }
    }
    __syncthreads();
    // slabs of this group with at least one listed row
    unsigned long long live = __ballot(cntv > 0);
    if constexpr (SG == 2) live &= 0x5555555555555555ull << grp;
    if (live == 0ull) continue;

    // ---- one visit = KS steps of 32 k of one live slab, all its listed rows.  The loads of the two visits after the one
    //      being computed are in flight; they cover the first two blocks of 16 rows (further blocks load their A rows one
    //      pair of blocks ahead).
    struct Visit { int j, c, n; };                  // slab of the batch, k chunk of the slab, listed rows
    struct Regs { u32x2_t b[8 * KS]; uint4 a[2][KS]; };
    auto next = [&](const Visit& u) -> Visit {      // after the last visit the same one is named again: its loads are repeated and dropped
      if (u.c + 1 < cps) return Visit{u.j, u.c + 1, u.n};
      if (live == 0ull) return u;
      const int j = __builtin_ctzll(live);
      live &= live - 1ull;
      return Visit{j, 0, __builtin_amdgcn_readlane(cntv, j)};
    };
    auto k_of = [&](const Visit& u) -> uint32_t { return (uint32_t)((s0 + u.j) * g.slab + u.c * (32 * KS)); };
    // this lane's offset of A for block b
    auto row_of = [&](const Visit& u, int b) -> uint32_t {
      const int pos = 16 * b + q;
      const uint32_t off = __umul24((uint32_t)s_list[u.j][min(pos, R - 1)], pitch_a) + 16u * (uint32_t)kb;
      return off | (pos < u.n ? 0u : NO_ROW);
    };
    auto load_a = [&](uint32_t k, uint32_t off, uint4 (&a)[KS]) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        a[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (int)off, (int)(2u * k + 64u * ks), 0));
    };
    // row i of the B rows of the visit that starts at k
    auto load_b = [&](uint32_t kp, int i) -> u32x2_t {
      const int so = (int)(kp + (uint32_t)(32 * (i >> 3) + (i & 7)) * pitch_b);
      return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(b_rsrc, (int)b_lane, so, 0));
    };
    // addresses (in floats) of the rows of C that this lane holds of block b
    auto c_at = [&](const Visit& u, int b, uint32_t rl, uint32_t (&at)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        at[e] = (16 * b + 4 * kb + e < u.n ? ((rl >> (8 * e)) & 255u) : (uint32_t)R) * (uint32_t)WC + (uint32_t)CW * (uint32_t)q;
    };
    auto rows4 = [&](const Visit& u, int b) -> uint32_t { return *reinterpret_cast<const uint32_t*>(&s_list[u.j][16 * b + 4 * kb]); };
    auto c_read = [&](const uint32_t (&at)[4], f32x4_t (&c)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = *reinterpret_cast<const f32x4_t*>(strip + at[e]);
    };
    auto c_write = [&](const uint32_t (&at)[4], const f32x4_t (&c)[4], const f32x4_t (&acc)[CW]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) *reinterpret_cast<f32x4_t*>(strip + at[e]) = c[e] + f32x4_t{acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
    };
    auto zero = [&](f32x4_t (&acc)[CW]) {
#pragma unroll
      for (int x = 0; x < CW; ++x) acc[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto mfmas = [&](const uint4 (&a)[KS], const uint4 (&bop)[KS][CW], f32x4_t (&acc)[CW]) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int x = 0; x < CW; ++x) acc[x] = mfma16<BF>(a[ks], bop[ks][x], acc[x]);
    };
    auto block = [&](const Visit& u, int b, const uint4 (&a)[KS], const uint4 (&bop)[KS][CW]) {
      uint32_t at[4];
      f32x4_t c[4], acc[CW];
      c_at(u, b, rows4(u, b), at);
      c_read(at, c);
      zero(acc);
      mfmas(a, bop, acc);
      c_write(at, c, acc);
    };
    // rl: the listed rows of block 0 (fetched during the previous visit); returns those of the next visit
    auto visit = [&](const Visit& u, const Visit& following, const Visit& ahead, Regs& r, uint32_t rl) -> uint32_t {
      const uint32_t off0 = row_of(ahead, 0), off1 = row_of(ahead, 1), rl_next = rows4(following, 0);
      uint32_t at[4];
      f32x4_t c[4], acc[CW];
      c_at(u, 0, rl, at);
      c_read(at, c);
      zero(acc);
      // (opaque: keeps the transposes behind the loads of the two visits ahead -- the compiler otherwise carries the
      // transposed registers around the loop and waits for loads just issued)
#pragma unroll
      for (int i = 0; i < 8 * KS; i += 8)
        asm volatile("" : "+v"(r.b[i]), "+v"(r.b[i + 1]), "+v"(r.b[i + 2]), "+v"(r.b[i + 3]), "+v"(r.b[i + 4]), "+v"(r.b[i + 5]), "+v"(r.b[i + 6]), "+v"(r.b[i + 7]));
      // block 0, with the B rows of the visit after the next requested between the MFMAs, as soon as a step's registers
      // are free: a wave that requests them all in a row stands still while the load path takes them
      const uint32_t kp = k_of(ahead) * pitch_b;    // (K * ldb * 2 < 2^32: checked on the host)
      uint4 bop[KS][CW];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int x = 0; x < CW; ++x) {
          const uint32_t sel = (x & 1) ? 0x07060302u : 0x05040100u;
          uint32_t d[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) d[i] = r.b[8 * ks + i][x >> 1];
          bop[ks][x] = make_uint4(__builtin_amdgcn_perm(d[1], d[0], sel), __builtin_amdgcn_perm(d[3], d[2], sel),
                                  __builtin_amdgcn_perm(d[5], d[4], sel), __builtin_amdgcn_perm(d[7], d[6], sel));
        }
        PIT_SCHED_FENCE();
#pragma unroll
        for (int x = 0; x < CW; ++x) {
          acc[x] = mfma16<BF>(r.a[0][ks], bop[ks][x], acc[x]);
#pragma unroll
          for (int i = 0; i < 8 / CW; ++i) r.b[8 * ks + (8 / CW) * x + i] = load_b(kp, 8 * ks + (8 / CW) * x + i);
          PIT_SCHED_FENCE();
        }
      }
      load_a(k_of(ahead), off0, r.a[0]);
      asm volatile("" ::: "memory");                // (the loads are not to be moved behind what follows)
      PIT_SCHED_FENCE();
      c_write(at, c, acc);
      if (u.n > 16) {
        block(u, 1, r.a[1], bop);
        if constexpr (R > 32)
          if (u.n > 32) {
            uint4 ax[2][KS], ay[2][KS];
            const uint32_t k = k_of(u);
            load_a(k, row_of(u, 2), ax[0]); load_a(k, row_of(u, 3), ax[1]);
            for (int b = 2; 16 * b < u.n; b += 4) {   // (two pairs per trip: no register copies)
              load_a(k, row_of(u, b + 2), ay[0]); load_a(k, row_of(u, b + 3), ay[1]);
              block(u, b, ax[0], bop);
              if (u.n > 16 * (b + 1)) block(u, b + 1, ax[1], bop);
              load_a(k, row_of(u, b + 4), ax[0]); load_a(k, row_of(u, b + 5), ax[1]);
              if (u.n > 16 * (b + 2)) block(u, b + 2, ay[0], bop);
              if (u.n > 16 * (b + 3)) block(u, b + 3, ay[1], bop);
            }
            // (no load of this branch may stay under way: the common path would have to wait for it, and with it for its
            // own loads, wherever it reuses one of these registers)
            __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
          }
      }
      PIT_SCHED_FENCE();
      if (ahead.n > 16) load_a(k_of(ahead), off1, r.a[1]);
      asm volatile("" ::: "memory");
      PIT_SCHED_FENCE();
      return rl_next;
    };
    const int visits = __builtin_popcountll(live) * cps;
    Visit u0 = next(Visit{0, cps, 0}), u1 = next(u0);
    Regs ra, rb;
    // (in the order in which they are awaited, and not to be mixed)
    auto first = [&](const Visit& u, Regs& r) {
      const uint32_t off0 = row_of(u, 0), off1 = row_of(u, 1), kp = k_of(u) * pitch_b;
      PIT_SCHED_FENCE();
#pragma unroll
      for (int i = 0; i < 8 * KS; ++i) r.b[i] = load_b(kp, i);
      load_a(k_of(u), off0, r.a[0]);
      load_a(k_of(u), off1, r.a[1]);
      asm volatile("" ::: "memory");
      PIT_SCHED_FENCE();
    };
    first(u0, ra);
    first(u1, rb);
    uint32_t rl = rows4(u0, 0);
    // (two visits per trip, no exit between them and no copy of one behind the loop -- an odd last visit gets a partner
    // without rows: otherwise the compiler folds the bodies into one that copies registers with loads still under
    // way, i.e. waits for everything)
    for (int i = 0; i < visits; i += 2) {
      const Visit u2 = next(u1);
      rl = visit(u0, u1, u2, ra, rl);
      const Visit u3 = next(u2);
      if (i + 1 == visits) u1.n = 0;
      rl = visit(u1, u2, u3, rb, rl);
      u0 = u2; u1 = u3;
    }
  }
  __syncthreads();
  // SWrite: the groups' strips in a fixed order; consecutive lanes store the contiguous bytes of a row that a wave's columns make
  for (int i = tid; i < R * 32; i += 64 * NW) {
    const int row = i >> 5, w = (i & 31) / (WC / 4), c = (i % (WC / 4)) * 4;
    if (row >= rows) break;
    f32x4_t v = *reinterpret_cast<const f32x4_t*>(&s_c[w][row * WC + c]);
#pragma unroll
    for (int gi = 1; gi < SG; ++gi) v += *reinterpret_cast<const f32x4_t*>(&s_c[GW * gi + w][row * WC + c]);
    *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(g.C) + (int64_t)(r0 + row) * g.ldc + n0 + WC * w + c) = v;
  }
}

// Which strips, by how many 128-column strips of 128 or 64 rows the product has (t128, t64) on 512 slots: two workgroups fit
// a compute unit (one with KS = 1 and 128 rows).  A taller strip reads B less often, and a last round of them that is
// nearly empty costs more.  Time over the 32-row kernel's, R = 64 / R = 128, as the mean over 1.5, 10 and 40 % kept
// (the sparsity is known on the device only), in parentheses the worst of the three:
//   64 k per visit (slabs of 64 / 128; K 768 - 3840)
//     t128 = 432 - 504  .92 (1.0) / .74 (1.0) and .96 (1.1) / .79 (1.1)     R = 128 from 400 to 512
//     t128 = 520 - 696  .78 - .91 / .88 - 1.01 and .88 - .96 / .93 - 1.06   R = 64; its t64 is beyond 1024
//     t128 = 792, 1024  .85 / .77 (1.05); .75 / .52 and .90 / .83 (1.17); .83 / .56      R = 128 again (768: the same)
//     t64 = 400 - 512   .83 - .88 (1.0) and .90 - .94 (1.1)                R = 64
//     t64 = 520 - 600   .92 - .99 (1.1) and .98 - 1.05 (1.2)               the 32-row kernel
//     t64 = 640 - 792   .82 - .93 (1.0) and .92 - .99 (1.2)                R = 64 for slabs of 64
//   slabs of 32: R = 64 from t64 = 250 (.95; 264 - 510 .82 - .72; 1008 .69).  R = 128 is as good in the mean from t128 = 1024
//     on, .58 (1.0) and .58 at 1.5 and 10 % against .62 (.69) -- and better where such micro-tiles are used, 4096^3 at 5 and
//     10 % kept 146 and 157 us against 184 and 197, at 40 % 406 against 278; below that it is not (t128 = 520: 1.3 at 40 %).
//   other slabs (96): R = 64 at t64 = 400 - 512 (.90 - .96) and from 820 on (.88 - 1.0); in between 1.0 - 1.1.
template <bool BF, int KS, int R, int SG>
int launch_slab_tall(const GemmArgs& g, hipStream_t st) {
  const dim3 grid((unsigned)(ceil_div(g.M, R) * (g.N / ST_W)));
  hipLaunchKernelGGL((k_slab_strip_tall<BF, KS, R, SG>), grid, dim3(128 * SG), 0, st, g);
  PIT_LAUNCH_CHECK();
  return PIT_OK;
}
template <bool BF>
int launch_slab_strip_bf(const GemmArgs& g, hipStream_t st) {
  const int64_t strips = ceil_div(g.M, StripShape<8>::R);
  if (strips > 65535) return PIT_ESHAPE;
  const int64_t tn = g.N / ST_W, slots = 2 * compute_units();
  const int64_t t128 = ceil_div(g.M, 128) * tn, t64 = ceil_div(g.M, 64) * tn;
  const bool t64_fill = 32 * t64 >= 25 * slots && t64 <= slots;      // one round, 400 - 512 strips
  if (g.slab % 64 == 0) {                            // 64 k per visit
    if (32 * t128 >= 25 * slots && (t128 <= slots || 2 * t128 > 3 * slots)) return launch_slab_tall<BF, 2, 128, 1>(g, st);
    if (t64_fill || t64 > 2 * slots || (g.slab == 64 && 4 * t64 >= 5 * slots)) return launch_slab_tall<BF, 2, 64, 2>(g, st);
  } else if (g.slab == 32) {
    if (t128 >= 2 * slots) return launch_slab_tall<BF, 1, 128, 2>(g, st);
    if (2 * t64 >= slots) return launch_slab_tall<BF, 1, 64, 2>(g, st);
  } else if (t64_fill || 5 * t64 > 8 * slots) {
    return launch_slab_tall<BF, 1, 64, 2>(g, st);
  }
  // 32 x 128 strips.  (64 x 64 strips, CW = 4, halve the traffic of B and double that of A: measured 10-15 %
  // faster at 90-95 % sparsity of a 4096^3 product, 10-20 % slower at 50 % and at 99 %.)
  constexpr int CW = 8;
  hipLaunchKernelGGL((k_slab_strip<BF, CW>), dim3((unsigned)(g.N / StripShape<CW>::W), (unsigned)strips), dim3(256), 0, st, g);
  PIT_LAUNCH_CHECK();
  return PIT_OK;
}

}  // namespace

int launch_slab_strip(bool bf, const GemmArgs& g, hipStream_t st) {
  const RingMTile ring = ring_slab_tile(g);
  if (ring != RINGM_NONE) return launch_slab_ring(bf, g, ring, st);
  return bf ? launch_slab_strip_bf<true>(g, st) : launch_slab_strip_bf<false>(g, st);
}

}  // namespace pit
