// Stores and the clearing of unlisted rows, shared by the GATHER_M kernels (gfx950).
#pragma once
#include "pit_gemm_dev.hpp"
#include <climits>

namespace pit {
namespace {

// f(store), where store(value, address) is an ordinary or a streaming store of 16 bytes of C (the rule is at launch_cfg).
// (The marks keep the compiler from merging the two paths, which would make all stores ordinary ones.)
template <bool CHOICE = true, typename F>
__device__ __forceinline__ void with_stores_of(const GemmArgs& g, F&& f) {
  if (CHOICE && g.stream_c) {
    asm volatile("; streaming stores");
    f([](const u32x4_t& v, void* at) { __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(at)); });
    asm volatile("; end of streaming stores");
  } else {
    f([](const u32x4_t& v, void* at) { *reinterpret_cast<u32x4_t*>(at) = v; });
  }
}

// Zero the rows of C that an ascending list does not name, for the rows [r_begin, r_end): the share of one
// workgroup without a tile (all of these shares together cover [0, M)).  One 64-ary search finds the list
// position of the first row (three or four dependent loads for a list of thousands); from there the list is
// read 64 entries at a time: the entries below the end of a chunk of 64 rows mark its covered rows in a 64-bit
// mask, and as many entries as the mask has bits are consumed.  Wave w of NW clears rows w, w + NW, ... of the chunk,
// 16 bytes per lane.
template <int ESIZE, int NW>
__device__ __forceinline__ void zero_unlisted_rows(const GemmArgs& g, int r_begin, int r_end, int wv, int lane) {
  const int n = g.seg_ptr[1] - g.seg_ptr[0];
  const int32_t* list = g.idx + g.seg_ptr[0];
  int lo = 0, hi = n;                      // smallest j with list[j] >= r_begin (n if none)
  while (lo < hi) {
    const int step = (hi - lo + 63) >> 6;
    const int p = lo + lane * step;
    const int v = p < hi ? list[p] : INT_MAX;
    const int k = __builtin_popcountll(__ballot(v < r_begin));   // the probes ascend: the first k are below
    if (k == 0) { hi = lo; break; }
    const int below = lo + (k - 1) * step;
    hi = min(hi, below + step);
    lo = below + 1;
  }
  const int64_t nbytes = (int64_t)g.N * ESIZE;
  for (int r0 = r_begin; r0 < r_end; r0 += 64) {
    const int v = lo + lane < n ? list[lo + lane] : INT_MAX;     // strictly ascending: entry j is >= r0 + j
    uint64_t m = (v < r0 + 64) ? (1ull << (v - r0)) : 0ull;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) m |= __shfl_xor(m, d);
    lo += __builtin_popcountll(m);
    for (int r = r0 + wv; r < min(r0 + 64, r_end); r += NW) {
      if ((m >> (r - r0)) & 1) continue;
      char* p = reinterpret_cast<char*>(g.C) + (int64_t)r * g.ldc * ESIZE;
      with_stores_of(g, [&](auto store) {
        for (int64_t b = (int64_t)lane * 16; b < nbytes; b += 64 * 16) store(u32x4_t{0u, 0u, 0u, 0u}, p + b);
      });
    }
  }
}

}  // namespace
}  // namespace pit
