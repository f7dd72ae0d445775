// Which rows of a tile the k-slabs of an index list, as bits in LDS (GATHER_M with micro-tiles along k; gfx950).
#pragma once
#include "pit_gemm_dev.hpp"

namespace pit {
namespace {

constexpr int SLABS_MAX = 512;                       // most slabs of a product whose masks are held in LDS

// s_mask[slab * TR / 32 + w] = bit r: row r0 + 32 w + r is listed for the slab.  All NW waves of the workgroup take part, wave w with
// slabs w, w + NW, .., eight of them in flight together: their list bounds, then rounds of a 64-ary search for the first entry
// >= r0 (none for lists of up to 64 entries, one up to 4096), then the entries from there on -- at most 64 before the tile's and TR
// of the tile.  Ends with a barrier.
template <int TR, int NW>
__device__ __forceinline__ void build_slab_masks(const GemmArgs& g, int r0, uint32_t* s_mask, int tid) {
  constexpr int MW = TR / 32, B = 8, WIN = (64 + TR + 63) / 64;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = tid; i < g.nseg * MW; i += 64 * NW) s_mask[i] = 0u;
  __syncthreads();
  const bool some = g.seg_ptr[g.nseg] > 0;           // (there is an entry 0)
  for (int j0 = 0; some && wv + NW * j0 < g.nseg; j0 += B) {
    int lo[B], hi[B], end[B];
    const int mine = wv + NW * (j0 + (lane & (B - 1)));
    const int pv = g.seg_ptr[(mine < g.nseg ? mine : 0) + ((lane >> 3) & 1)];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const bool valid = wv + NW * (j0 + j) < g.nseg;
      lo[j] = valid ? __builtin_amdgcn_readlane(pv, j) : 0;
      end[j] = valid ? __builtin_amdgcn_readlane(pv, B + j) : 0;
      hi[j] = end[j];
    }
    // invariant: lo <= p* <= hi for the position p* of the first entry >= r0
    for (;;) {
      bool any_wide = false;
#pragma unroll
      for (int j = 0; j < B; ++j) any_wide |= hi[j] - lo[j] > 64;
      if (!any_wide) break;
      int smp[B], step[B];
#pragma unroll
      for (int j = 0; j < B; ++j) {
        step[j] = (hi[j] - lo[j] + 63) / 64;
        const int pos = lo[j] + lane * step[j];
        const int v = g.idx[max(min(pos, hi[j] - 1), 0)];
        smp[j] = pos < hi[j] ? v : 0x7fffffff;
      }
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const int c = __popcll(__ballot(smp[j] < r0));
        const int hi_new = (c < 64 && lo[j] + c * step[j] < hi[j]) ? lo[j] + c * step[j] : hi[j];
        hi[j] = c == 0 ? lo[j] : hi_new;
        lo[j] = c == 0 ? lo[j] : lo[j] + (c - 1) * step[j] + 1;
      }
    }
    int e[B][WIN];
#pragma unroll
    for (int j = 0; j < B; ++j)
#pragma unroll
      for (int w = 0; w < WIN; ++w) {
        const int p = lo[j] + 64 * w + lane, v = g.idx[max(min(p, end[j] - 1), 0)];
        e[j][w] = p < end[j] ? v - r0 : -1;
      }
#pragma unroll
    for (int j = 0; j < B; ++j)
#pragma unroll
      for (int w = 0; w < WIN; ++w)
        if (e[j][w] >= 0 && e[j][w] < TR) atomicOr(&s_mask[(wv + NW * (j0 + j)) * MW + (e[j][w] >> 5)], 1u << (e[j][w] & 31));
  }
  __syncthreads();
}

}  // namespace
}  // namespace pit
