// Types, tile constants and host-side launchers shared by the SRead -> dense MFMA tile -> SWrite
// kernels for gfx950 (paper Section 3.1, sparse kernel template).  The kernels themselves:
//   pit_gemm.hip    GATHER_K (k is the PIT-axis, operands register-direct)
//   pit_gemm_ring.hip  GATHER_K for products with few tiles (operands through rings in LDS)
//   pit_slab.hip    GATHER_M with several k-slabs per row (strips of C in LDS)
//   pit_gemm_m.hip  GATHER_M with whole-row micro-tiles (operands staged through LDS by direct loads)
//   pit_gemm_m_ring.hip  the same with few tiles or few rows per segment
// Their device-side helpers are in pit_gemm_dev.hpp.
#pragma once
#include "pit_common.hpp"

namespace pit {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef short v4i16_t __attribute__((__vector_size__(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
#define PIT_LDS __attribute__((address_space(3)))

constexpr int TM = 128, TN = 128;   // GATHER_K: rows (at most) and columns of a tile

enum { EPI_STORE = 0, EPI_GELU = 2 };

struct GemmArgs {
  const void* A; int64_t lda;
  const void* B; int64_t ldb; int64_t b_seg_stride;   // elements between the B matrices of two segments (MoE), else 0
  void* C; int64_t ldc;
  const int32_t* seg_ptr; const int32_t* idx;
  const float* gate;                                   // per C row (EPI_STORE with scatter), or nullptr
  int nseg, M, N, K;
  int slab;          // GATHER_M: k extent of one segment's slab (K when nseg == 1 or per-segment weights)
                     // GATHER_K: micro-tile height of the index (128, 64 or 32); a tile has as many rows or fewer
  int a_gather;      // GATHER_M: 1 = A rows come from idx, 0 = A rows are seg_ptr[s] + r (compact)
  int c_scatter;     // GATHER_M: 1 = C rows go to idx, 0 = C rows are seg_ptr[s] + r (compact)
  int slab_per_seg;  // GATHER_M: 1 = segment s covers k in [s*slab, (s+1)*slab), 0 = every segment covers [0, K)
  int k_stagger;     // GATHER_M, set by the launcher: 1 = tiles of different segments / column tiles start their walk
                     // over k at different steps (per-segment B)
  int xcd_cols;      // GATHER_M, set by the launcher: the 8 XCDs form 8 / xcd_cols row groups x xcd_cols column groups
  int zero_rest;     // GATHER_M, one segment: 1 = the rows of C that the list does not name are set to zero by the
                     // workgroups of the grid that have no tile
  int stream_c;      // GATHER_M, set by the launcher: 1 = C is written by streaming stores
  // Mixture of experts without an index (both products: gather_m_routes): expert ids of the M <= 64 tokens; rows of A and C are
  // tokens.  route_rest: count the tokens without an expert in *status (if given) and clear their rows of C.
  const int32_t* route; int32_t* status; int route_rest;
};

// Host-side launchers shared by pit_sread_gemm and pit_moe_dispatch_gemm.
// GATHER_M with operands staged through LDS by direct loads (pit_gemm_m.hip).  total_rows = upper bound of the
// number of listed rows over all segments (the grid is sized for the worst case; the counts stay on the device).
int launch_gather_m(bool bf, int epi, int c_is_in_type, const GemmArgs& g, int64_t total_rows, hipStream_t st);
// Whether a product with a B per segment takes a kernel that can do without the index (then g.route may be set).
bool gather_m_routes(const GemmArgs& g);
int launch_zero_rows(void* C, int64_t ld_bytes, int M, int64_t row_bytes, hipStream_t st);
// GATHER_K for few tiles (pit_gemm_ring.hip): the tile it has for a product, or none
enum RingTile { RING_NONE, RING_32x32, RING_32x64, RING_64x64, RING_64x64_SHORT };
RingTile ring_tile(const GemmArgs& g);
int launch_gather_k_ring(bool bf, int c_is_in_type, const GemmArgs& g, RingTile tile, hipStream_t st);
// GATHER_M for few tiles or few rows per segment (pit_gemm_m_ring.hip): the tile it has for a product (rows x columns; _8: eight waves
// instead of four; 16 x 32 and 32 x 32 have eight), or none
enum RingMTile { RINGM_NONE, RINGM_16x32, RINGM_16x64, RINGM_16x64_8, RINGM_32x32, RINGM_32x64, RINGM_32x64_8, RINGM_64x64, RINGM_64x64_8 };
RingMTile ring_m_tile(int epi, const GemmArgs& g, int64_t total_rows);
int launch_gather_m_ring(bool bf, int epi, int c_is_in_type, const GemmArgs& g, int64_t total_rows, RingMTile tile, hipStream_t st);
// the same for several k-slabs per row (micro-tiles along k), fp32 results
RingMTile ring_slab_tile(const GemmArgs& g);
int launch_slab_ring(bool bf, const GemmArgs& g, RingMTile tile, hipStream_t st);
// GATHER_M with several k-slabs per row (pit_slab.hip); fp32 results
int launch_slab_strip(bool bf, const GemmArgs& g, hipStream_t st);

}  // namespace pit
