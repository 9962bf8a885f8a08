// Which entries of the row list and which parts of A the forward of small and mid-sized batches (k_encode_mid,
// k_encode_square) and the 256-row contraction (k_gemm_nt_bf16) ask memory for.  Plain C++ as well as device code, so that
// the limits can be walked on the CPU.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define GRAM_HD __host__ __device__ __forceinline__
#else
#define GRAM_HD inline
#endif

namespace gram {

constexpr uint32_t kPastEnd = 0xFFFFFFF0u;      // an offset no descriptor covers: reads zeros

// Entry of the list for row j of the product (U: the items it holds, at least 1).
GRAM_HD int mid_list_entry(int j, int U) { return j < U ? j : U - 1; }

// Byte offset of the lane's first chunk (element xk) of row `row` of A; the rows of the padding item and those
// behind the U items are not read.
GRAM_HD uint32_t mid_row_offset(int j, int U, bool pad, uint32_t row, uint32_t d_in, uint32_t xk)
{
    return pad || j >= U ? kPastEnd : (row * d_in + xk) * 2u;
}

// The chunk of 8 elements at k0 + xk of that row, k0 the first element of the slab.
GRAM_HD uint32_t mid_slab_offset(uint32_t row_offset, int k0, int xk, int d_in)
{
    return k0 + xk < d_in && row_offset != kPastEnd ? row_offset + (uint32_t)k0 * 2u : kPastEnd;
}

// ---- the 256-row contraction: slabs of 64 along K (a multiple of 32) -----------------------------
//
// An odd multiple leaves half a slab: it is the first, 64 elements of which only the lower 32 are multiplied, and the second
// starts at 32.  (As the last one, its upper half would lie behind the row, and behind the matrix for the last row.)  For
// K = 32 both halves of the one slab hold the row.
constexpr int kBigSlab = 64;

// First element of slab 0 .. last (loads for slabs past the last fetch nothing, or the last one again).
GRAM_HD int big_slab_start(int slab, int k) { return slab ? slab * kBigSlab - (k & 32) : 0; }

// The part of a slab (of `size` elements of K each) that a load for part `part` fetches, counted from the slab's start.
GRAM_HD int big_slab_part(int part, int size, int k) { return k < kBigSlab ? part & (32 / size - 1) : part; }

// The slab whose upper half is not multiplied, -1 if there is none.
GRAM_HD int big_half_slab(int k) { return k & 32 ? 0 : -1; }

}  // namespace gram
