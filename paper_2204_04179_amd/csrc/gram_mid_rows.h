// Which entries of the row list and which rows of A the forward of small and mid-sized batches
// (k_encode_mid) asks memory for.  Plain C++ as well as device code, so that the limits can be walked on the CPU.
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

}  // namespace gram
