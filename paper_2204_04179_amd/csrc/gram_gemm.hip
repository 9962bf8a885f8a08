// The two dense contractions of the GRAM step, with the dense linear stand-in
// for the content encoder:
//   forward  (Algorithm 1 step 1, Eq. 4):  E[j,:]  = X[uniq[j],:] . W
//   wgrad    (Algorithm 1 step 4, Eq. 7/9): dW[i,c] = sum_s X[item_s, i] * G[s, c]
// bf16 inputs run on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).
//   forward: k_gemm_nt_bf16, C = A . B^T with both operands stored with the
//            contraction index contiguous: A = rows of X gathered through the
//            unique-ID list inside the tile loads (the unique items' features are
//            never copied), B = W^T.  For large batches its epilogue is the gather
//            as well: every representation is stored straight to the positions of
//            its item.  Small and mid-sized batches take k_encode_mid or, with long K and a 128 x 128 tile for
//            every CU, k_encode_square; what those do not take k_encode_bf16.
//   wgrad:   k_wgrad_tn_bf16 contracts over the rows of the gradient buffer, which
//            is the slow dimension of both operands in memory, with transposing
//            LDS reads; split-K over blocks, float32 partials added in split order.
//            Rows that are bf16 already take k_wgrad_rows_bf16, short windows k_wgrad_short.
//   Operands are addressed through buffer descriptors (32-bit offsets, out-of-range
//   reads return zero); matrices beyond the 4 GiB a descriptor can address take the
//   WIDE variants of both kernels, which form 64-bit addresses per lane.
// The float32 variants are plain FMA code for small problems.
#include <algorithm>

#include "gram_internal.h"
#include "gram_mid_rows.h"

namespace gram {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4_ __attribute__((ext_vector_type(4)));
constexpr uint32_t kRawBuffer = 0x00027000;     // descriptor flags: 32-bit elements, no swizzle

// What a contraction kernel does with its output elements before storing them (template parameter EPI
// of the kernels below).  `aux` has the row pitch of C.
//   kEpiPlain      C = v                                   (float32)
//   kEpiReluBf16   C = bf16(max(v, 0))                     (C is a bf16 matrix)
//   kEpiMinus      C = v - aux                             (aux float32: stored targets)
//   kEpiMinusBf16  C = bf16(v - aux)                       (what the contractions that read it would round)
//   kEpiGateBf16   C = bf16(v) where aux > 0, else 0       (aux bf16: kept activations)
// A row flagged `zero` (the padding item) is stored as zeros in every mode.  With the two subtracting modes a
// kernel can also leave, per block, the sum of the squares of what it stored (before rounding to bf16), in
// double and in a fixed order: the pseudo-loss without another pass over the matrix.
__host__ __device__ constexpr bool epi_subtracts(int epi) { return epi == kEpiMinus || epi == kEpiMinusBf16; }
__host__ __device__ constexpr bool epi_stores_bf16(int epi) { return epi == kEpiReluBf16 || epi == kEpiMinusBf16 || epi == kEpiGateBf16; }

// The aux values of 4 consecutive elements (at: a multiple of 4) are fetched ahead of the stores: the
// targets, or 1 / 0 for an open / closed gate.
template <int EPI>
__device__ __forceinline__ f32x4_ epi_load4(const void* __restrict__ aux, int64_t at)
{
    if (epi_subtracts(EPI)) return *reinterpret_cast<const f32x4_*>(static_cast<const float*>(aux) + at);
    f32x4_ r = {0.f, 0.f, 0.f, 0.f};
    if (EPI == kEpiGateBf16) {
        typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
        const u16x4 a = *reinterpret_cast<const u16x4*>(static_cast<const uint16_t*>(aux) + at);
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = ((a[k] & 0x8000u) || !(a[k] & 0x7fffu)) ? 0.f : 1.f;   // positive bf16 only
    }
    return r;
}

// The value stored (float32, before a rounding to bf16).
template <int EPI>
__device__ __forceinline__ float epi_value(float v, float a, bool zero)
{
    if (EPI == kEpiReluBf16) return !zero && v > 0.f ? v : 0.f;
    if (epi_subtracts(EPI)) return zero ? 0.f : v - a;
    if (EPI == kEpiGateBf16) return zero || a == 0.f ? 0.f : v;
    return zero ? 0.f : v;
}

template <int EPI>
__device__ __forceinline__ void epi_store4(float* __restrict__ C, int64_t at, f32x4_ v)
{
    if (epi_stores_bf16(EPI)) {
        typedef uint32_t u32x2_ __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u32x2_*>(reinterpret_cast<uint16_t*>(C) + at) = u32x2_{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else {
        *reinterpret_cast<f32x4_*>(C + at) = v;
    }
}

// Sum of one double per thread over a block of whole waves, in a fixed order; thread 0 writes it.
__device__ __forceinline__ void block_sum_double(double v, int threads, double* sm /*[threads / 64]*/, double* out)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < threads / 64; ++w) s += sm[w];
        *out = s;
    }
}

// ---- small forward kernel: latency first ------------------------------------------
//
// Batches whose unique items give the 256x256 kernel fewer tiles than there are CUs (and any
// d_in that is not a multiple of 32), where k_encode_mid below does not apply: the gate epilogue, a width
// that is not a multiple of 8, a matrix beyond 4 GiB.  Such a launch is bound by the latency of its loads,
// not by arithmetic: a 64x64 tile per block (one 32x32 MFMA tile per wave) puts a block on
// nearly every CU, K advances in slabs of 64, and the loads of three slabs are in flight in
// registers ahead of the one being multiplied.  Two LDS buffers, one barrier per slab.

constexpr int BM = 64, BN = 64, BK = 64, kSmallDepth = 3;
constexpr int LDS_STRIDE = BK + 8;   // bf16 elements per LDS row (144 bytes: 16-byte aligned, staggers banks)

// W[d_in,d] -> Wt[d,d_in] (bf16)
__global__ __launch_bounds__(kBlock) void k_transpose_u16(const uint16_t* __restrict__ W, int rows,
                                                          int cols, uint16_t* __restrict__ Wt)
{
    __shared__ uint16_t tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    for (int y = ty; y < 32; y += 8)
        if (r0 + y < rows && c0 + tx < cols) tile[y][tx] = W[(int64_t)(r0 + y) * cols + c0 + tx];
    __syncthreads();
    for (int y = ty; y < 32; y += 8)
        if (c0 + y < cols && r0 + tx < rows) Wt[(int64_t)(c0 + y) * rows + r0 + tx] = tile[tx][y];
}

__device__ __forceinline__ uint4 and4(uint4 v, uint32_t m) { return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m); }

// BDIRECT: the second operand is W [d_in, d] as the caller holds it (d a multiple of 8), not its
// transpose: a slab of W is parked as 64 rows of k with 64 values of n each, and the MFMA fragments
// (8 consecutive k for one n) come from the transposing LDS read of gfx950 (ds_read_b64_tr_b16;
// see k_wgrad_tn_bf16 for its lane layout).  Saves the separate transpose launch, which matters
// where this kernel is used: batches that are bound by launch latency.
typedef short sv4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) sv4i16 lds_sv4i16;

template <int EPI, bool BDIRECT = false>
__global__ __launch_bounds__(kBlock) void k_encode_bf16(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ Wt, const int* __restrict__ uniq,
    const int* __restrict__ u_dev, int d_in, int d, const int* __restrict__ zero_ids, int pad_id,
    float* __restrict__ E, const void* __restrict__ aux, double* __restrict__ loss_part)
{
    __shared__ __attribute__((aligned(16))) uint16_t sA[2][BM * LDS_STRIDE];
    __shared__ __attribute__((aligned(16))) uint16_t sB[2][BN * LDS_STRIDE];
    const int U = *u_dev;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    if (epi_subtracts(EPI) && loss_part) loss_part += blockIdx.y * gridDim.x + blockIdx.x;
    if (m0 >= U) {
        if (epi_subtracts(EPI) && loss_part && threadIdx.x == 0) *loss_part = 0.0;
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // each thread moves two 16-byte chunks of A and of B per slab: chunk cid = tid + 256 h is
    // bytes [16 (cid % 8), +16) of row cid / 8.  Rows past the end are clamped to a valid row
    // (their products are never stored); chunks past d_in are loaded from the row's start and
    // replaced by zeros.
    const uint16_t* pa0;
    const uint16_t* pa1;
    const uint16_t* pb0;
    const uint16_t* pb1;
    const int kc0 = (tid & 7) * 8, kc1 = kc0;               // 256 is a multiple of 8: same chunk column
    const int lrow0 = tid >> 3, lrow1 = (tid + kBlock) >> 3;
    {
        const int j0 = m0 + lrow0 < U ? m0 + lrow0 : U - 1, j1 = m0 + lrow1 < U ? m0 + lrow1 : U - 1;
        pa0 = X + (int64_t)uniq[j0] * d_in;
        pa1 = X + (int64_t)uniq[j1] * d_in;
        if (BDIRECT) {
            // chunk of 8 values of n at column n0 + kc0 of row k = slab start + lrow; a column past
            // the matrix is fetched from column 0 (its products are never stored)
            pb0 = pb1 = Wt + (n0 + kc0 < d ? n0 + kc0 : 0);
        } else {
            const int c0 = n0 + lrow0 < d ? n0 + lrow0 : d - 1, c1 = n0 + lrow1 < d ? n0 + lrow1 : d - 1;
            pb0 = Wt + (int64_t)c0 * d_in;
            pb1 = Wt + (int64_t)c1 * d_in;
        }
    }
    uint4 a00, a01, b00, b01, a10, a11, b10, b11, a20, a21, b20, b21;     // three register sets
#define GRAM_LOAD_SLAB(S, K0)                                                                       \
    {                                                                                               \
        const int k_ = (K0) + kc0;                                                                  \
        const int ks_ = k_ < d_in ? k_ : 0;                                                         \
        a##S##0 = *reinterpret_cast<const uint4*>(pa0 + ks_);                                       \
        a##S##1 = *reinterpret_cast<const uint4*>(pa1 + ks_);                                       \
        if (BDIRECT) {                                                                              \
            const int r0_ = (K0) + lrow0 < d_in ? (K0) + lrow0 : 0;                                 \
            const int r1_ = (K0) + lrow1 < d_in ? (K0) + lrow1 : 0;                                 \
            b##S##0 = *reinterpret_cast<const uint4*>(pb0 + (int64_t)r0_ * d);                      \
            b##S##1 = *reinterpret_cast<const uint4*>(pb1 + (int64_t)r1_ * d);                      \
        } else {                                                                                    \
            b##S##0 = *reinterpret_cast<const uint4*>(pb0 + ks_);                                   \
            b##S##1 = *reinterpret_cast<const uint4*>(pb1 + ks_);                                   \
        }                                                                                           \
    }
#define GRAM_PARK_SLAB(S, K0, BUF)                                                                  \
    {                                                                                               \
        const uint32_t keep_ = (K0) + kc0 < d_in ? 0xFFFFFFFFu : 0u;                                \
        *reinterpret_cast<uint4*>(&sA[BUF][lrow0 * LDS_STRIDE + kc0]) = and4(a##S##0, keep_);       \
        *reinterpret_cast<uint4*>(&sA[BUF][lrow1 * LDS_STRIDE + kc1]) = and4(a##S##1, keep_);       \
        const uint32_t kb0_ = BDIRECT ? ((K0) + lrow0 < d_in ? 0xFFFFFFFFu : 0u) : keep_;           \
        const uint32_t kb1_ = BDIRECT ? ((K0) + lrow1 < d_in ? 0xFFFFFFFFu : 0u) : keep_;           \
        *reinterpret_cast<uint4*>(&sB[BUF][lrow0 * LDS_STRIDE + kc0]) = and4(b##S##0, kb0_);        \
        *reinterpret_cast<uint4*>(&sB[BUF][lrow1 * LDS_STRIDE + kc1]) = and4(b##S##1, kb1_);        \
    }

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    const int nslab = (d_in + BK - 1) / BK;
    const int arow = (wm * 32 + (lane & 31)) * LDS_STRIDE + (lane >> 5) * 8;
    // BDIRECT: sB rows are k; group g = lane / 16 of a transposing read covers k rows
    // (g / 2) * 8 + 4 h + j / 4 and columns wn * 32 + (g % 2) * 16 + 4 (j % 4) .. + 3, j = lane % 16
    const int brow = BDIRECT ? (((lane >> 5) * 8 + ((lane & 15) >> 2)) * LDS_STRIDE + wn * 32 +
                                ((lane >> 4) & 1) * 16 + (lane & 3) * 4)
                             : ((wn * 32 + (lane & 31)) * LDS_STRIDE + (lane >> 5) * 8);
    // slab sl lives in register set sl % 3; in iteration sl the set of slab sl + 1 is parked in
    // the other LDS buffer and refilled with slab sl + 4.  Nothing is conditional (slabs past the
    // end park zeros), so the count of loads in flight is known at every wait.
#define GRAM_SMALL_ITER(SNEXT, SL)                                                                  \
    {                                                                                               \
        GRAM_PARK_SLAB(SNEXT, ((SL) + 1) * BK, ((SL) + 1) & 1)                                      \
        GRAM_LOAD_SLAB(SNEXT, ((SL) + 1 + kSmallDepth) * BK)                                        \
        const uint16_t* a_ = &sA[(SL) & 1][arow];                                                   \
        const uint16_t* b_ = &sB[(SL) & 1][brow];                                                   \
        _Pragma("unroll") for (int ks = 0; ks < BK / 16; ++ks) {                                    \
            const bf16x8 fa = *reinterpret_cast<const bf16x8*>(a_ + ks * 16);                       \
            bf16x8 fb;                                                                              \
            if (BDIRECT) {                                                                          \
                const uint16_t* t_ = b_ + ks * 16 * LDS_STRIDE;                                     \
                const sv4i16 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)t_);        \
                const sv4i16 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)(t_ + 4 * LDS_STRIDE)); \
                fb = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7)); \
            } else {                                                                                \
                fb = *reinterpret_cast<const bf16x8*>(b_ + ks * 16);                                \
            }                                                                                       \
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc, 0, 0, 0);                    \
        }                                                                                           \
        __syncthreads();                                                                            \
    }
    GRAM_LOAD_SLAB(0, 0)
    GRAM_LOAD_SLAB(1, BK)
    GRAM_LOAD_SLAB(2, 2 * BK)
    GRAM_PARK_SLAB(0, 0, 0)
    GRAM_LOAD_SLAB(0, 3 * BK)
    __syncthreads();
    for (int s0 = 0; s0 < nslab; s0 += kSmallDepth) {
        GRAM_SMALL_ITER(1, s0)
        GRAM_SMALL_ITER(2, s0 + 1)
        GRAM_SMALL_ITER(0, s0 + 2)
    }
#undef GRAM_LOAD_SLAB
#undef GRAM_PARK_SLAB
#undef GRAM_SMALL_ITER

    // accumulator element r of a lane sits at (row, col) = ((r / 4) * 8 + (lane / 32) * 4 + r % 4, lane % 32).
    // The tile goes through LDS (the slabs are dead), so that a thread stores 4 consecutive columns.
    // Everything the stores need is fetched first (the aux values and the IDs that tell the padding
    // row): fetched in the store loop, each store would wait for its own load and, with it, for the
    // stores before it.
    constexpr int LD = BN + 4;
    __shared__ __attribute__((aligned(16))) float s_tile[BM * LD];
    __shared__ double s_loss[kBlock / 64];
#pragma unroll
    for (int r = 0; r < 16; ++r)
        s_tile[(wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * LD + wn * 32 + (lane & 31)] = acc[r];
    f32x4_ av[BM * BN / 4 / kBlock];
    int idr[BM * BN / 4 / kBlock];
    const int erow = tid / (BN / 4), ecol = tid % (BN / 4) * 4;
    const bool col_ok = n0 + ecol < d;
#pragma unroll
    for (int h = 0; h < BM * BN / 4 / kBlock; ++h) {
        const int j = m0 + erow + h * (kBlock * 4 / BN);
        av[h] = (j < U && col_ok) ? epi_load4<EPI>(aux, (int64_t)j * d + n0 + ecol) : f32x4_{0.f, 0.f, 0.f, 0.f};
        idr[h] = j < U ? zero_ids[j] : 0;
    }
    __syncthreads();
    double sq = 0.0;
#pragma unroll
    for (int h = 0; h < BM * BN / 4 / kBlock; ++h) {
        const int row = erow + h * (kBlock * 4 / BN), j = m0 + row;
        f32x4_ v = *reinterpret_cast<const f32x4_*>(&s_tile[row * LD + ecol]);
        if (j < U && col_ok) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = epi_value<EPI>(v[k], av[h][k], idr[h] == pad_id);
                if (epi_subtracts(EPI)) sq += (double)v[k] * v[k];
            }
            epi_store4<EPI>(E, (int64_t)j * d + n0 + ecol, v);
        }
    }
    if (epi_subtracts(EPI) && loss_part) block_sum_double(sq, kBlock, s_loss, loss_part);
}

// ---- the forward of small and mid-sized batches ------------------------------------------
//
// What such a launch spends its time on is not arithmetic but the wait for its operands: two dependent
// round trips (unique list, rows of X) before the first slab, and with the four waves per block of the kernel
// above a third of K in flight at 19 B/clk per CU.  Here the waves of a block cut K between KG groups,
// which walk every KG-th slab of 64 side by side and add their tiles through LDS at the end: twice as
// many waves and bytes in flight per tile.  W is read as the caller holds it; loads go through descriptors
// (rows of the padding item and everything past an edge read zeros), so the loads in flight are known at
// every wait.  Neither the list nor A is read behind the U items: both may be the caller's and hold no more
// than those (reading the list ahead of U saves nothing: the compiler waits for U before it either way).
// A wave has WR tiles of 32 x 32 below each other.  Four groups (all of K in flight) were slower: the tile
// then takes longer to add up than its slabs to arrive.
// LDS: rows of X are 128 bytes (chunk c of row r at c ^ ((r >> 1) & 7)); rows of W as in k_wgrad_short.
constexpr int SK = 64;
template <int TM_, int TN, int KG, int WR>
struct Mid {
    static constexpr int kGroupThreads = (TM_ / (32 * WR)) * (TN / 32) * 64, kThreads = KG * kGroupThreads;
    static constexpr size_t kStageB = TM_ * SK * 2 + SK * TN * 2;               // bytes per group
    static constexpr size_t kTilesB = (size_t)KG * TM_ * (TN + 8) * 4;
    static constexpr size_t kLds = kTilesB > KG * kStageB ? kTilesB : KG * kStageB;
};

template <int SM, int TN, int KG, int WR, int DEPTH, int EPI>
__device__ __forceinline__ void encode_mid_tile(
    const uint16_t* __restrict__ X, uint32_t x_bytes, const uint16_t* __restrict__ W, uint32_t w_bytes,
    const int* __restrict__ uniq, int U, int d_in, int d, const int* __restrict__ zero_ids, int pad_id,
    float* __restrict__ E, const void* __restrict__ aux, double* __restrict__ loss_part, int m0, int n0,
    unsigned char* smem, int* s_ids, double* s_loss)
{
    constexpr int GT = Mid<SM, TN, KG, WR>::kGroupThreads, STHREADS = KG * GT;
    constexpr size_t kStageB = Mid<SM, TN, KG, WR>::kStageB;                       // threads per group
    constexpr int XT = SM * 8 / GT, WT = SK * (TN / 8) / GT; // 16-byte chunks per thread and slab
    constexpr int WROW = TN * 2;                            // bytes per row of W in LDS
    static_assert(WROW == 128, "the swizzle of its rows");
    constexpr int WM = SM / (32 * WR);                      // waves along the rows
    const int tid = threadIdx.x, grp = __builtin_amdgcn_readfirstlane(tid / GT), gt = tid % GT;
    const int lane = tid & 63, wave = gt >> 6, wm = wave % WM, wn = wave / WM;

    const int xrow = gt >> 3, xpos = gt & 7;                // + (GT / 8) t
    int id[XT], zid[XT];
#pragma unroll
    for (int t = 0; t < XT; ++t) {
        const int jj = mid_list_entry(m0 + xrow + t * (GT / 8), U);
        id[t] = uniq[jj];
        zid[t] = zero_ids[jj];
    }
    const __amdgpu_buffer_rsrc_t rsX = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(X), 0, x_bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(W), 0, w_bytes, kRawBuffer);
    if (grp == 0 && xpos == 0)
#pragma unroll
        for (int t = 0; t < XT; ++t) s_ids[xrow + t * (GT / 8)] = zid[t];
    // rows xrow + (GT / 8) t swizzle alike: GT / 8 is a multiple of 16
    static_assert(GT / 8 % 16 == 0, "row swizzle");
    const int xk = (xpos ^ ((xrow >> 1) & 7)) * 8;
    uint32_t ox[XT];
#pragma unroll
    for (int t = 0; t < XT; ++t)
        ox[t] = mid_row_offset(m0 + xrow + t * (GT / 8), U, zid[t] == pad_id, (uint32_t)id[t], (uint32_t)d_in, (uint32_t)xk);
    constexpr int WC = TN / 8;                              // chunks per row of W
    const int wrow = gt / WC, wpos = gt % WC;               // + (GT / WC) t
    const int wcol = n0 + (wpos ^ ((wrow & 2) << 1)) * 8;
    static_assert(GT / WC % 4 == 0, "row swizzle");
    const bool wcol_ok = wcol < d;

    typedef int v4 __attribute__((ext_vector_type(4)));
    v4 rx[DEPTH][XT], rw[DEPTH][WT];
#define GRAM_MID_LOAD(SET, IT)                                                                      \
    {                                                                                               \
        const int k0_ = (grp + (IT) * KG) * SK;                                                     \
        _Pragma("unroll") for (int t = 0; t < XT; ++t) {                                            \
            const uint32_t o_ = mid_slab_offset(ox[t], k0_, xk, d_in);                              \
            rx[SET][t] = __builtin_amdgcn_raw_buffer_load_b128(rsX, o_, 0, 0);                      \
        }                                                                                           \
        _Pragma("unroll") for (int t = 0; t < WT; ++t) {                                            \
            const int k_ = k0_ + wrow + t * (GT / WC);                                              \
            const uint32_t o_ = k_ < d_in && wcol_ok ? ((uint32_t)k_ * (uint32_t)d + (uint32_t)wcol) * 2u : kPastEnd; \
            rw[SET][t] = __builtin_amdgcn_raw_buffer_load_b128(rsW, o_, 0, 0);                      \
        }                                                                                           \
    }
    const int nslab = (d_in + SK - 1) / SK, iters = (nslab + KG - 1) / KG;
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) GRAM_MID_LOAD(s, s)

    f32x16 acc[WR];
#pragma unroll
    for (int i = 0; i < WR; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    unsigned char* stage = smem + grp * kStageB;
    unsigned char* wstage = stage + SM * SK * 2;
    const int j16 = lane & 15, g16 = lane >> 4;
    const int f_row = (g16 >> 1) * 8 + (j16 >> 2), f_ch = wn * 4 + (g16 & 1) * 2 + ((j16 & 3) >> 1);
    const unsigned char* fw = wstage + f_row * WROW + ((f_ch ^ ((f_row & 2) << 1)) * 16) + (j16 & 1) * 8;
    const int a_row = wm * (32 * WR) + (lane & 31), a_x = (a_row >> 1) & 7;      // + 32 i: the same swizzle
#define GRAM_MID_ITER(SET, IT, MORE)                                                                \
    {                                                                                               \
        _Pragma("unroll") for (int t = 0; t < XT; ++t)                                              \
            *reinterpret_cast<v4*>(stage + (xrow + t * (GT / 8)) * 128 + xpos * 16) = rx[SET][t];   \
        _Pragma("unroll") for (int t = 0; t < WT; ++t)                                              \
            *reinterpret_cast<v4*>(wstage + (wrow + t * (GT / WC)) * WROW + wpos * 16) = rw[SET][t]; \
        if (MORE) GRAM_MID_LOAD(SET, (IT) + DEPTH)                                                  \
        __syncthreads();                                                                            \
        _Pragma("unroll") for (int ks = 0; ks < SK / 16; ++ks) {                                    \
            const unsigned char* b_ = fw + ks * 16 * WROW;                                          \
            const sv4i16 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)b_);            \
            const sv4i16 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)(b_ + 4 * WROW)); \
            const bf16x8 fb = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7)); \
            _Pragma("unroll") for (int i = 0; i < WR; ++i) {                                         \
                const bf16x8 fa = *reinterpret_cast<const bf16x8*>(                                 \
                    stage + (a_row + i * 32) * 128 + (((ks * 2 + (lane >> 5)) ^ a_x) * 16));        \
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[i], 0, 0, 0);          \
            }                                                                                       \
        }                                                                                           \
        __syncthreads();                                                                            \
    }
    // A trip count rounded up to DEPTH costs whole slabs of zeros (776 features are 7 trips, not 9).
    static_assert(DEPTH == 2 || DEPTH == 3, "the ends of the loop");
    if constexpr (DEPTH == 3) {
        for (int it = 0;; it += DEPTH) {
            GRAM_MID_ITER(0, it, true)
            if (it + 1 >= iters) break;
            GRAM_MID_ITER(1, it + 1, true)
            if (it + 2 >= iters) break;
            GRAM_MID_ITER(2, it + 2, true)
            if (it + 3 >= iters) break;
        }
    } else {        // (exits inside the loop cost the two 128-row tiles registers: 27 spilled)
        int it = 0;
        for (; it + 1 < iters; it += DEPTH) {
            GRAM_MID_ITER(0, it, true)
            GRAM_MID_ITER(1, it + 1, true)
        }
        if (it < iters) GRAM_MID_ITER(0, it, false)
    }
#undef GRAM_MID_LOAD
#undef GRAM_MID_ITER

    // the groups' tiles, added in group order; rows of 16-byte pieces to memory
    constexpr int LD = TN + 8;
    float* parked = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < WR; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            parked[(grp * SM + wm * (32 * WR) + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * LD + wn * 32 + (lane & 31)] = acc[i][r];
    __syncthreads();
    constexpr int OUT = SM * TN / 4 / STHREADS;
    f32x4_ av[OUT];
#pragma unroll
    for (int h = 0; h < OUT; ++h) {
        const int e = tid + h * STHREADS, row = e / (TN / 4), c4 = n0 + e % (TN / 4) * 4;
        av[h] = m0 + row < U && c4 < d ? epi_load4<EPI>(aux, (int64_t)(m0 + row) * d + c4) : f32x4_{0.f, 0.f, 0.f, 0.f};
    }
    double sq = 0.0;
#pragma unroll
    for (int h = 0; h < OUT; ++h) {
        const int e = tid + h * STHREADS, row = e / (TN / 4), c = e % (TN / 4) * 4;
        f32x4_ s = *reinterpret_cast<const f32x4_*>(&parked[row * LD + c]);
#pragma unroll
        for (int g = 1; g < KG; ++g) s += *reinterpret_cast<const f32x4_*>(&parked[(g * SM + row) * LD + c]);
        if (m0 + row < U && n0 + c < d) {
            // (the padding item's product is zero only where the weights are finite)
            const bool zero = s_ids[row] == pad_id;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s[k] = epi_value<EPI>(s[k], av[h][k], zero);
                if (epi_subtracts(EPI)) sq += (double)s[k] * s[k];
            }
            epi_store4<EPI>(E, (int64_t)(m0 + row) * d + n0 + c, s);
        }
    }
    if (epi_subtracts(EPI) && loss_part) block_sum_double(sq, STHREADS, s_loss, loss_part);
}

// One tile per block; the column tiles of a row tile run on one XCD and share its rows of X.  Tiles of 64 x 64, or
// 128 x 64 (the same threads) where the items make more than `most_low` of those.
struct MidShape {
    static constexpr int kCols = 64;
    using Low = Mid<64, kCols, 2, 1>;
    using Tall = Mid<128, kCols, 2, 2>;
    static constexpr int kThreads = Tall::kThreads;
    static constexpr size_t kLds = Tall::kLds;
    static_assert(Low::kThreads == kThreads && Low::kLds <= kLds, "either tile by the same block");
};

template <int EPI>
__global__ __launch_bounds__(MidShape::kThreads, 4) void k_encode_mid(
    const uint16_t* __restrict__ X, uint32_t x_bytes, const uint16_t* __restrict__ W, uint32_t w_bytes,
    const int* __restrict__ uniq, const int* __restrict__ u_dev, int most_low, int d_in, int d,
    const int* __restrict__ zero_ids, int pad_id, float* __restrict__ E, const void* __restrict__ aux,
    double* __restrict__ loss_part)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ int s_ids[128];
    __shared__ double s_loss[MidShape::kThreads / 64];
    constexpr int TN = MidShape::kCols;
    if (epi_subtracts(EPI) && loss_part) loss_part += blockIdx.x;
    const int n_tiles = (d + TN - 1) / TN, q = blockIdx.x >> 3, qr = q / n_tiles;
    const int mt = qr * 8 + (blockIdx.x & 7), n0 = (q - qr * n_tiles) * TN;
    const int U = *u_dev;
    const bool low = (U + 63) / 64 * n_tiles <= most_low;
    const int m0 = mt * (low ? 64 : 128);
    if (m0 >= U) {
        if (epi_subtracts(EPI) && loss_part && threadIdx.x == 0) *loss_part = 0.0;
        return;
    }
    if (low)
        encode_mid_tile<64, TN, 2, 1, 3, EPI>(X, x_bytes, W, w_bytes, uniq, U, d_in, d, zero_ids, pad_id, E, aux, loss_part, m0, n0,
                                              smem, s_ids, s_loss);
    else
        encode_mid_tile<128, TN, 2, 2, 2, EPI>(X, x_bytes, W, w_bytes, uniq, U, d_in, d, zero_ids, pad_id, E, aux, loss_part, m0, n0,
                                               smem, s_ids, s_loss);
}

// ---- C[M,N] = A[M,K] . B[N,K]^T, bf16 in, fp32 out ---------------------------------
//
// 256x256 block tile, 8 waves (2 x 4, each 128 x 64 as 4 x 2 MFMA tiles of 32 x 32), K in slabs of 64, two LDS
// stages of 64 KiB.  Block indices are decoded so that the column tiles of one row tile run on the same XCD
// (consecutive block indices are dealt round-robin to the 8 XCDs) and share the strip of A through that XCD's
// L2.  Row j of A is A[row_ids[j]]; a row whose ID equals pad_id yields zeros.
//
// What bounds the loop is the matrix pipe, and with it the power the chip may draw: a slab takes 2,070 to 2,200
// cycles, its MFMAs 2,112, at 1.4 to 1.65 GHz; the epilogues of the same launch run at 2.36 (clock reads per tile).
// Three things got it there (before: slabs of 32 through registers, one barrier for
// all waves per slab, 3,400 cycles per 64 of K at 2.0 GHz):
//   - loads go straight to LDS (buffer_load ... lds), 1 KiB per wave-wide instruction: no registers, no LDS
//     store instructions.  They are throughput bound (8 rows of 128 bytes: 50 cycles each from HBM, 26 from L2),
//     so how far ahead they are requested matters little beyond the 4 segments it is here;
//   - a slab is four segments, each ended by a barrier: read the fragments of B and of the first half of the
//     wave's rows; multiply; read the second half's; multiply.  The waves of the lower row half are one segment
//     behind those of the upper: of the two waves on a SIMD one multiplies while the other reads;
//   - whatever a segment has read is in registers before its barrier, so the part of the stage that is free
//     afterwards is known, and its refill (two slabs ahead) is issued in the next reading segment.
// LDS rows: of A (and of a K-contiguous B) 128 bytes, 16-byte chunk c of row r at c ^ ((r >> 1) & 7); of an untransposed B
// (W [k, n]) 512 bytes, chunk c of row r at c ^ ((r & 3) << 2).  Either way the pieces of a fragment read cover
// every bank once.  A load writes 64 consecutive chunks, so the swizzle is applied by choosing which global
// chunk each lane fetches.
// Operands are addressed through buffer descriptors (base + 32-bit byte offset); a matrix A beyond the 4 GiB such
// a descriptor can address takes the WIDE variant, whose lanes keep 64-bit row pointers (every address it
// forms is a valid one: rows past the end are clamped).  K is a multiple of 32; an odd one is made up by the first slab, of
// which only the lower half is multiplied, so that no slab reaches behind a row (see gram_mid_rows.h).
constexpr int TM = 256, TN = 256, TK = 64;
constexpr int kGemmWaves = 8;
constexpr int TROWB = TK * 2;                          // bytes per LDS row of a K-contiguous operand
constexpr int TOPB = TM * TROWB;                       // bytes per operand and stage: A 0 and 1, then B 0 and 1
constexpr size_t TSMEM = 4 * (size_t)TOPB;
typedef int v4i32 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// fused-gather epilogue: 64 staged rows of TN floats (+16 bytes against bank conflicts)
constexpr int kScatterRowB = TN * 4 + 16;
constexpr int kScatterTileB = 64 * kScatterRowB;
constexpr size_t TSMEM_SC = 2 * (size_t)kScatterTileB;     // two staging buffers (they overlay the dead stages)
constexpr uint32_t kBufferFlags = 0x00027000;   // raw buffer: 32-bit elements, no swizzle
constexpr uint32_t kOutOfRange = 0xFFFFFFF0u;

// Loads to LDS: lane l's 16 bytes go to lds + 16 l.  Written in asm because the compiler, which cannot tell the
// stages apart, puts a wait for all of them in front of every LDS read; there is no result in a register, and the
// kernel counts the loads itself (wait_loads) before the barrier that publishes them.
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 ::"v"(voff), "s"(rsrc), "s"(soff), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void load_to_lds(const unsigned char* p, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(lds) : "memory", "m0");
}
// Waits until at most N of the wave's loads are outstanding.
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// A barrier that waits for no memory operation, and that nothing is scheduled across.
__device__ __forceinline__ void segment_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ u32x4 buffer_words(const void* base, uint32_t bytes)
{
    const uint64_t a = (uint64_t)base;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) & 0xffffu,
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), kBufferFlags};
}

// ---- the forward of mid-sized batches, long K: tiles of 128 x 128 --------------------------------
//
// About one such tile falls to a CU, so the launch lasts as long as a tile: 8 waves (2 x 4, each 64 x 32), slabs of 64
// straight to LDS in a ring of four stages of 32 KiB, requested three slabs ahead (96 KiB on their way: the rows come
// from HBM), two segments per slab as above.  (Through registers, with K cut between two groups of 8 waves whose tiles
// are added at the end, LDS stores and the second barrier took as long as the products.)
// LDS rows of X as above; rows of W are 256 bytes, chunk c of row r at c ^ ((r & 3) << 2).  Offsets out of range (padding item, rows
// behind the items, K, columns) write zeros.  Neither the list nor A is read behind the items.
// Whole forward with position copies, us, before / now: 51,200 positions over 20,000 IDs 776 x 392 48.4 / 44.4, 20,000 over
// 20,000 776 x 256 21.7 / 19.0, 16,000 over 1,000,000 776 x 1024 45.0 / 41.0; over 156 shapes (K 264 to 1,024, widths 128 to 1,024)
// none slower by more than 2 %, the geometric mean 0.963.
constexpr int QT = 128, QROWW = QT * 2, QXB = QT * TROWB, QSTAGEB = QXB + TK * QROWW, QSTAGES = 4;
constexpr int QLD = QT + 8;                             // floats per row of the parked tile
static_assert(QT * QLD * 4 <= QSTAGES * QSTAGEB, "the tile overlays the stages");

template <int EPI>
__global__ __launch_bounds__(kGemmWaves * 64) void k_encode_square(
    const uint16_t* __restrict__ X, uint32_t x_bytes, const uint16_t* __restrict__ W, uint32_t w_bytes,
    const int* __restrict__ uniq, const int* __restrict__ u_dev, int d_in, int d, const int* __restrict__ zero_ids, int pad_id,
    float* __restrict__ E, const void* __restrict__ aux, double* __restrict__ loss_part)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ int s_ids[QT];
    __shared__ double s_loss[kGemmWaves];
    if (epi_subtracts(EPI) && loss_part) loss_part += blockIdx.x;
    // the column tiles of a row tile run on one XCD and share its rows of X
    const int n_tiles = (d + QT - 1) / QT, q = blockIdx.x >> 3, qr = q / n_tiles;
    const int m0 = (qr * 8 + (blockIdx.x & 7)) * QT, n0 = (q - qr * n_tiles) * QT;
    const int U = *u_dev;
    if (m0 >= U) {
        if (epi_subtracts(EPI) && loss_part && threadIdx.x == 0) *loss_part = 0.0;
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const u32x4 rsX = buffer_words(X, x_bytes), rsW = buffer_words(W, w_bytes);

    // wave w moves rows 16 w + 8 t + lane / 8 of X, and rows 8 w + 4 t + lane / 16 of a slab of W, t = 0, 1
    uint32_t xo[2], wo[2];
    int xk[2];
    int id[2], zid[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int j = mid_list_entry(m0 + wave * 16 + t * 8 + (lane >> 3), U);
        id[t] = uniq[j];
        zid[t] = zero_ids[j];
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = wave * 16 + t * 8 + (lane >> 3);
        xk[t] = ((lane & 7) ^ (r >> 1 & 7)) * 8;
        xo[t] = mid_row_offset(m0 + r, U, zid[t] == pad_id, (uint32_t)id[t], (uint32_t)d_in, (uint32_t)xk[t]);
        const int k = wave * 8 + t * 4 + (lane >> 4), col = n0 + ((lane & 15) ^ ((k & 3) << 2)) * 8;
        wo[t] = col < d ? ((uint32_t)k * (uint32_t)d + (uint32_t)col) * 2u : kOutOfRange;
        if ((lane & 7) == 0) s_ids[r] = zid[t];
    }
    typedef __attribute__((address_space(3))) unsigned char lds_u8;
    typedef __attribute__((address_space(3))) const bf16x8 lds_frag;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem, to_w = lds0 + wave * 2048;
    const int nslab = (d_in + TK - 1) / TK;
#define GRAM_LOAD(SL)                                                                               \
    {                                                                                               \
        const uint32_t to_ = to_w + ((SL) & (QSTAGES - 1)) * QSTAGEB;                               \
        const uint32_t wk_ = (SL) < nslab ? (uint32_t)(SL) * (uint32_t)(TK * 2) * (uint32_t)d : kOutOfRange; \
        _Pragma("unroll") for (int t = 0; t < 2; ++t)                                               \
            load_to_lds(rsX, mid_slab_offset(xo[t], (SL) * TK, xk[t], d_in), 0u, to_ + t * 1024);   \
        _Pragma("unroll") for (int t = 0; t < 2; ++t)                                               \
            load_to_lds(rsW, __builtin_elementwise_add_sat(wo[t], wk_), 0u, to_ + QXB + t * 1024);  \
    }
    GRAM_LOAD(0)
    GRAM_LOAD(1)
    GRAM_LOAD(2)

    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    const int row = wm * 64 + (lane & 31);
    uint32_t ra[4], rb;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) ra[ks] = lds0 + row * TROWB + (((ks * 2 + (lane >> 5)) ^ (row >> 1 & 7)) * 16);
    {
        const int j16 = lane & 15, grp = lane >> 4, f_row = (grp >> 1) * 8 + (j16 >> 2);
        rb = lds0 + QXB + f_row * QROWW + (((wn * 4 + (grp & 1) * 2 + ((j16 & 3) >> 1)) ^ ((f_row & 3) << 2)) * 16) + (j16 & 1) * 8;
    }
    constexpr int kAhead = 2 * 4;            // loads that may be in flight when a slab is published: the next two slabs'
    wait_loads<kAhead>();
    segment_barrier();
    if (wm == 1) segment_barrier();          // the lower row half runs a segment behind
    for (int sl = 0; sl < nslab; ++sl) {
        const uint32_t stage = (uint32_t)(sl & (QSTAGES - 1)) * QSTAGEB;
        bf16x8 fa[2][4], fb[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const sv4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)(uintptr_t)(rb + stage + ks * (16 * QROWW)));
            const sv4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)(uintptr_t)(rb + stage + ks * (16 * QROWW) + 4 * QROWW));
            fb[ks] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int i = 0; i < 2; ++i) fa[i][ks] = *(lds_frag*)(uintptr_t)(ra[ks] + stage + i * (32 * TROWB));
        }
        __builtin_amdgcn_sched_barrier(0);
        GRAM_LOAD(sl + 3)
        wait_loads<kAhead>();
        wait_lds();
        segment_barrier();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][ks], fb[ks], acc[i], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        segment_barrier();
    }
#undef GRAM_LOAD
    if (wm == 0) segment_barrier();
    wait_loads<0>();
    __syncthreads();

    // the tile through LDS; rows of 16-byte pieces to memory
    float* parked = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            parked[(wm * 64 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * QLD + wn * 32 + (lane & 31)] = acc[i][r];
    constexpr int OUT = QT * QT / 4 / (kGemmWaves * 64);
    f32x4_ av[OUT];
#pragma unroll
    for (int h = 0; h < OUT; ++h) {
        const int e = tid + h * (kGemmWaves * 64), r = e / (QT / 4), c4 = n0 + e % (QT / 4) * 4;
        av[h] = m0 + r < U && c4 < d ? epi_load4<EPI>(aux, (int64_t)(m0 + r) * d + c4) : f32x4_{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    double sq = 0.0;
#pragma unroll
    for (int h = 0; h < OUT; ++h) {
        const int e = tid + h * (kGemmWaves * 64), r = e / (QT / 4), c = e % (QT / 4) * 4;
        f32x4_ s = *reinterpret_cast<const f32x4_*>(&parked[r * QLD + c]);
        if (m0 + r < U && n0 + c < d) {
            // (the padding item's product is zero only where the weights are finite)
            const bool zero = s_ids[r] == pad_id;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s[k] = epi_value<EPI>(s[k], av[h][k], zero);
                if (epi_subtracts(EPI)) sq += (double)s[k] * s[k];
            }
            epi_store4<EPI>(E, (int64_t)(m0 + r) * d + n0 + c, s);
        }
    }
    if (epi_subtracts(EPI) && loss_part) block_sum_double(sq, kGemmWaves * 64, s_loss, loss_part);
}

// How many row tiles of 256 are taken whole.  A block fills its CU (8 waves, over 200 VGPRs), so the tiles
// go in rounds of num_cus; those left over after the last full round are cut in two where the halves still
// fit one round, which then takes about 0.6 of a round of whole tiles.  The number of items is known on
// the device only, so each block works this out, by multiplications: divisions cost the prologue of every
// block 0.25 us.  (Rounded quotients only move the cut; the grid is made with the same ones.)
// Measured (with loads through registers and slabs of 32; now about a tenth less on both sides), all whole / the last ones cut: 56 x 2 tiles (K = 1536, positions stored) 53.5 / 40.5 us, 56 x 6
// tiles (K = 768) 55.7 / 51.4, the forward of 204,800 positions 1024 x 1024 to bf16 178 / 169.  Nothing left
// over, or more than half a round (where a round of halves would be followed by another): the same tiles as
// before; the cut in the prologue costs up to 1 us there (2 to 3.5 % at 24 of 384 shapes of K 32 to 1024, short K
// above all; the geometric mean over the 384 is 0.93 of the time without it).
struct TileCut {
    uint32_t rounds_per_tile;  // ceil(2^32 n_tiles / num_cus): a row tile in rounds of blocks
    uint32_t tiles_per_round;  // ceil(2^16 num_cus / n_tiles)
    int most;                  // row tiles that are cut at most

    TileCut(int n_tiles, int num_cus)
        : rounds_per_tile((uint32_t)std::min<uint64_t>((((uint64_t)n_tiles << 32) + num_cus - 1) / num_cus, UINT32_MAX)),
          tiles_per_round((uint32_t)((((uint64_t)num_cus << 16) + n_tiles - 1) / n_tiles)), most(num_cus / (2 * n_tiles)) {}
    __host__ __device__ int full_rounds(int tiles) const     // in row tiles, a multiple of the 8 XCDs
    {
        const uint32_t rounds = (uint32_t)(((uint64_t)(uint32_t)tiles * rounds_per_tile) >> 32);
        return (int)(((uint64_t)rounds * tiles_per_round) >> 16) & ~7;
    }
    __host__ __device__ int whole(int tiles) const
    {
        const int f = full_rounds(tiles);
        return tiles - f <= most ? f : tiles;
    }
    int row_tiles_max(int tiles) const       // whole and half ones that up to `tiles` of 256 rows may come to
    {
        const int f = full_rounds(tiles);
        return std::max(tiles, f + 2 * std::min(tiles - f, most));
    }
};

// MI = 32-row MFMA tiles per wave: 4 (a tile of 256 rows) or 2 (128 rows).
//
// SCATTER (forward only): the epilogue is the gather of Section 3.1 as well.  Row j of the
// product is the representation of unique item j; instead of only storing it to C it is stored
// to H[p,:] for every position p of that item (the positions of item j are perm[seg_off[j] ..
// seg_off[j+1]) in the sorted order of the dedup step), so the representations never make a
// round trip through memory.  Items with more than kLightMax positions are written to C once
// and copied to their positions by k_gather_heavy: a few hundred very popular items own half
// of the positions, and unrolling their copies here would stall a whole tile on one row.
struct ScatterArgs {
    const int* seg_off;   // [U + 1]
    const int* perm;      // [m] positions in sorted order
    void* H;              // [m, ldh] float32, or bf16 with h_bf16 (selects the kernel's HB variant)
    int64_t ldh;
    int write_all;        // also store every row to C (the caller asked for E)
    int h_bf16;
};

// HB (with SCATTER): H holds bf16, values are rounded to nearest even as they are stored.
// BDIRECT: B is not the K-contiguous [n, k] matrix but its transpose as the caller holds it,
// W [k, n] (n a multiple of 8, ldb = n): a slab of it is 64 rows of k with 256 values of n each, and the
// MFMA fragments (8 consecutive k for one n) come from the transposing LDS read, exactly as
// in k_wgrad_tn_bf16 below.  Saves the transposed copy of the weights and its launch.
template <int MI, bool SCATTER, int EPI, bool HB, bool WIDE, bool BDIRECT>
__device__ __forceinline__ void gemm_nt_tile(
    const uint16_t* __restrict__ A, int64_t lda, uint32_t a_bytes, const int* __restrict__ row_ids, int M,
    const uint16_t* __restrict__ B, int64_t ldb, uint32_t b_bytes, int n, int ktot, const int* __restrict__ zero_ids,
    int pad_id, int m0, int n0, float* __restrict__ C, int64_t ldc, const ScatterArgs& sc,
    const void* __restrict__ aux, double* __restrict__ loss_part, unsigned char* smem, uint32_t* s_pad_rows)
{
    constexpr int TM = MI * 64, NW = kGemmWaves, NT = 2, MH = MI / 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    if (tid < TM / 32) s_pad_rows[tid] = 0;      // one bit per row of the tile: the padding item
    __syncthreads();

    static_assert(TK == kBigSlab, "the slabs of gram_mid_rows.h");
    const int nslab = (ktot + TK - 1) / TK;

    // A load moves 8 rows of A (lane l: position l & 7 of row l >> 3).  Wave w moves groups MH w + t of either half:
    // half h is the rows h * 16 MI + 0 .. 16 MI - 1 of both wave rows.  Rows past M are clamped to a valid row
    // (their products are never stored).
    const u32x4 rsA = buffer_words(A, a_bytes), rsB = buffer_words(B, b_bytes);
    uint32_t oa[2][MH], la[2][MH];
    const unsigned char* pa[2][WIDE ? MH : 1];
    const int a_chunk = (lane & 7) ^ (lane >> 4 & 3);     // of the rows with (row >> 1 & 4) == 0; the others: ^ 4
    int ids[2][MH], zids[2][MH];             // (the two-layer encoder's second contraction tells the padding item by another list than its rows)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < MH; ++t) {
            const int g = wave * MH + t, r0 = g / (2 * MI) * (32 * MI) + h * (16 * MI) + g % (2 * MI) * 8;
            const int r = m0 + r0 + (lane >> 3);
            la[h][t] = r0 * TROWB;
            ids[h][t] = row_ids[r < M ? r : M - 1];
            zids[h][t] = zero_ids[r < M ? r : M - 1];
        }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < MH; ++t) {
            const int chunk = big_slab_part(a_chunk ^ ((wave * MH + t) & 1) * 4, 8, ktot);
            oa[h][t] = (uint32_t)(((int64_t)ids[h][t] * lda + chunk * 8) * 2);
            if (WIDE) pa[h][t] = reinterpret_cast<const unsigned char*>(A) + ((int64_t)ids[h][t] * lda + chunk * 8) * 2;
        }
    // A load moves 2 rows of W [k, n] (columns past n are clamped to the last chunk: their products are never
    // stored) or 8 rows of the K-contiguous B.  Wave w moves 4 of them in a row.
    uint32_t ob[BDIRECT ? 2 : 4];
#pragma unroll
    for (int t = 0; t < (BDIRECT ? 2 : 4); ++t) {
        if (BDIRECT) {
            const int krow = (wave * 4 + t) * 2 + (lane >> 5);
            int ncol = n0 + (((lane & 31) ^ ((krow & 3) << 2)) << 3);
            if (ncol > n - 8) ncol = n - 8;
            ob[t] = (uint32_t)(((int64_t)big_slab_part(krow, 1, ktot) * ldb + ncol) * 2);
        } else {
            const int r = (wave * 4 + t) * 8 + (lane >> 3), nn = n0 + r < n ? n0 + r : n - 1;
            ob[t] = (uint32_t)(((int64_t)nn * ldb + big_slab_part((lane & 7) ^ (r >> 1 & 7), 8, ktot) * 8) * 2);
        }
    }
    const uint32_t b_k_bytes = BDIRECT ? (uint32_t)(ldb * 2) : 2u;
    const int last = nslab - 1;
    typedef __attribute__((address_space(3))) unsigned char lds_u8;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem, lds_b = lds0 + 2 * TOPB + wave * 4096;

    // (fused gather) position ranges and position lists of the rows this wave will store in the
    // epilogue; fetched here so that their latency hides behind the contraction
    constexpr int RPW = 64 / NW;             // rows per wave and epilogue round
    int seg_o = 0, seg_n = 0;
    int pv[SCATTER ? MI * RPW : 1];
    if (SCATTER) {
        {
            const int k = lane & (MI * RPW - 1);
            const int lr = (wave / (NW / 2)) * (MI * 32) + (k / RPW) * 32 + (wave % (NW / 2)) * RPW + k % RPW;
            if (m0 + lr < M) {
                seg_o = sc.seg_off[m0 + lr];
                seg_n = sc.seg_off[m0 + lr + 1] - seg_o;
            }
        }
#pragma unroll
        for (int k = 0; k < MI * RPW; ++k) {
            const int cnt = __builtin_amdgcn_readlane(seg_n, k);
            const int o = __builtin_amdgcn_readlane(seg_o, k);
            pv[k] = (cnt <= kLightMax && lane < cnt) ? sc.perm[o + lane] : 0;
        }
    }

    f32x16 acc[MI][NT];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // fragment addresses: of A per k-step of 16 (+ 32 rows per MFMA tile), of W per MFMA tile (group g = lane / 16,
    // j = lane % 16, see the header comment of k_wgrad_tn_bf16)
    bf16x8 fa[MH][4], fb[NT][4];
    uint32_t ra[4], rb[BDIRECT ? NT : 4];
    {
        const int row = wm * (MI * 32) + (lane & 31), x = row >> 1 & 7;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) ra[ks] = lds0 + row * TROWB + (((ks * 2 + (lane >> 5)) ^ x) * 16);
        const int j16 = lane & 15, grp = lane >> 4;
        const int f_row = (grp >> 1) * 8 + (j16 >> 2), f_x = (j16 >> 2 & 3) << 2;
        const int brow = wn * 64 + (lane & 31);
#pragma unroll
        for (int i = 0; i < (BDIRECT ? NT : 4); ++i)
            rb[i] = lds0 + 2 * TOPB + (BDIRECT ? f_row * 512 + (((wn * (NT * 4) + i * 4 + (grp & 1) * 2 + ((j16 & 3) >> 1)) ^ f_x) * 16) + (j16 & 1) * 8
                                               : brow * TROWB + (((i * 2 + (lane >> 5)) ^ (brow >> 1 & 7)) * 16));
    }
    typedef __attribute__((address_space(3))) const bf16x8 lds_frag;
#define GRAM_LOAD_A(H, SLAB)                                                                        \
    {                                                                                               \
        const uint32_t k_ = (uint32_t)big_slab_start(WIDE && (SLAB) > last ? last : (SLAB), ktot) * 2u;\
        const uint32_t to_ = lds0 + ((SLAB) & 1) * TOPB;                                            \
        u32x4 rs_ = rsA;                                                                            \
        rs_.z = (SLAB) <= last ? rs_.z : 0u;                                                        \
        const uint32_t so_ = (SLAB) <= last ? k_ : 0u;                                              \
        _Pragma("unroll") for (int g_ = 0; g_ < MH; ++g_) {                                         \
            if (WIDE) load_to_lds(pa[H][g_] + k_, to_ + la[H][g_]);                                 \
            else load_to_lds(rs_, oa[H][g_], so_, to_ + la[H][g_]);                                 \
        }                                                                                           \
    }
#define GRAM_LOAD_B(SLAB)                                                                           \
    {                                                                                               \
        u32x4 rs_ = rsB;                                                                            \
        rs_.z = (SLAB) <= last ? rs_.z : 0u;                                                        \
        const uint32_t k_ = (uint32_t)big_slab_start(SLAB, ktot) * b_k_bytes;                       \
        const uint32_t to_ = lds_b + ((SLAB) & 1) * TOPB;                                           \
        _Pragma("unroll") for (int g_ = 0; g_ < 4; ++g_)                                            \
            load_to_lds(rs_, ob[BDIRECT ? g_ & 1 : g_], (SLAB) <= last ? (BDIRECT ? k_ + (uint32_t)(g_ >> 1) * (uint32_t)(8 * ldb) : k_) : 0u, to_ + g_ * 1024); \
    }
#define GRAM_READ_A(H, STAGE)                                                                       \
    _Pragma("unroll") for (int i = 0; i < MH; ++i)                                                  \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks)                                            \
            fa[i][ks] = *(lds_frag*)(uintptr_t)(ra[ks] + (STAGE) * TOPB + ((H) * MH + i) * (32 * TROWB));
#define GRAM_READ_B(STAGE)                                                                          \
    _Pragma("unroll") for (int j = 0; j < NT; ++j)                                                  \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {                                          \
            if (BDIRECT) {                                                                          \
                const uint32_t at_ = rb[j] + (STAGE) * TOPB + ks * (16 * 512);                      \
                const sv4i16 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)(uintptr_t)at_); \
                const sv4i16 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_sv4i16*)(uintptr_t)(at_ + 4 * 512)); \
                fb[j][ks] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7)); \
            } else {                                                                                \
                fb[j][ks] = *(lds_frag*)(uintptr_t)(rb[BDIRECT ? 0 : ks] + (STAGE) * TOPB + j * (32 * TROWB)); \
            }                                                                                       \
        }
    // (of a half slab the upper half is the next slab's: it is not multiplied here)
#define GRAM_MMA_STEPS(H, FROM)                                                                     \
    _Pragma("unroll") for (int ks = (FROM); ks < (FROM) + 2; ++ks)                                  \
        _Pragma("unroll") for (int i = 0; i < MH; ++i)                                              \
            _Pragma("unroll") for (int j = 0; j < NT; ++j)                                          \
                acc[(H) * MH + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][ks], fb[j][ks], acc[(H) * MH + i][j], 0, 0, 0);
#define GRAM_MMA(H, SL, STAGE)                                                                      \
    __builtin_amdgcn_s_setprio(1);                                                                  \
    GRAM_MMA_STEPS(H, 0)                                                                            \
    if ((STAGE) == 1 || (SL) != half_at) { GRAM_MMA_STEPS(H, 2) }                                   \
    __builtin_amdgcn_s_setprio(0);
    // Loads in flight at the end of a reading segment: what its successors wait for was issued before the last
    // kAhead (a slab's worth).  Slabs past the end write zeros (WIDE: the last one again) and are never multiplied.
    constexpr int kAhead = 4 + 2 * MH;
#define GRAM_SLAB(SL, STAGE)                                                                        \
    {                                                                                               \
        GRAM_READ_B(STAGE)                                                                          \
        GRAM_READ_A(0, STAGE)                                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                          \
        GRAM_LOAD_A(1, (SL) + 1)                                                                    \
        wait_loads<kAhead>();                                                                       \
        wait_lds();                                                                                 \
        segment_barrier();                                                                          \
        GRAM_MMA(0, SL, STAGE)                                                                      \
        segment_barrier();                                                                          \
        GRAM_READ_A(1, STAGE)                                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                          \
        if (epi_subtracts(EPI) && (SL) == last) {                                                   \
            wait_loads<0>();                                                                        \
            if (BDIRECT) { GRAM_AUX(0) }                                                            \
        } else {                                                                                    \
            GRAM_LOAD_B((SL) + 2)                                                                   \
            GRAM_LOAD_A(0, (SL) + 2)                                                                \
            wait_loads<kAhead>();                                                                   \
        }                                                                                           \
        wait_lds();                                                                                 \
        segment_barrier();                                                                          \
        GRAM_MMA(1, SL, STAGE)                                                                      \
        segment_barrier();                                                                          \
    }
    // (subtracting) the targets of the epilogue's first round are requested ahead of the last products, behind the wait for
    // whatever still lands in the stages: these are loads of the compiler's, which no count of the kernel's may include.
    // (With a K-contiguous B, whose fragments take more addresses, four registers spilled for it: 32,768 x 1024 x 1020 218.0 us with
    // the weight gradient, 215.5 without either; 33,000 x 64 x 508 61.4 and 62.7.)
    f32x4_ av[epi_subtracts(EPI) ? RPW : 1];
#define GRAM_AUX(I)                                                                                 \
    _Pragma("unroll") for (int u = 0; u < (epi_subtracts(EPI) ? RPW : 0); ++u) {                    \
        const int row_ = m0 + (wave >> 2) * (MI * 32) + (I) * 32 + (wave & 3) * RPW + u, col_ = n0 + lane * 4; \
        av[u] = epi_load4<EPI>(aux, (int64_t)(row_ < M ? row_ : M - 1) * ldc + (col_ < n ? col_ : 0)); \
    }
    // slab 0, then B and the first halves of slab 1 (its second halves are requested in slab 0)
    GRAM_LOAD_B(0)
    GRAM_LOAD_A(0, 0)
    GRAM_LOAD_A(1, 0)
    GRAM_LOAD_B(1)
    GRAM_LOAD_A(0, 1)
    // (a batch listed by the caller may hold the padding item any number of times)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < MH; ++t) {
            const int r = la[h][t] / TROWB + (lane >> 3);
            if (m0 + r < M && (lane & 7) == 0 && zids[h][t] == pad_id) atomicOr(&s_pad_rows[r >> 5], 1u << (r & 31));
        }
    wait_loads<kAhead>();
    segment_barrier();
    if (wm == 1) segment_barrier();          // the lower row half runs a segment behind
    const int half_at = big_half_slab(ktot);
    int sl = 0;
    for (; sl < last; sl += 2) {
        GRAM_SLAB(sl, 0)
        GRAM_SLAB(sl + 1, 1)
    }
    if (sl == last) GRAM_SLAB(sl, 0)
    if (wm == 0) segment_barrier();
    if (!epi_subtracts(EPI)) wait_loads<0>();        // the stages become the epilogue's (behind its barrier)

    // accumulator element r of a lane sits at (row, col) = ((r / 4) * 8 + (lane / 32) * 4 + r % 4, lane % 32)
    // the rows a wave stores are the 32 of MFMA row block i of its wave row: their padding bits
    const int cr0 = (wave / (NW / 2)) * 32 + (wave % (NW / 2)) * RPW;           // first staged row
    uint32_t pads[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) pads[i] = __builtin_amdgcn_readfirstlane(s_pad_rows[(cr0 >> 5) * MI + i]) >> (cr0 & 31) & ((1u << RPW) - 1);
    if (SCATTER) {
        // The stages are dead.  The tile goes through LDS 64 rows at a time (the 32 rows of MFMA
        // row block i of both wave rows), so that a wave can then store whole 1 KiB row pieces,
        // 16 bytes per lane: once to C for a heavy item, once per position for a light one.
        // Wave w stores rows (w / 4) * 128 + i * 32 + (w % 4) * 8 + u of the tile (u < 8) in round
        // i; lane l < 32 fetches the position range of row i = l / 8, u = l % 8, and the position
        // lists themselves (lane t: position t of the row) are fetched for all 32 rows at once,
        // so their latency is paid once.
        const bool col_ok = n0 + lane * 4 < n;
        // The position lists arrived long ago.  Reading them here once makes the compiler wait for
        // them here once; otherwise every row's store loop would begin with a wait for all vector
        // memory operations, i.e. for the stores of the rows before it.
#pragma unroll
        for (int k = 0; k < MI * RPW; ++k) asm volatile("" : "+v"(pv[k]));
        __syncthreads();
        // two staging buffers: a wave that has stored its rows of round i stages round i + 1
        // while the others still store, and one barrier per round is enough (round i + 2 reuses
        // the buffer of round i only after the barrier of round i + 1)
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            unsigned char* stage = smem + (i & 1) * kScatterTileB;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rr = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                float* dst = reinterpret_cast<float*>(stage + (wm * 32 + rr) * kScatterRowB) +
                             wn * (NT * 32) + (lane & 31);
#pragma unroll
                for (int jj = 0; jj < NT; ++jj) dst[jj * 32] = acc[i][jj][r];
            }
            __syncthreads();
            f32x4 v[RPW];
#pragma unroll
            for (int u = 0; u < RPW; ++u)
                v[u] = *reinterpret_cast<const f32x4*>(stage + (cr0 + u) * kScatterRowB + lane * 16);
            if (pads[i] != 0) {
#pragma unroll
                for (int u = 0; u < RPW; ++u)
                    if (pads[i] >> u & 1) v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < RPW; ++u) {
                const int lr = (cr0 >> 5) * (MI * 32) + i * 32 + (cr0 & 31) + u;         // row of the tile
                const int cnt = __builtin_amdgcn_readlane(seg_n, i * RPW + u);
                if (cnt == 0) continue;
                if (cnt > kLightMax || sc.write_all) {
                    if (col_ok) *reinterpret_cast<f32x4*>(C + (int64_t)(m0 + lr) * ldc + n0 + lane * 4) = v[u];
                    if (cnt > kLightMax) continue;
                }
                if (HB) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    const u32x2 h = {pack_bf16x2(v[u].x, v[u].y), pack_bf16x2(v[u].z, v[u].w)};
                    for (int t = 0; t < cnt; ++t) {
                        const int pos = __builtin_amdgcn_readlane(pv[i * RPW + u], t);
                        if (col_ok)
                            __builtin_nontemporal_store(h, reinterpret_cast<u32x2*>(static_cast<uint16_t*>(sc.H) + (int64_t)pos * sc.ldh + n0 + lane * 4));
                    }
                } else {
                    for (int t = 0; t < cnt; ++t) {
                        const int pos = __builtin_amdgcn_readlane(pv[i * RPW + u], t);
                        if (col_ok)
                            __builtin_nontemporal_store(v[u], reinterpret_cast<f32x4*>(static_cast<float*>(sc.H) + (int64_t)pos * sc.ldh + n0 + lane * 4));
                    }
                }
            }
        }
    } else if constexpr (EPI == kEpiReluBf16 || EPI == kEpiGateBf16) {
        // Straight from the accumulators: neighbouring lanes exchange a value, so that the even one holds two columns of its row
        // r and the odd one of row r + 1, 4 bytes each, 64 bytes of four rows per store.  What lies behind M or n falls out of
        // the descriptors: by the lane's own offset, the only one that the range check is sure to cover.  32,768 x 1024 x 1024 with the rectifier 69 us, 72 through LDS (49,152 rows: 102.5, 106).  The
        // modes with float32 targets are better off in whole row pieces: subtracting 97 us through LDS, 100 straight.
        const int rows = M - m0 < TM ? M - m0 : TM, odd = lane & 1;
        const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<uint16_t*>(C) + (int64_t)m0 * ldc, 0, (uint32_t)rows * (uint32_t)ldc * 2u, kBufferFlags);
        const __amdgpu_buffer_rsrc_t rsX = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(static_cast<const uint16_t*>(EPI == kEpiGateBf16 ? aux : C)) + (int64_t)m0 * ldc, 0,
            (uint32_t)rows * (uint32_t)ldc * 2u, kBufferFlags);
        uint32_t at[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = n0 + wn * 64 + j * 32 + (lane & 31);
            at[j] = col < n ? ((uint32_t)(wm * (MI * 32) + (lane >> 5) * 4 + odd) * (uint32_t)ldc + (uint32_t)(col - odd)) * 2u : kOutOfRange;
        }
        auto below = [&](uint32_t from, int down) { return __builtin_elementwise_add_sat(from, (uint32_t)down * (uint32_t)ldc * 2u); };
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            // register pair r (even): rows i * 32 + (r / 4) * 8 + r % 4 and the next, + 4 (lane / 32)
            uint32_t av[NT][8];
            if (EPI == kEpiGateBf16)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int p = 0; p < 8; ++p)
                        av[j][p] = __builtin_amdgcn_raw_buffer_load_b32(rsX, below(at[j], i * 32 + (p >> 1) * 8 + (p & 1) * 2), 0, 0);
            const uint32_t pads = s_pad_rows[wm * MI + i] >> ((lane >> 5) * 4);
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const int row = (p >> 1) * 8 + (p & 1) * 2;
                    constexpr int kMode = EPI == kEpiGateBf16 ? kEpiPlain : EPI;
                    const float lo = epi_value<kMode>(acc[i][j][2 * p], 0.f, pads >> row & 1);
                    const float hi = epi_value<kMode>(acc[i][j][2 * p + 1], 0.f, pads >> row & 2);
                    const float got = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(odd ? lo : hi), 0xb1, 0xf, 0xf, false));
                    uint32_t h = odd ? pack_bf16x2(got, hi) : pack_bf16x2(lo, got);
                    if (EPI == kEpiGateBf16)        // open where the activation is positive
                        h &= ((av[j][p] & 0xffffu) - 1u < 0x7fffu ? 0xffffu : 0u) | ((av[j][p] >> 16) - 1u < 0x7fffu ? 0xffff0000u : 0u);
                    __builtin_amdgcn_raw_buffer_store_b32(h, rsC, below(at[j], i * 32 + row), 0, 0);
                }
        }
    } else if constexpr (EPI == kEpiPlain) {
        // Straight from the accumulators as well, 128 bytes of two rows per store: 33,000 x 64 x 512 19.6 us, 20.4 through LDS.
        const int rows = M - m0 < TM ? M - m0 : TM;
        const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(C + (int64_t)m0 * ldc, 0, (uint32_t)rows * (uint32_t)ldc * 4u, kBufferFlags);
        uint32_t at[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = n0 + wn * 64 + j * 32 + (lane & 31);
            at[j] = col < n ? ((uint32_t)(wm * (MI * 32) + (lane >> 5) * 4) * (uint32_t)ldc + (uint32_t)col) * 4u : kOutOfRange;
        }
        auto below = [&](uint32_t from, int down) { return __builtin_elementwise_add_sat(from, (uint32_t)down * (uint32_t)ldc * 4u); };
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const uint32_t pads = s_pad_rows[wm * MI + i] >> ((lane >> 5) * 4);
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int row = (r >> 2) * 8 + (r & 3);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(pads >> row & 1 ? 0.f : acc[i][j][r]), rsC, below(at[j], i * 32 + row), 0, 0);
                }
        }
    } else {
        static_assert(epi_subtracts(EPI), "what the branches above leave");
        // Staged like the fused gather's epilogue, 64 rows at a time: a wave then loads and stores whole row
        // pieces, 4 columns per lane.
        const int col = n0 + lane * 4;
        const bool col_ok = col < n;
        double sq = 0.0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row0 = m0 + (cr0 >> 5) * (MI * 32) + i * 32 + (cr0 & 31);           // + u
            if (i > 0 || !BDIRECT) { GRAM_AUX(i) }
            unsigned char* stage = smem + (i & 1) * kScatterTileB;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rr = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                float* dst = reinterpret_cast<float*>(stage + (wm * 32 + rr) * kScatterRowB) + wn * (NT * 32) + (lane & 31);
#pragma unroll
                for (int jj = 0; jj < NT; ++jj) dst[jj * 32] = acc[i][jj][r];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < RPW; ++u) {
                f32x4_ v = *reinterpret_cast<const f32x4_*>(stage + (cr0 + u) * kScatterRowB + lane * 16);
                const bool zero = pads[i] >> u & 1;
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = epi_value<EPI>(v[k], av[u][k], zero);
                if (row0 + u < M && col_ok) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) sq += (double)v[k] * v[k];
                    epi_store4<EPI>(C, (int64_t)(row0 + u) * ldc + col, v);
                }
            }
        }
        if (loss_part) {
            __syncthreads();
            block_sum_double(sq, NW * 64, reinterpret_cast<double*>(smem), loss_part);
        }
    }
}
#undef GRAM_LOAD_A
#undef GRAM_LOAD_B
#undef GRAM_READ_A
#undef GRAM_READ_B
#undef GRAM_MMA_STEPS
#undef GRAM_MMA
#undef GRAM_SLAB
#undef GRAM_AUX

// One tile per block, of 256 rows or (the last ones, see TileCut) of 128.
template <bool SCATTER, int EPI = kEpiPlain, bool HB = false, bool WIDE = false, bool BDIRECT = false>
__global__ __launch_bounds__(kGemmWaves * 64) void k_gemm_nt_bf16(
    const uint16_t* __restrict__ A, int64_t lda, uint32_t a_bytes, const int* __restrict__ row_ids,
    const int* __restrict__ m_dev, const uint16_t* __restrict__ B, int64_t ldb, uint32_t b_bytes, int n,
    int ktot, const int* __restrict__ zero_ids, int pad_id, int n_tiles, TileCut cut, float* __restrict__ C, int64_t ldc,
    ScatterArgs sc, const void* __restrict__ aux, double* __restrict__ loss_part)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ uint32_t s_pad_rows[TM / 32];
    const int M = *m_dev;
    // row tiles are dealt to the XCDs; the column tiles of a row tile stay together
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int u = (q / n_tiles) * 8 + xcd, n0 = (q % n_tiles) * TN;
    const int full = cut.whole((M + TM - 1) / TM);
    const int m0 = u < full ? u * TM : full * TM + (u - full) * (TM / 2);
    if (epi_subtracts(EPI) && loss_part) loss_part += blockIdx.x;
    if (m0 >= M) {
        if (epi_subtracts(EPI) && loss_part && threadIdx.x == 0) *loss_part = 0.0;
        return;
    }
    if (u < full)
        gemm_nt_tile<4, SCATTER, EPI, HB, WIDE, BDIRECT>(A, lda, a_bytes, row_ids, M, B, ldb, b_bytes, n, ktot, zero_ids,
                                                                     pad_id, m0, n0, C, ldc, sc, aux, loss_part, smem, s_pad_rows);
    else
        gemm_nt_tile<2, SCATTER, EPI, HB, WIDE, BDIRECT>(A, lda, a_bytes, row_ids, M, B, ldb, b_bytes, n, ktot, zero_ids,
                                                                     pad_id, m0, n0, C, ldc, sc, aux, loss_part, smem, s_pad_rows);
}

template <bool SCATTER, int EPI, bool HB, bool WIDE, bool BDIRECT = false>
static void launch_gemm_variant(Ctx* c, int kid, unsigned blocks, hipStream_t s, const uint16_t* A, int64_t lda,
                                int64_t a_bytes, const int* row_ids, const int* m_dev, const uint16_t* B,
                                int64_t ldb, int64_t b_bytes, int n, int k, const int* zero_ids, int pad_id, int n_tiles,
                                float* C, int64_t ldc, const ScatterArgs& sc, const void* aux, double* loss_part)
{
    constexpr auto kern = k_gemm_nt_bf16<SCATTER, EPI, HB, WIDE, BDIRECT>;
    constexpr size_t smem = TSMEM_SC > TSMEM ? TSMEM_SC : TSMEM;
    ensure_dynamic_lds<kern>((int)smem);
    // the descriptor of a WIDE operand is not used; any size that fits its field will do
    launch_smem(c, kid, kern, dim3(blocks), dim3(kGemmWaves * 64), smem, s, A, lda,
                (uint32_t)(WIDE ? 0 : a_bytes), row_ids, m_dev, B, ldb, (uint32_t)b_bytes, n, k, zero_ids, pad_id, n_tiles, TileCut(n_tiles, c->num_cus), C,
                ldc, sc, aux, loss_part);
}

// C[j,:] = epi(A[row_ids[j],:k] . B^T) for j < *m_dev <= m_bound with the 256x256 kernel.
// a_rows / b_rows: rows of the matrices A and B as allocated (A: all rows that row_ids may
// name).  A may lie beyond 4 GiB for the plain epilogue (with or without the fused gather);
// the other epilogue modes and B need buffer descriptors (callers check).
// b_direct: B is the [k, n] matrix as the caller holds it (ldb = n, b_rows = k, n a multiple of 8)
// instead of its K-contiguous transpose; available for A below 4 GiB and every mode but "gate".
static void launch_gemm_nt(Ctx* c, const uint16_t* A, int64_t lda, int64_t a_rows, const int* row_ids,
                           const int* m_dev, int64_t m_bound, const uint16_t* B, int64_t ldb, int64_t b_rows,
                           int n, int k, float* C, int64_t ldc, hipStream_t s, const ScatterArgs* scatter,
                           const int* zero_ids, int pad_id, int epi, const void* aux, const EpiLoss* loss, bool b_direct = false)
{
    const int n_tiles = (n + TN - 1) / TN;
    const unsigned blocks =
        (unsigned)((TileCut(n_tiles, c->num_cus).row_tiles_max((int)((m_bound + TM - 1) / TM)) + 7) / 8 * 8 * n_tiles);
    const int64_t a_bytes = a_rows * lda * 2, b_bytes = b_rows * ldb * 2;
    const bool wide = a_bytes >= kBufferWindow;
    double* loss_part = loss ? loss->part : nullptr;
    if (loss) *loss->blocks = (int)blocks;
    const int kid = wide ? KID_ENCODE_BF16_WIDE : KID_ENCODE_BF16;
    const ScatterArgs none = {nullptr, nullptr, nullptr, 0, 0, 0};
#define GRAM_GO(SC, EPI, HB, WIDE, ARGS)                                                            \
    launch_gemm_variant<SC, EPI, HB, WIDE>(c, kid, blocks, s, A, lda, a_bytes, row_ids, m_dev, B, ldb, b_bytes, n, \
                                           k, zero_ids, pad_id, n_tiles, C, ldc, ARGS, aux, loss_part)
#define GRAM_GO_DIRECT(SC, EPI, HB, ARGS)                                                           \
    launch_gemm_variant<SC, EPI, HB, false, true>(c, kid, blocks, s, A, lda, a_bytes, row_ids, m_dev, B, ldb, b_bytes, n, \
                                                  k, zero_ids, pad_id, n_tiles, C, ldc, ARGS, aux, loss_part)
    if (b_direct) {
        if (epi == kEpiReluBf16) GRAM_GO_DIRECT(false, kEpiReluBf16, false, none);
        else if (epi == kEpiMinus) GRAM_GO_DIRECT(false, kEpiMinus, false, none);
        else if (epi == kEpiMinusBf16) GRAM_GO_DIRECT(false, kEpiMinusBf16, false, none);
        else if (scatter && scatter->h_bf16) GRAM_GO_DIRECT(true, kEpiPlain, true, *scatter);
        else if (scatter) GRAM_GO_DIRECT(true, kEpiPlain, false, *scatter);
        else GRAM_GO_DIRECT(false, kEpiPlain, false, none);
    } else if (epi == kEpiReluBf16) GRAM_GO(false, kEpiReluBf16, false, false, none);
    else if (epi == kEpiMinus) GRAM_GO(false, kEpiMinus, false, false, none);
    else if (epi == kEpiMinusBf16) GRAM_GO(false, kEpiMinusBf16, false, false, none);
    else if (epi == kEpiGateBf16) GRAM_GO(false, kEpiGateBf16, false, false, none);
    else if (scatter && scatter->h_bf16) {
        if (wide) GRAM_GO(true, kEpiPlain, true, true, *scatter);
        else GRAM_GO(true, kEpiPlain, true, false, *scatter);
    } else if (scatter) {
        if (wide) GRAM_GO(true, kEpiPlain, false, true, *scatter);
        else GRAM_GO(true, kEpiPlain, false, false, *scatter);
    } else {
        if (wide) GRAM_GO(false, kEpiPlain, false, true, none);
        else GRAM_GO(false, kEpiPlain, false, false, none);
    }
#undef GRAM_GO
#undef GRAM_GO_DIRECT
}

// ---- 64x64 bf16 transpose through LDS (16-byte global accesses both ways) ----------

constexpr int TT = 64;   // transpose tile edge

// Wt[cols, rows] = W[rows, cols]^T; rows and cols multiples of 8.
__global__ __launch_bounds__(kBlock) void k_transpose_w(const uint16_t* __restrict__ W, int rows, int cols,
                                                        uint16_t* __restrict__ Wt)
{
    __shared__ uint16_t tile[TT][TT + 2];     // [row of W][column of W]
    const int r_tiles = (rows + TT - 1) / TT, c_tiles = (cols + TT - 1) / TT;
    for (int t = blockIdx.x; t < r_tiles * c_tiles; t += gridDim.x) {
        const int r0 = (t / c_tiles) * TT, c0 = (t % c_tiles) * TT;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int cid = threadIdx.x + h * kBlock;
            const int row = cid >> 3, ch = (cid & 7) * 8;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (r0 + row < rows && c0 + ch < cols)
                v = *reinterpret_cast<const uint4*>(W + (int64_t)(r0 + row) * cols + c0 + ch);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) tile[row][ch + e] = (uint16_t)(w[e >> 1] >> ((e & 1) * 16));
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int cid = threadIdx.x + h * kBlock;
            const int r = cid >> 3, ch = (cid & 7) * 8;
            if (c0 + r < cols && r0 + ch < rows) {
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = (uint32_t)tile[ch + 2 * e][r] | ((uint32_t)tile[ch + 2 * e + 1][r] << 16);
                *reinterpret_cast<uint4*>(Wt + (int64_t)(c0 + r) * rows + r0 + ch) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
        __syncthreads();
    }
}

// ---- forward, float32 --------------------------------------------------------

// The operands of 16 products are requested together (one product at a time, each term of the sum waited
// for a round trip of its own: 10.0 us for 64 terms, now 3.7).
__global__ __launch_bounds__(kBlock) void k_encode_f32(
    const float* __restrict__ X, const float* __restrict__ W, const int* __restrict__ uniq,
    const int* __restrict__ u_dev, int d_in, int d, int pad_id, float* __restrict__ E)
{
    const int U = *u_dev;
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (j >= U || c >= d) return;
    const int id = uniq[j];
    float acc = 0.f;
    if (id != pad_id) {
        const float* x = X + (int64_t)id * d_in;
        const float* w = W + c;
        int k = 0;
        for (; k + 16 <= d_in; k += 16) {
            float xv[16], wv[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                xv[u] = x[k + u];
                wv[u] = w[(int64_t)(k + u) * d];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) acc = fmaf(xv[u], wv[u], acc);
        }
        for (; k < d_in; ++k) acc = fmaf(x[k], w[(int64_t)k * d], acc);
    }
    E[(int64_t)j * d + c] = acc;
}

// Wt[cols, rows] = W[rows, cols]^T for a bf16 matrix whose rows count is a multiple of 8.
void transpose_weight(Ctx* c, const void* W, int rows, int cols, void* Wt, hipStream_t s)
{
    // 16-byte row chunks of W^T never straddle its end because rows is a multiple of 8
    if (cols % 8 == 0) {
        const int tiles = ((rows + TT - 1) / TT) * ((cols + TT - 1) / TT);
        launch(c, KID_TRANSPOSE_U16, k_transpose_w, dim3(tiles < 1024 ? tiles : 1024), dim3(kBlock), s,
               static_cast<const uint16_t*>(W), rows, cols, static_cast<uint16_t*>(Wt));
    } else {
        launch(c, KID_TRANSPOSE_U16, k_transpose_u16, dim3((cols + 31) / 32, (rows + 31) / 32), dim3(kBlock), s,
               static_cast<const uint16_t*>(W), rows, cols, static_cast<uint16_t*>(Wt));
    }
}

static bool takes_mid_kernel(int64_t a_rows, int k, int n_out, int epi);

// Up to K = 160 tiles of 256 columns lose to tiles of 64 where the latter span at most half of the columns (widths to 128) or,
// in batches that are not too large, 5/8 of them (257 to 320).  Whole content-encoder batch in us, 256 x 256 / mid-sized kernel,
// subtracting: 66,000 rows K = 96 width 64 44.1 / 34.4, 128 48.7 / 41.3, 168 51.2 / 49.9; 400,000 rows 173 / 127, 300 / 288 and 308 / 345;
// 33,000 rows K = 160 width 264 50.5 / 48.7, 336 55.7 / 58.9; 100,000 rows K = 128 width 264 105.8 / 99.1, K = 160 136.8 / 142.3;
// 200,000 rows K = 64 width 304 223.6 / 230.7.  Two-layer backward (the rectified form): 66,000 rows K = 96 hidden width 64 91.4 / 74.4,
// 264 126.2 / 122.1; 400,000 rows 332 / 263 and 746 / 754.
static bool narrow_short_k(int64_t rows_max, int n_out, int k)
{
    if (k > 160) return false;
    const int64_t tiles64 = ((int64_t)n_out + 63) / 64, span64 = ((int64_t)n_out + TN - 1) / TN * (TN / 64);
    return 2 * tiles64 <= span64 || (8 * tiles64 <= 5 * span64 && rows_max <= (k <= 128 ? 131072 : 49152));
}

// Batches that give the 256x256 kernel a tile for every CU (and a K that fits its slabs) take it, but for narrow ones
// of short K (not in the plain form, whose 256-row kernel stores the positions too);
// the rest take k_encode_mid or, where that does not apply, the 64-row kernel, which addresses its operands
// through plain pointers and therefore also serves the epilogue modes when A lies beyond 4 GiB.
static bool takes_big_kernel(const Ctx* c, int64_t rows_max, int n_out, int k, int64_t a_rows, int epi)
{
    const int64_t tile_bound = ((rows_max + TM - 1) / TM) * ((n_out + TN - 1) / TN);
    if (epi != kEpiPlain && a_rows * k * 2 >= kBufferWindow) return false;
    if (epi != kEpiPlain && narrow_short_k(rows_max, n_out, k) && takes_mid_kernel(a_rows, k, n_out, epi)) return false;
    return tile_bound >= c->num_cus && k % 32 == 0 && n_out < (1 << 22);     // (32-bit offsets within a tile of C)
}

// The 256x256 kernel reads the second operand untransposed for these shapes and modes.
static bool big_kernel_reads_plain_b(int64_t a_rows, int k, int n_out, int epi)
{
    return n_out % 8 == 0 && n_out >= 8 && epi != kEpiGateBf16 && a_rows * k * 2 < kBufferWindow &&
           (int64_t)k * n_out * 2 < kBufferWindow;
}

// Blocks of the widest grid gemm_rows_bf16 launches for up to `rows` rows: the 64 x 64 tiles.  (The big kernel
// has at least num_cus tiles r x t of 256 x 256, so the row tiles that may be cut are at most r / 2 and its
// blocks at most 8 ceil(1.5 r / 8) t, below the 8 ceil((4 r - 3) / 8) (4 t - 3) of these.)
int64_t epi_loss_blocks_max(int64_t rows, int64_t n_out)
{
    return ((rows + BM - 1) / BM + 7) / 8 * 8 * ((n_out + BN - 1) / BN);
}

// The kernel for small and mid-sized batches: the second operand untransposed, descriptors for both.
static bool takes_mid_kernel(int64_t a_rows, int k, int n_out, int epi)
{
    return n_out % 8 == 0 && epi != kEpiGateBf16 && a_rows * k * 2 < kBufferWindow && (int64_t)k * n_out * 2 < kBufferWindow;
}

// Whether gemm_rows_bf16 will read B_plain (the [k, n_out] matrix as the caller holds it) instead of
// the transposed copy Bt for this problem: callers skip the transpose launch then.
bool gemm_reads_plain_b(const Ctx* c, int64_t rows_max, int64_t a_rows, int k, int n_out, int epi)
{
    if (takes_big_kernel(c, rows_max, n_out, k, a_rows, epi)) return big_kernel_reads_plain_b(a_rows, k, n_out, epi);
    if (takes_mid_kernel(a_rows, k, n_out, epi)) return true;
    return n_out % 8 == 0 && (epi == kEpiPlain || epi == kEpiMinus);
}

bool gemm_rows_bf16(Ctx* c, const void* A, int64_t a_rows, int k, const int* row_ids, int pad_id,
                    const int* n_dev, int64_t rows_max, const void* Bt, int n_out, float* C, hipStream_t s,
                    void* H_scatter, bool caller_wants_C, int epi, const void* aux, const void* B_plain,
                    const int* zero_ids, const EpiLoss* loss)
{
    if (rows_max <= 0) return false;
    if (!zero_ids) zero_ids = row_ids;
    double* loss_part = loss ? loss->part : nullptr;
    if (takes_big_kernel(c, rows_max, n_out, k, a_rows, epi)) {
        // Fusing the gather pays when there are tiles for every CU: with a handful of tiles the
        // position stores of a tile run on one CU while a separate gather spreads over all.
        const bool fuse = H_scatter && epi == kEpiPlain;
        const ScatterArgs sc = {c->offsets, c->perm, H_scatter, (int64_t)n_out, caller_wants_C ? 1 : 0,
                               c->cfg.h_dtype == GRAM_BF16 ? 1 : 0};
        if (big_kernel_reads_plain_b(a_rows, k, n_out, epi) && B_plain)
            launch_gemm_nt(c, static_cast<const uint16_t*>(A), k, a_rows, row_ids, n_dev, rows_max,
                           static_cast<const uint16_t*>(B_plain), n_out, k, n_out, k, C, n_out, s,
                           fuse ? &sc : nullptr, zero_ids, pad_id, epi, aux, loss, true);
        else
            launch_gemm_nt(c, static_cast<const uint16_t*>(A), k, a_rows, row_ids, n_dev, rows_max,
                           static_cast<const uint16_t*>(Bt), k, n_out, n_out, k, C, n_out, s, fuse ? &sc : nullptr,
                           zero_ids, pad_id, epi, aux, loss);
        return fuse;
    }
    if (B_plain && takes_mid_kernel(a_rows, k, n_out, epi)) {
        const uint32_t x_bytes = (uint32_t)(a_rows * k * 2), w_bytes = (uint32_t)((int64_t)k * n_out * 2);
        // The number of items is known on the device only, and the kernel chooses between tiles of 64 and 128
        // rows by it: the lower ones up to one per CU.  Only the 128 x 128 tiles (k_encode_square) have to be
        // chosen here, from a guess: all IDs of a vocabulary met many times over, 0.6 of one met a few times, else
        // 0.4 of the positions (Zipf laws of the tests and the benchmark: 0.22 to 0.6).  They gain where about one of them
        // falls to a CU, the more the longer K is; up to K = 256 a guess that fails costs more than they gain: chosen from
        // K > 128 and from fewer tiles they were 3 to 20 % faster where most positions name an item of their own and 5 to 16 %
        // slower where few do.  (One kernel that holds all three shapes and goes by the number of items: more than 2 % slower at
        // 79 of 287 shapes, since every block then asks for 128 KiB of LDS and a CU holds one.)
        // Event to event with cold operands, position copies included, in us for 64 x 64 / 128 x 64 tiles (the
        // 64-row kernel in brackets): 1,200 items 768 x 776 19.5 / 19.4 (18.0); 4,000 items 1544 x 256
        // 24.9 / 30.5 (25.0); 17,300 items 264 x 192 33.9 / 32.3 (33.0).
        int64_t guess = rows_max;
        if (n_dev != c->scal + kSChunkN)
            guess = c->cur_m >= 8 * (int64_t)c->cfg.vocab_n ? rows_max : c->cur_m >= c->cfg.vocab_n ? rows_max * 3 / 5 : rows_max * 2 / 5;
        const int64_t tiles_c = (n_out + 63) / 64, tiles64 = (guess + 63) / 64 * tiles_c;
        const bool wide = k > 256 && tiles64 * 2 > 5 * (int64_t)c->num_cus;
        // tiles of 64 rows as long as they may be chosen, tiles of 128 rows
        const int64_t most_low = c->num_cus, low_rows = std::min((rows_max + 63) / 64, most_low / tiles_c);
        const int64_t tall_rows = (rows_max + 127) / 128;
        const unsigned blocks = (unsigned)((wide ? tall_rows : std::max(low_rows, tall_rows)) + 7) / 8 * 8 *
                                (unsigned)(wide ? (n_out + 127) / 128 : tiles_c);
        if (loss) *loss->blocks = (int)blocks;
#define GRAM_GO_MID(EPI_)                                                                           \
    if (wide) {                                                                                     \
        constexpr auto kern = k_encode_square<EPI_>;                                                \
        ensure_dynamic_lds<kern>(QSTAGES * QSTAGEB);                                                \
        launch_smem(c, KID_ENCODE_BF16, kern, dim3(blocks), dim3(kGemmWaves * 64), QSTAGES * QSTAGEB, s, static_cast<const uint16_t*>(A), \
                    x_bytes, static_cast<const uint16_t*>(B_plain), w_bytes, row_ids, n_dev, k, n_out, zero_ids, pad_id, C, aux, loss_part); \
    } else {                                                                                        \
        constexpr auto kern = k_encode_mid<EPI_>;                                                   \
        ensure_dynamic_lds<kern>((int)MidShape::kLds);                                              \
        launch_smem(c, KID_ENCODE_BF16, kern, dim3(blocks), dim3(MidShape::kThreads), MidShape::kLds, s, static_cast<const uint16_t*>(A), \
                    x_bytes, static_cast<const uint16_t*>(B_plain), w_bytes, row_ids, n_dev, (int)most_low, k, n_out, \
                    zero_ids, pad_id, C, aux, loss_part);                                           \
    }
        if (epi == kEpiMinus) { GRAM_GO_MID(kEpiMinus) }
        else if (epi == kEpiMinusBf16) { GRAM_GO_MID(kEpiMinusBf16) }
        else if (epi == kEpiReluBf16) { GRAM_GO_MID(kEpiReluBf16) }
        else { GRAM_GO_MID(kEpiPlain) }
#undef GRAM_GO_MID
        return false;
    }
    const dim3 grid((n_out + BN - 1) / BN, (unsigned)((rows_max + BM - 1) / BM));
    if (loss) *loss->blocks = (int)(grid.x * grid.y);
    // the untransposed second operand, where the kernel reads it itself
    const bool plain = B_plain && n_out % 8 == 0 && (epi == kEpiPlain || epi == kEpiMinus);
    const void* B = plain ? B_plain : Bt;
    auto go = [&](auto kern) {
        launch(c, KID_ENCODE_BF16, kern, grid, dim3(kBlock), s, static_cast<const uint16_t*>(A),
               static_cast<const uint16_t*>(B), row_ids, n_dev, k, n_out, zero_ids, pad_id, C, aux, loss_part);
    };
    if (plain && epi == kEpiMinus) go(k_encode_bf16<kEpiMinus, true>);
    else if (plain) go(k_encode_bf16<kEpiPlain, true>);
    else if (epi == kEpiReluBf16) go(k_encode_bf16<kEpiReluBf16>);
    else if (epi == kEpiMinus) go(k_encode_bf16<kEpiMinus>);
    else if (epi == kEpiMinusBf16) go(k_encode_bf16<kEpiMinusBf16>);
    else if (epi == kEpiGateBf16) go(k_encode_bf16<kEpiGateBf16>);
    else go(k_encode_bf16<kEpiPlain>);
    return false;
}

bool encode_forward(Ctx* c, const void* X, const void* W, const int* uniq, const int* u_dev,
                    int64_t rows_max, float* E, hipStream_t s, void* H_scatter, bool caller_wants_E, int epi,
                    const void* aux, const EpiLoss* loss)
{
    if (rows_max <= 0) return false;
    const int d_in = c->cfg.d_in, d = c->cfg.d;
    if (c->cfg.xw_dtype == GRAM_BF16) {
        // both kernels can read W as it is for most shapes (no transposed copy, one launch less)
        const bool direct = gemm_reads_plain_b(c, rows_max, c->cfg.vocab_n, d_in, d, epi);
        if (!direct) transpose_weight(c, W, d_in, d, c->Wt, s);
        return gemm_rows_bf16(c, X, c->cfg.vocab_n, d_in, uniq, c->cfg.pad_id, u_dev, rows_max, c->Wt, d, E, s,
                              H_scatter, caller_wants_E, epi, aux, direct ? W : nullptr, nullptr, loss);
    }
    launch(c, KID_ENCODE_F32, k_encode_f32, dim3((d + 63) / 64, (unsigned)((rows_max + 3) / 4)),
           dim3(kBlock), s, static_cast<const float*>(X), static_cast<const float*>(W), uniq, u_dev,
           d_in, d, c->cfg.pad_id, E);
    return false;
}

// ---- weight gradient -----------------------------------------------------------
//
// The output is small (d_in x d) and the contraction runs over all rows of the
// persistent buffer, so the rows are cut into `splits` contiguous ranges
// (split-K); each range writes a float32 partial and k_wgrad_reduce adds the
// partials in range order.  The ranges depend only on the number of rows in
// the buffer, so the result is reproducible.
//
// ---- weight gradient without transposed copies ---------------------------------------
//
// dW[i,c] = sum_s X[item_s, i] * bf16(G[s, c]): both operands have the contraction
// index s (buffer row) as their slow dimension in memory.  Instead of first
// writing transposed copies, this kernel loads 32 buffer rows x 256 features of
// X (gathered through id_of_slot) and 32 x 256 columns of G per slab, rounds G
// to bf16 in registers, parks both in LDS as [s][256] rows and builds the MFMA
// fragments with the transposing LDS read of gfx950 (ds_read_b64_tr_b16): the
// 16 lanes of a group supply the addresses of a 4 (s) x 16 (m) block as 8-byte
// pieces (lane j: row j / 4, columns 4 (j % 4) .. + 3) and lane i of the group
// receives column i of the 4 rows, i.e. 4 consecutive values of the contraction
// index for one output row, which is the operand layout of
// v_mfma_f32_32x32x16_bf16 (two such reads per 8-value fragment).
// LDS rows are 512 bytes; 16-byte chunk p of row s sits at p ^ ((s & 3) << 2).  A half-wave of
// such a read is two groups, i.e. 4 rows x 4 neighbouring chunks; with the row number XOR-ed
// into bits 2-3 of the chunk index those 16 pieces land in 16 different chunk positions of the
// 256-byte bank period: every bank once (XOR-ing bits 1-2 instead left half of the banks idle
// and showed as bank conflicts in 37 % of the LDS cycles).
// Loads go through buffer descriptors; a row past the end of the buffer, a
// padding item or a column past the matrix edge is turned into an out-of-range
// offset, for which the hardware returns zeros.  WIDE (an operand beyond the 4 GiB
// of a descriptor): plain 64-bit addresses, and such a load is skipped instead.
// Loads go through registers (the float32 rows are rounded there), two LDS stages, one
// barrier per slab of 32 buffer rows; split-K with one K range per XCD.
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;
constexpr int WK = 32;                       // buffer rows per slab
constexpr int WROWB = 512;                   // bytes per LDS row (256 bf16)
constexpr int WOPB = WK * WROWB;             // bytes per operand and stage
constexpr int WSTAGEB = 2 * WOPB;
constexpr size_t WSMEM = 2 * (size_t)WSTAGEB;
constexpr int kNonTemporal = 2;              // cache policy bits of a buffer store (nt)
constexpr int kWgradWaves = 8;

// 8 waves per block (128x64 each, two per SIMD).
// EXPORT: the end of a window also copies the buffer rows out in ascending-ID order
// (gram_flush); this kernel has every row of G in registers anyway, so it writes row s to
// G_total[rank_of_slot[s]] (rank_of_slot NULL: the buffer is in that order already) and the
// export kernel's second read of the buffer is saved.  The feature tiles that share a slab of G
// share its rows: tile f writes the rows t of a wave with t % f_tiles == f.
struct WgradExport {
    float* G_total;            // [rows held, d]
    const int* rank_of_slot;   // [rows held] or NULL
    // one-step windows: the last meta_blocks blocks of the grid export IDs and counts and clear the
    // slot map (what k_flush_meta does), so the end of such a window is two launches
    int meta_blocks;
    const long long* cnt_of_slot;
    int* slot_of;
    int* uniq_total;           // nullable
    int* counts_total;         // nullable
    int* u_total_dev;          // nullable
    int* scal;
};
// GB: the rows are bf16 already (what an earlier contraction stored rounded); only with WIDE, what a descriptor can
// address takes k_wgrad_rows_bf16.
template <bool WIDE = false, bool EXPORT = false, bool GB = false>
__global__ __launch_bounds__(kWgradWaves * 64) void k_wgrad_tn_bf16(
    const uint16_t* __restrict__ X, uint32_t x_bytes, const int* __restrict__ id_of_slot,
    const float* __restrict__ G, uint32_t g_bytes, const int* __restrict__ rows_dev, int d_in, int d,
    int pad_id, int splits, float* __restrict__ partial, int row_begin, int row_end, WgradExport ex)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    if (EXPORT && ex.meta_blocks > 0 && blockIdx.x >= gridDim.x - ex.meta_blocks) {
        const int n_ = *rows_dev;
        const int mb = blockIdx.x - (gridDim.x - ex.meta_blocks);
        for (int r = mb * (kWgradWaves * 64) + threadIdx.x; r < n_; r += ex.meta_blocks * (kWgradWaves * 64))
            flush_meta_row(r, id_of_slot, nullptr, ex.cnt_of_slot, ex.slot_of, ex.uniq_total, ex.counts_total, nullptr);
        if (mb == 0 && threadIdx.x == 0) {
            if (ex.u_total_dev) *ex.u_total_dev = n_;
            ex.scal[kSFlushN] = n_;
        }
        return;
    }
    const int tiles_c = (d + 255) / 256, tiles = ((d_in + 255) / 256) * tiles_c;
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int z = xcd + 8 * (q / tiles);
    const int i0 = ((q % tiles) / tiles_c) * 256, c0 = ((q % tiles) % tiles_c) * 256;
    if (z >= splits) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    static_assert(!GB || WIDE, "bf16 rows that a descriptor can address have a kernel of their own");
    constexpr int NT = 2;                        // 32-column MFMA tiles per wave
    constexpr int RW = WK / kWgradWaves;         // buffer rows of a slab this wave loads
    // two register sets for loads in flight: a load has two slabs of MFMAs to land (246 VGPRs
    // with 8 waves, so two waves per SIMD still fit)
    constexpr int SETS = 2;
    const int wm = wave >> 2, wn = wave & 3;

    // buffer rows [row_begin, U) take part (row_end clips U: the chunked call); slabs stay aligned
    // to multiples of WK rows, rows outside the range are loaded as zeros
    const int rows_held = *rows_dev;
    const int U = rows_held < row_end ? rows_held : row_end;
    const int sl0 = row_begin / WK;
    const int slabs_all = U > row_begin ? (U + WK - 1) / WK - sl0 : 0;
    const int per = (slabs_all + splits - 1) / splits;
    const int sl_begin = sl0 + z * per;
    int nslab = sl0 + slabs_all - sl_begin;
    if (nslab > per) nslab = per;
    partial += (int64_t)z * d_in * d;

    const __amdgpu_buffer_rsrc_t rsX = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(X), 0, x_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rsG = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(G), 0, g_bytes, kBufferFlags);

    // X loader: instruction t of wave w moves buffer rows RW w + 2 t and + 1 (lane / 32 picks the
    // row), lane % 32 = position of the 16-byte chunk in the LDS row
    const int a_row = wave * RW + (lane >> 5);                        // + 2 t
    const int a_pos = lane & 31;
    // G loader: instruction t of wave w moves buffer row RW w + t; lane l holds columns 4 l .. 4 l + 3
    const int g_col = c0 + 4 * lane;
    const bool g_col_ok = g_col < d;
    unsigned char* parkA = smem + (wave * RW) * WROWB + lane * 16;   // + t * 1024 (two rows per t)
    unsigned char* parkG = smem + WOPB + (wave * RW) * WROWB + (lane & 1) * 8;

    f32x16 acc[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // fragment addresses (see the header comment): group g = lane / 16, j = lane % 16
    const int j16 = lane & 15, grp = lane >> 4;
    const int f_row = (grp >> 1) * 8 + (j16 >> 2);                   // + 16 ks + 4 h
    const int f_x = ((j16 >> 2) & 3) << 2;
    // chunk index within the whole 512-byte row (the swizzle acts on it): the wave's quadrant starts
    // at chunk 16 wm (A) / NT 4 wn (B)
    int f_offA[4], f_offB[NT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        f_offA[i] = f_row * WROWB + (((wm * 16 + i * 4 + (grp & 1) * 2 + ((j16 & 3) >> 1)) ^ f_x) * 16) + (j16 & 1) * 8;
#pragma unroll
    for (int i = 0; i < NT; ++i)
        f_offB[i] = WOPB + f_row * WROWB +
                    (((wn * (NT * 4) + i * 4 + (grp & 1) * 2 + ((j16 & 3) >> 1)) ^ f_x) * 16) + (j16 & 1) * 8;

    bf16x8 fa[2][4], fb[2][NT];
    v4i32 ra[SETS][RW / 2], rg[SETS][GB ? RW / 2 : RW];
    // (EXPORT) rk[set]: lane t < RW holds the output row of the t-th buffer row of the slab in that
    // set, -1 if the row is not to be written; fetched BEFORE the slab's data loads (see below)
    int rk[EXPORT ? SETS : 1];
    bool ex_mine[RW];
    {
        const int f_tiles = (d_in + 255) / 256, f_idx = i0 / 256;
#pragma unroll
        for (int t = 0; t < RW; ++t) ex_mine[t] = EXPORT && (t % f_tiles) == f_idx;
    }
    // item IDs: ids_next receives the load for the slab after next, ids_cur holds the ones the next
    // data loads use.  The ID load is issued BEFORE the data loads of an iteration: memory operations
    // return in order, so waiting for an ID load that was issued after them would drain them all
    // and leave a single slab of loads in flight.
    int ids_next[RW / 2], ids_cur[RW / 2];

#define GRAM_TR(PTR) __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(PTR))
#define GRAM_FRAGS(FS, STAGE, KS)                                                                   \
    {                                                                                               \
        const unsigned char* sb_ = smem + (STAGE) * WSTAGEB + (KS) * 16 * WROWB;                    \
        _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                             \
            const v4i16 a0 = GRAM_TR(sb_ + f_offA[i]);                                       \
            const v4i16 a1 = GRAM_TR(sb_ + f_offA[i] + 4 * WROWB);                           \
            fa[FS][i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7)); \
        }                                                                                           \
        _Pragma("unroll") for (int i = 0; i < NT; ++i) {                                            \
            const v4i16 b0 = GRAM_TR(sb_ + f_offB[i]);                                       \
            const v4i16 b1 = GRAM_TR(sb_ + f_offB[i] + 4 * WROWB);                           \
            fb[FS][i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7)); \
        }                                                                                           \
    }
    // (Raising the wave priority around the fragment reads and MFMAs of a k-step paid while a
    // single slab of loads was in flight; with two it costs 4 %.)
#define GRAM_MMA(FS)                                                                                \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                   \
        _Pragma("unroll") for (int j = 0; j < NT; ++j)                                              \
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[FS][i], fb[FS][j], acc[i][j], 0, 0, 0);
    // item IDs of the X rows this lane will fetch for slab SLAB (clamped: a slab past the end is
    // loaded but never multiplied)
#define GRAM_IDS(SLAB)                                                                              \
    {                                                                                               \
        const int sb_ = (sl_begin + ((SLAB) < last ? (SLAB) : last)) * WK;                          \
        _Pragma("unroll") for (int t = 0; t < RW / 2; ++t) {                                        \
            const int slot = sb_ + a_row + 2 * t;                                                   \
            ids_next[t] = (slot < U && slot >= row_begin) ? (id_of_slot ? id_of_slot[slot] : slot) : pad_id; \
        }                                                                                           \
    }
#define GRAM_IDS_TAKE                                                                               \
    _Pragma("unroll") for (int t = 0; t < RW / 2; ++t) ids_cur[t] = ids_next[t];
#define GRAM_LOAD(SET, SLAB)                                                                        \
    {                                                                                               \
        const int sb_ = (sl_begin + ((SLAB) < last ? (SLAB) : last)) * WK;                          \
        if (EXPORT) {                                                                               \
            const int slot = sb_ + wave * RW + lane;                                                \
            const bool okr = lane < RW && slot < U && slot >= row_begin;                            \
            rk[(SET) % SETS] = okr ? (ex.rank_of_slot ? ex.rank_of_slot[slot] : slot) : -1;         \
        }                                                                                           \
        _Pragma("unroll") for (int t = 0; t < RW / 2; ++t) {                                        \
            const int kk = a_row + 2 * t;                                                           \
            const int feat = i0 + ((a_pos ^ ((kk & 3) << 2)) * 8);                                  \
            const int id = ids_cur[t];                                                              \
            const bool ok = id != pad_id && feat < d_in && sb_ + kk < U && sb_ + kk >= row_begin;   \
            if (WIDE) {                                                                             \
                v4i32 v_ = {0, 0, 0, 0};                                                            \
                if (ok) v_ = *reinterpret_cast<const v4i32*>(X + (int64_t)id * d_in + feat);        \
                ra[(SET) % SETS][t] = v_;                                                           \
            } else {                                                                                \
                const uint32_t off = ok ? (uint32_t)(((int64_t)id * d_in + feat) * 2) : kOutOfRange; \
                ra[(SET) % SETS][t] = __builtin_amdgcn_raw_buffer_load_b128(rsX, off, 0, 0);        \
            }                                                                                       \
        }                                                                                           \
        if (GB) _Pragma("unroll") for (int t = 0; t < RW / 2; ++t) {                                \
            const int slot = sb_ + a_row + 2 * t;                                                   \
            const int col = c0 + ((a_pos ^ ((slot & 3) << 2)) * 8);                                 \
            const bool okg = col < d && slot < U && slot >= row_begin;                              \
            v4i32 v_ = {0, 0, 0, 0};                                                                \
            if (okg) v_ = *reinterpret_cast<const v4i32*>(reinterpret_cast<const uint16_t*>(G) + (int64_t)slot * d + col); \
            rg[(SET) % SETS][t] = v_;                                                               \
        }                                                                                           \
        if (!GB) _Pragma("unroll") for (int t = 0; t < RW; ++t) {                                   \
            const int slot = sb_ + wave * RW + t;                                                    \
            const bool okg = g_col_ok && slot < U && slot >= row_begin;                             \
            if (WIDE) {                                                                             \
                v4i32 v_ = {0, 0, 0, 0};                                                            \
                if (okg) v_ = *reinterpret_cast<const v4i32*>(G + (int64_t)slot * d + g_col);       \
                rg[(SET) % SETS][t] = v_;                                                           \
            } else {                                                                                \
                const uint32_t off = okg ? (uint32_t)(((int64_t)slot * d + g_col) * 4) : kOutOfRange; \
                rg[(SET) % SETS][t] = __builtin_amdgcn_raw_buffer_load_b128(rsG, off, 0, 0);        \
            }                                                                                       \
        }                                                                                           \
    }
#define GRAM_PARK(SET, STAGE)                                                                       \
    {                                                                                               \
        unsigned char* pa_ = parkA + (STAGE) * WSTAGEB;                                             \
        unsigned char* pg_ = parkG + (STAGE) * WSTAGEB;                                             \
        _Pragma("unroll") for (int t = 0; t < RW / 2; ++t)                                          \
            *reinterpret_cast<v4i32*>(pa_ + t * 1024) = ra[(SET) % SETS][t];                                 \
        if (GB) _Pragma("unroll") for (int t = 0; t < RW / 2; ++t)                                  \
            *reinterpret_cast<v4i32*>(pa_ + WOPB + t * 1024) = rg[(SET) % SETS][t];                 \
        if (!GB) _Pragma("unroll") for (int t = 0; t < RW; ++t) {                                   \
            const v4i32 v = rg[(SET) % SETS][t];                                                             \
            const uint32_t lo = pack_bf16x2(__int_as_float(v.x), __int_as_float(v.y));              \
            const uint32_t hi = pack_bf16x2(__int_as_float(v.z), __int_as_float(v.w));              \
            const int pos = (lane >> 1) ^ ((t & 3) << 2);        /* row RW w + t: (row & 3) == (t & 3) */ \
            *reinterpret_cast<uint2*>(pg_ + t * WROWB + pos * 16) = make_uint2(lo, hi);             \
            if (EXPORT && ex_mine[t]) {                                                             \
                const int r_ = __builtin_amdgcn_readlane(rk[(SET) % SETS], t);                      \
                if (r_ >= 0 && g_col_ok)                                                            \
                    __builtin_nontemporal_store(v, reinterpret_cast<v4i32*>(ex.G_total + (int64_t)r_ * d + g_col)); \
            }                                                                                       \
        }                                                                                           \
    }
    // (fixed interleaving patterns measured slower here than the compiler's own order)
#define GRAM_ITER(SL, P)                                                                            \
    {                                                                                               \
        GRAM_FRAGS(1, (SL) & 1, 1)                                                                  \
        GRAM_MMA(0)                                                                                 \
        GRAM_PARK(P, ((SL) + 1) & 1)                                                                \
        __syncthreads();                                                                            \
        GRAM_IDS_TAKE                                                                               \
        GRAM_IDS((SL) + 2 + SETS)                                                                   \
        GRAM_LOAD(P, (SL) + 1 + SETS)                                                               \
        GRAM_FRAGS(0, ((SL) + 1) & 1, 0)                                                            \
        GRAM_MMA(1)                                                                                 \
    }

    if (nslab > 0) {
        const int last = nslab - 1;
        GRAM_IDS(0)
        GRAM_IDS_TAKE
        GRAM_IDS(1)
        GRAM_LOAD(0, 0)
        GRAM_IDS_TAKE
        GRAM_IDS(2)
        GRAM_LOAD(1, 1)
        GRAM_PARK(0, 0)
        GRAM_IDS_TAKE
        GRAM_IDS(SETS + 1)
        GRAM_LOAD(0, SETS)
        __syncthreads();
        GRAM_FRAGS(0, 0, 0)
        int sl = 0;
        for (; sl + 1 < last; sl += 2) {
            GRAM_ITER(sl, 1)          // set 1 holds slab sl+1, set 0 holds slab sl+2
            GRAM_ITER(sl + 1, 0)
        }
        if (sl < last) GRAM_ITER(sl, 1)
        GRAM_FRAGS(1, last & 1, 1)
        GRAM_MMA(0)
        GRAM_MMA(1)
    }

    // accumulator element r of a lane sits at (row, col) = ((r / 4) * 8 + (lane / 32) * 4 + r % 4, lane % 32)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int fi = i0 + wm * 128 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (fi < d_in) {
                float* row = partial + (int64_t)fi * d + c0 + wn * (NT * 32) + (lane & 31);
#pragma unroll
                for (int jj = 0; jj < NT; ++jj)
                    if (c0 + wn * (NT * 32) + jj * 32 + (lane & 31) < d) row[jj * 32] = acc[i][jj][r];
            }
        }
}
#undef GRAM_TR
#undef GRAM_FRAGS
#undef GRAM_MMA
#undef GRAM_IDS
#undef GRAM_IDS_TAKE
#undef GRAM_LOAD
#undef GRAM_PARK
#undef GRAM_ITER

// ---- weight gradient of rows that are bf16 already -----------------------------------------
//
// Both operands (features through the row list, rows as an earlier contraction stored them) can go straight to LDS, so the loop
// is the forward's (see k_gemm_nt_bf16): slabs of 32 rows of 512 bytes in a ring of four stages of 32 KiB, two segments per
// slab (read the fragments and request the slab three ahead; multiply), the lower half of the features a segment behind.  The
// row list goes through LDS too, 8 slabs' entries at a time: a load into registers would have to be waited for in the queue of
// the others (scalar loads: 123 us where the list is the identity 82).
// Padding, rows past the range and features or columns past the edge are offsets out of range, which write zeros to LDS.
// 32,768 rows, 1024 x 1024, without the reduction: 85 us through registers with one barrier per slab, now 76 (identity) and 80
// (listed); 13 of it are the partials (64 MiB written).  The same two segments with loads through registers: 92 us, the wait
// for them then stands between the other waves and the matrix pipe.
constexpr int PSTAGEB = 2 * WOPB, PSTAGES = 4, kPairLds = PSTAGES * PSTAGEB + 4096;

template <bool LISTED>
__global__ __launch_bounds__(kWgradWaves * 64) void k_wgrad_rows_bf16(
    const uint16_t* __restrict__ X, uint32_t x_bytes, const int* __restrict__ row_list, const uint16_t* __restrict__ G,
    uint32_t g_bytes, const int* __restrict__ rows_dev, int d_in, int d, int pad_id, int splits,
    float* __restrict__ partial, int row_begin, int row_end)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tiles_c = (d + 255) / 256, tiles = ((d_in + 255) / 256) * tiles_c;
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int z = xcd + 8 * (q / tiles);
    const int i0 = ((q % tiles) / tiles_c) * 256, c0 = ((q % tiles) % tiles_c) * 256;
    if (z >= splits) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    // rows [row_begin, U), slabs aligned to multiples of WK rows, a contiguous range of them per block
    const int rows_held = *rows_dev;
    const int U = rows_held < row_end ? rows_held : row_end;
    const int sl0 = row_begin / WK;
    const int slabs_all = U > row_begin ? (U + WK - 1) / WK - sl0 : 0;
    const int per = (slabs_all + splits - 1) / splits;
    const int sl_begin = sl0 + z * per;
    int nslab = sl0 + slabs_all - sl_begin;
    if (nslab > per) nslab = per;
    partial += (int64_t)z * d_in * d;

    const u32x4 rsX = buffer_words(X, x_bytes), rsG = buffer_words(G, g_bytes);
    // wave w moves rows 4 w + 2 t + lane / 32 of a slab, t = 0, 1, of either operand
    uint32_t xo[2], go[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int chunk = (lane & 31) ^ ((2 * t + (lane >> 5)) << 2);
        xo[t] = i0 + chunk * 8 < d_in ? (uint32_t)(i0 + chunk * 8) * 2u : kOutOfRange;
        go[t] = c0 + chunk * 8 < d ? (uint32_t)(c0 + chunk * 8) * 2u : kOutOfRange;
    }
    typedef __attribute__((address_space(3))) unsigned char lds_u8;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem, to_w = lds0 + wave * 2048;
    // entries of the list: ring of 4 pieces of 256, piece k holds those of slabs 8 k .. 8 k + 7 of the block's range
    // (its descriptor ends with a whole load of 4 entries, so that no load is partly out of range: the list has the room)
    const u32x4 rsI = buffer_words(row_list, LISTED ? ((uint32_t)row_end + 3u & ~3u) * 4u : 0u);
    const uint32_t list0 = lds0 + PSTAGES * PSTAGEB, list_l = list0 + (uint32_t)(wave * 4 + (lane >> 5)) * 4u;
    typedef const __attribute__((address_space(3))) int lds_i32;
#define GRAM_IDS(PIECE)                                                                             \
    load_to_lds(rsI, (uint32_t)(sl_begin * WK + (PIECE) * 256 + lane * 4) * 4u, 0u, list0 + ((PIECE) & 3) * 1024);
#define GRAM_LOAD(SL)                                                                               \
    {                                                                                               \
        const uint32_t to_ = to_w + ((SL) & (PSTAGES - 1)) * PSTAGEB;                               \
        const int slot0_ = (sl_begin + (SL)) * WK + wave * 4 + (lane >> 5);                         \
        _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                             \
            const int slot_ = slot0_ + 2 * t;                                                       \
            const bool held_ = (SL) < nslab && slot_ < U && slot_ >= row_begin;                     \
            const int id_ = LISTED ? *(lds_i32*)(uintptr_t)(list_l + ((uint32_t)(SL) & 31u) * (WK * 4) + t * 8) : slot_; \
            const uint32_t xr_ = held_ && id_ != pad_id ? (uint32_t)id_ * (uint32_t)(d_in * 2) : kOutOfRange; \
            const uint32_t gr_ = held_ ? (uint32_t)slot_ * (uint32_t)(d * 2) : kOutOfRange;         \
            load_to_lds(rsX, __builtin_elementwise_add_sat(xr_, xo[t]), 0u, to_ + t * 1024);        \
            load_to_lds(rsG, __builtin_elementwise_add_sat(gr_, go[t]), 0u, to_ + WOPB + t * 1024); \
        }                                                                                           \
    }

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int j16 = lane & 15, grp = lane >> 4;
    const int f_row = (grp >> 1) * 8 + (j16 >> 2), f_x = (j16 >> 2 & 3) << 2;
    uint32_t ra[4], rb[2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        ra[i] = lds0 + f_row * WROWB + (((wm * 16 + i * 4 + (grp & 1) * 2 + ((j16 & 3) >> 1)) ^ f_x) * 16) + (j16 & 1) * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j)
        rb[j] = lds0 + WOPB + f_row * WROWB + (((wn * 8 + j * 4 + (grp & 1) * 2 + ((j16 & 3) >> 1)) ^ f_x) * 16) + (j16 & 1) * 8;
    bf16x8 fa[2][4], fb[2][2];
    auto frag = [](uint32_t at) {
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(uintptr_t)at);
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(uintptr_t)(at + 4 * WROWB));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    if (nslab > 0) {
        constexpr int kAhead = 2 * 4;        // loads that may be in flight when a slab is published: the next two slabs'
        if (LISTED) {
            if (wave == 0) {
                GRAM_IDS(0)
                GRAM_IDS(1)
            }
            wait_loads<0>();
            segment_barrier();
        }
        GRAM_LOAD(0)
        GRAM_LOAD(1)
        GRAM_LOAD(2)
        wait_loads<kAhead>();
        segment_barrier();
        if (wm == 1) segment_barrier();
        for (int sl = 0; sl < nslab; ++sl) {
            const uint32_t stage = (uint32_t)(sl & (PSTAGES - 1)) * PSTAGEB;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[ks][j] = frag(rb[j] + stage + ks * (16 * WROWB));
#pragma unroll
                for (int i = 0; i < 4; ++i) fa[ks][i] = frag(ra[i] + stage + ks * (16 * WROWB));
            }
            __builtin_amdgcn_sched_barrier(0);
            // (the piece after next: first read 13 slabs on, what it replaces was last read 12 slabs ago)
            if (LISTED && wave == 0 && (sl & 7) == 0) { GRAM_IDS((sl >> 3) + 2) }
            GRAM_LOAD(sl + 3)
            wait_loads<kAhead>();
            wait_lds();
            segment_barrier();
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
            segment_barrier();
        }
        if (wm == 0) segment_barrier();
        wait_loads<0>();
    }
#undef GRAM_IDS
#undef GRAM_LOAD
    // accumulator element r of a lane sits at (row, col) = ((r / 4) * 8 + (lane / 32) * 4 + r % 4, lane % 32)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int fi = i0 + wm * 128 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (fi < d_in) {
                float* row = partial + (int64_t)fi * d + c0 + wn * 64 + (lane & 31);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (c0 + wn * 64 + j * 32 + (lane & 31) < d) row[j * 32] = acc[i][j][r];
            }
        }
}

// ---- weight gradient of short windows -------------------------------------------------
//
// A window of a few thousand buffer rows over a 768 x 256 matrix is 1 GFLOP: nothing but latency.  The
// kernel above gives it 24 blocks of 256 x 256 with ten slabs each, one after the other (14 us, 21 with
// the reduction, at 2,500 rows; this one with its reduction 12).  This one cuts the output into 128 x 64 tiles and the rows twice: over blocks (partials
// through memory, as above) and inside a block over four groups of four waves, which walk different
// slabs side by side and add their tiles through LDS at the end.  16 waves per CU with the loads of
// three slabs each in flight is also what it takes to draw on L2 at 47 instead of 19 B/clk.  Slab i of
// group g of range z is slab (4 z + g) + 4 S i: which rows a wave starts with does not depend on the row
// count, so its first loads go out with the load of that count; rows past it are zeroed on their way
// into LDS (offsets that leave a matrix return zeros).
// LDS rows of X are 256 bytes (chunk c of row r at c ^ ((r & 3) << 2)), rows of G 128 bytes (chunk c at
// c ^ ((r & 2) << 1)): either way the 16 pieces of a transposing read cover every bank once.
constexpr int VM = 128, VN = 64, VGROUPS = 4, VTHREADS = VGROUPS * 256, VDEPTH = 2;
constexpr int VXB = 32 * VM * 2, VSTAGEB = VXB + 32 * VN * 2;      // bytes per group and stage
constexpr int VACC_STRIDE = VN + 8;                                 // floats per row of a parked tile
constexpr size_t VSMEM = (size_t)VGROUPS * VM * VACC_STRIDE * 4;
static_assert(VSMEM >= 2 * (size_t)VGROUPS * VSTAGEB, "the tiles overlay the stages");

// LISTED: the items of the rows are listed (else row r pairs with item r).  GB: the rows are bf16 already.
template <bool EXPORT, bool LISTED, bool GB = false>
__global__ __launch_bounds__(VTHREADS) void k_wgrad_short(
    const uint16_t* __restrict__ X, uint32_t x_bytes, const int* __restrict__ id_of_slot,
    const float* __restrict__ G, uint32_t g_bytes, const int* __restrict__ rows_dev, int d_in, int d,
    int pad_id, int splits, float* __restrict__ partial, int row_begin, int row_end, int accumulate, WgradExport ex)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    if (EXPORT && ex.meta_blocks > 0 && blockIdx.x >= gridDim.x - ex.meta_blocks) {
        const int n_ = *rows_dev;
        const int mb = blockIdx.x - (gridDim.x - ex.meta_blocks);
        for (int r = mb * VTHREADS + threadIdx.x; r < n_; r += ex.meta_blocks * VTHREADS)
            flush_meta_row(r, id_of_slot, nullptr, ex.cnt_of_slot, ex.slot_of, ex.uniq_total, ex.counts_total, nullptr);
        if (mb == 0 && threadIdx.x == 0) {
            if (ex.u_total_dev) *ex.u_total_dev = n_;
            ex.scal[kSFlushN] = n_;
        }
        return;
    }
    // the tiles of one range of rows run on one XCD (or, with fewer than 8 ranges, on 8 / splits of them)
    // and share the rows through its L2
    const int tiles_c = (d + VN - 1) / VN, f_tiles = (d_in + VM - 1) / VM, tiles = f_tiles * tiles_c;
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int z = splits >= 8 ? xcd + 8 * (q / tiles) : xcd % splits;
    const int tile = splits >= 8 ? q % tiles : q * (8 / splits) + xcd / splits;
    const int f_idx = tile / tiles_c;
    const int i0 = f_idx * VM, c0 = (tile % tiles_c) * VN;
    if (z >= splits || tile >= tiles) return;
    const int tid = threadIdx.x, grp = __builtin_amdgcn_readfirstlane(tid >> 8), gt = tid & 255;
    const int lane = tid & 63, wave = (tid >> 6) & 3;
    const int wm = wave >> 1, wn = wave & 1;

    const __amdgpu_buffer_rsrc_t rsX = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(X), 0, x_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rsG = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(G), 0, g_bytes, kBufferFlags);

    // loader: thread gt of a group moves chunk gt & 15 of rows gt >> 4 and (gt >> 4) + 16 of a slab, of
    // X (16 bytes of bf16) and of G (4 floats)
    const int lrow = gt >> 4, lpos = gt & 15;
    const int feat = i0 + ((lpos ^ ((lrow & 3) << 2)) * 8);         // rows lrow and lrow + 16 swizzle alike
    const bool feat_ok = feat < d_in;
    const int g_col = c0 + 4 * lpos;
    const bool g_col_ok = g_col < d;
    // (GB: one 16-byte chunk per thread, chunk gt & 7 of row gt >> 3)
    const int brow = gt >> 3, bcol = c0 + (((gt & 7) ^ ((brow & 2) << 1)) * 8);
    const int first = row_begin / WK + z * VGROUPS + grp, stride = splits * VGROUPS;
    bool ex_mine[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) ex_mine[t] = EXPORT && (lrow + 16 * t) % f_tiles == f_idx;

    // row_end bounds the rows as allocated: what lies between the rows held and row_end is loaded and
    // dropped.  Nothing in the loop is conditional (offsets out of range read zeros and store nothing),
    // so that the loads in flight are known at every wait.
    const __amdgpu_buffer_rsrc_t rsI = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(id_of_slot), 0, LISTED ? row_end * 4 : 0, kBufferFlags);
    const bool ranked = EXPORT && ex.rank_of_slot;
    const __amdgpu_buffer_rsrc_t rsR = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(ex.rank_of_slot), 0, ranked ? row_end * 4 : 0, kBufferFlags);
    const __amdgpu_buffer_rsrc_t rsT = __builtin_amdgcn_make_buffer_rsrc(ex.G_total, 0, EXPORT ? g_bytes : 0, kBufferFlags);
    int ids_next[VDEPTH][2], ids_cur[2], rk[VDEPTH][2];
    v4i32 rx[VDEPTH][2], rg[VDEPTH][GB ? 1 : 2];
#define GRAM_SLOT(IT, T_) (((first + (IT) * stride) * WK) + lrow + 16 * (T_))
#define GRAM_IDS(SET, IT)                                                                           \
    _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                                 \
        const int slot = GRAM_SLOT(IT, t);                                                          \
        ids_next[SET][t] = LISTED ? __builtin_amdgcn_raw_buffer_load_b32(rsI, slot < row_end ? (uint32_t)slot * 4u : kOutOfRange, 0, 0) : slot; \
    }
#define GRAM_LOAD(SET, IT)                                                                          \
    _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                                 \
        const int slot = GRAM_SLOT(IT, t);                                                          \
        const bool in_ = slot < row_end;                                                            \
        if (EXPORT) rk[SET][t] = __builtin_amdgcn_raw_buffer_load_b32(rsR, in_ ? (uint32_t)slot * 4u : kOutOfRange, 0, 0); \
        const uint32_t ox = in_ && feat_ok && ids_cur[t] != pad_id ? ((uint32_t)ids_cur[t] * (uint32_t)d_in + (uint32_t)feat) * 2u : kOutOfRange; \
        rx[SET][t] = __builtin_amdgcn_raw_buffer_load_b128(rsX, ox, 0, 0);                          \
        if (!GB) {                                                                                  \
            const uint32_t og = in_ && g_col_ok ? ((uint32_t)slot * (uint32_t)d + (uint32_t)g_col) * 4u : kOutOfRange; \
            rg[SET][t % (GB ? 1 : 2)] = __builtin_amdgcn_raw_buffer_load_b128(rsG, og, 0, 0);       \
        }                                                                                           \
    }                                                                                               \
    if (GB) {                                                                                       \
        const int slot = (first + (IT) * stride) * WK + brow;                                       \
        const uint32_t og = slot < row_end && bcol < d ? ((uint32_t)slot * (uint32_t)d + (uint32_t)bcol) * 2u : kOutOfRange; \
        rg[SET][0] = __builtin_amdgcn_raw_buffer_load_b128(rsG, og, 0, 0);                          \
    }
#define GRAM_PARK(SET, IT, STAGE)                                                                   \
    {                                                                                               \
        unsigned char* s_ = smem + ((STAGE) * VGROUPS + grp) * VSTAGEB;                             \
        _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                             \
            const int row = lrow + 16 * t, slot = GRAM_SLOT(IT, t);                                 \
            const bool held = slot < U && slot >= row_begin;                                        \
            const v4i32 zero_ = {0, 0, 0, 0};                                                       \
            *reinterpret_cast<v4i32*>(s_ + row * (VM * 2) + lpos * 16) = held ? rx[SET][t] : zero_; \
            if (GB) continue;                                                                       \
            const v4i32 v = held ? rg[SET][t % (GB ? 1 : 2)] : zero_;                               \
            const uint32_t lo = pack_bf16x2(__int_as_float(v.x), __int_as_float(v.y));              \
            const uint32_t hi = pack_bf16x2(__int_as_float(v.z), __int_as_float(v.w));              \
            *reinterpret_cast<uint2*>(s_ + VXB + row * (VN * 2) + (((lpos >> 1) ^ ((row & 2) << 1)) * 16) + (lpos & 1) * 8) = \
                make_uint2(lo, hi);                                                                 \
            if (EXPORT) {                                                                           \
                const uint32_t to = held && ex_mine[t] && g_col_ok                                  \
                                        ? ((uint32_t)(ranked ? rk[SET][t] : slot) * (uint32_t)d + (uint32_t)g_col) * 4u : kOutOfRange; \
                __builtin_amdgcn_raw_buffer_store_b128(v, rsT, to, 0, kNonTemporal);                \
            }                                                                                       \
        }                                                                                           \
        if (GB) {                                                                                   \
            const int slot = (first + (IT) * stride) * WK + brow;                                   \
            const v4i32 zero_ = {0, 0, 0, 0};                                                       \
            *reinterpret_cast<v4i32*>(s_ + VXB + brow * (VN * 2) + (gt & 7) * 16) = slot < U && slot >= row_begin ? rg[SET][0] : zero_; \
        }                                                                                           \
    }
#define GRAM_IDS_TAKE(SET) ids_cur[0] = ids_next[SET][0]; ids_cur[1] = ids_next[SET][1];
    // The IDs of the first slabs, then the row count, then the slabs.  Memory operations return in
    // order: the IDs of a slab are fetched two slabs before its data and ahead of them, so that waiting
    // for them leaves the data of the slabs in between in flight.
    GRAM_IDS(0, 0)
    GRAM_IDS(1, 1)
    const int rows_held = *rows_dev;
    GRAM_IDS_TAKE(0)
    GRAM_IDS(0, 2)
    GRAM_LOAD(0, 0)
    GRAM_IDS_TAKE(1)
    GRAM_IDS(1, 3)
    GRAM_LOAD(1, 1)
    const int U = rows_held < row_end ? rows_held : row_end;
    // slabs that hold rows: the trip count of the block's first group, which has the most
    const int slabs_end = (U + WK - 1) / WK;
    const int lead = row_begin / WK + z * VGROUPS;
    const int iters = slabs_end > lead ? (slabs_end - lead + stride - 1) / stride : 0;

    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    // fragment addresses (see k_wgrad_tn_bf16)
    const int j16 = lane & 15, g16 = lane >> 4;
    const int f_row = (g16 >> 1) * 8 + (j16 >> 2), f_ch = (g16 & 1) * 2 + ((j16 & 3) >> 1), f_b = (j16 & 1) * 8;
    int f_offA[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) f_offA[i] = f_row * (VM * 2) + (((wm * 8 + i * 4 + f_ch) ^ ((f_row & 3) << 2)) * 16) + f_b;
    const int f_offB = VXB + f_row * (VN * 2) + (((wn * 4 + f_ch) ^ ((f_row & 2) << 1)) * 16) + f_b;
#define GRAM_TR(PTR) __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(PTR))
#define GRAM_FRAG(P_, ROWB)                                                                         \
    __builtin_bit_cast(bf16x8, __builtin_shufflevector(GRAM_TR(P_), GRAM_TR((P_) + 4 * (ROWB)), 0, 1, 2, 3, 4, 5, 6, 7))
#define GRAM_MULTIPLY(STAGE)                                                                        \
    {                                                                                               \
        const unsigned char* s_ = smem + ((STAGE) * VGROUPS + grp) * VSTAGEB;                       \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {                                          \
            const bf16x8 fb = GRAM_FRAG(s_ + f_offB + ks * 16 * (VN * 2), VN * 2);                  \
            _Pragma("unroll") for (int i = 0; i < 2; ++i) {                                         \
                const bf16x8 fa = GRAM_FRAG(s_ + f_offA[i] + ks * 16 * (VM * 2), VM * 2);           \
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[i], 0, 0, 0);          \
            }                                                                                       \
        }                                                                                           \
    }
    // slab i sits in register set and LDS stage i % 2, one barrier per slab; a slab past the end parks
    // zeros
#define GRAM_ITER(I)                                                                                \
    GRAM_PARK(I, i + (I), I)                                                                        \
    GRAM_IDS_TAKE(I)                                                                                \
    GRAM_IDS(I, i + (I) + 4)                                                                        \
    GRAM_LOAD(I, i + (I) + 2)                                                                       \
    __syncthreads();                                                                                \
    GRAM_MULTIPLY(I)
    static_assert(VDEPTH == 2, "the set indices of the loop");
    for (int i = 0; i < iters; i += 2) {
        GRAM_ITER(0)
        GRAM_ITER(1)
    }
    // the groups' tiles are parked in LDS and added in group order
    __syncthreads();
    float* parked = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            parked[(grp * VM + wm * 64 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)) * VACC_STRIDE + wn * 32 + (lane & 31)] =
                acc[i][r];
    __syncthreads();
    partial += (int64_t)z * d_in * d;
#pragma unroll
    for (int h = 0; h < VM * VN / 4 / VTHREADS; ++h) {
        const int e = tid + h * VTHREADS, row = e / (VN / 4), c4 = e % (VN / 4) * 4;
        f32x4 s = *reinterpret_cast<const f32x4*>(&parked[row * VACC_STRIDE + c4]);
#pragma unroll
        for (int g = 1; g < VGROUPS; ++g) s += *reinterpret_cast<const f32x4*>(&parked[(g * VM + row) * VACC_STRIDE + c4]);
        if (i0 + row < d_in && c0 + c4 < d) {
            f32x4* out = reinterpret_cast<f32x4*>(partial + (int64_t)(i0 + row) * d + c0 + c4);
            *out = accumulate ? *out + s : s;
        }
    }
}
#undef GRAM_SLOT
#undef GRAM_IDS
#undef GRAM_IDS_TAKE
#undef GRAM_LOAD
#undef GRAM_PARK
#undef GRAM_TR
#undef GRAM_FRAG
#undef GRAM_MULTIPLY
#undef GRAM_ITER

__device__ __forceinline__ void split_range(int u_total, int splits, int z, int* kb, int* ke)
{
    const int chunk = (u_total + splits - 1) / splits;
    const int b = z * chunk;
    int e = b + chunk;
    if (e > u_total) e = u_total;
    *kb = b < u_total ? b : u_total;
    *ke = e < *kb ? *kb : e;
}

__global__ __launch_bounds__(kBlock) void k_wgrad_f32(
    const float* __restrict__ X, const int* __restrict__ id_of_slot, const float* __restrict__ G,
    const int* __restrict__ rows_dev, int d_in, int d, int pad_id, int splits,
    float* __restrict__ partial, int row_begin, int row_end, int accumulate)
{
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    // (i is the same in all lanes of a wave, but the wave's loads of X stay vector loads: as scalar ones, 16 rows ahead,
    // they thrash the scalar cache: 400 rows of 768 x 256 46.5 us, 38.0 like this, 40.0 a row at a time)
    const int i = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int z = blockIdx.z;
    if (i >= d_in || c >= d) return;
    int kb, ke;
    const int rows_held = *rows_dev;
    const int u_end = rows_held < row_end ? rows_held : row_end;
    split_range(u_end > row_begin ? u_end - row_begin : 0, splits, z, &kb, &ke);
    kb += row_begin;
    ke += row_begin;
    float acc = 0.f;
    int sidx = kb;
    for (; sidx + 16 <= ke; sidx += 16) {       // sixteen rows' IDs, then their operands, requested together
        int id[16];
        float xv[16], gv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) id[u] = id_of_slot ? id_of_slot[sidx + u] : sidx + u;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            xv[u] = X[(int64_t)id[u] * d_in + i];
            gv[u] = G[(int64_t)(sidx + u) * d + c];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (id[u] != pad_id) acc = fmaf(xv[u], gv[u], acc);
    }
    for (; sidx < ke; ++sidx) {
        const int id = id_of_slot ? id_of_slot[sidx] : sidx;
        if (id != pad_id) acc = fmaf(X[(int64_t)id * d_in + i], G[(int64_t)sidx * d + c], acc);
    }
    float* out = partial + ((int64_t)z * d_in + i) * d + c;
    *out = accumulate ? *out + acc : acc;
}

__global__ __launch_bounds__(kBlock) void k_wgrad_reduce(const float4* __restrict__ partial,
                                                         int64_t n4, int splits,
                                                         float4* __restrict__ dW, int accumulate, LossSum loss)
{
    if (loss.out && blockIdx.x == gridDim.x - 1) {       // (one more block: the pseudo-loss, a launch less)
        half_sum_of(loss.part, loss.parts, loss.out);
        return;
    }
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= n4) return;
    float4 acc = accumulate ? dW[e] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int z = 0; z < splits; ++z) {
        const float4 v = partial[(int64_t)z * n4 + e];
        acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    dW[e] = acc;
}

int wgrad_splits_for(const gram_config& cfg)
{
    return wgrad_splits_dims(cfg.d_in, cfg.d, cfg.xw_dtype == GRAM_BF16);
}

int wgrad_splits_dims(int d_in, int d, bool bf16)
{
    if (!bf16) return 4;
    const int tiles = ((d_in + TM - 1) / TM) * ((d + TN - 1) / TN);
    int s = 256 / tiles / 8 * 8;      // one block per CU; a multiple of 8 (one K range per XCD)
    if (s < 8) s = 8;
    if (s > 64) s = 64;
    return s;
}

bool encoder_wgrad(Ctx* c, const void* X, float* dW, hipStream_t s, int64_t first_row, int64_t n_rows,
                   bool accumulate, const WgradRows* other, float* export_G, const int* rank_of_slot,
                   const WindowMeta* meta, const LossSum* loss)
{
    bool exported = false, direct = false;
    const int d_in = other && other->d_in ? other->d_in : c->cfg.d_in;
    const int d = other && other->d ? other->d : c->cfg.d;
    const int64_t x_rows = other && other->x_rows ? other->x_rows : c->cfg.vocab_n;
    const int pad_id = other && other->d_in ? other->pad_id : c->cfg.pad_id;
    int S = other && other->d_in ? wgrad_splits_dims(d_in, d, c->cfg.xw_dtype == GRAM_BF16) : c->wg_splits;
    // the rows contracted over: the persistent buffer (id_of_slot is NULL for the dense layout:
    // the item of row r is r), or the caller's (ids, rows) pairs
    const int64_t cap = other ? other->n_max : c->cap_total;
    const int* ids = other ? other->ids : c->id_of_slot;
    const float* rows = other ? other->rows : c->G;
    const int* rows_dev = other ? other->n_dev : c->scal + kSUTotal;
    const int row_begin = (int)(first_row < cap ? first_row : cap);
    const int row_end = (int)(n_rows < cap - row_begin ? row_begin + n_rows : cap);
    if (c->cfg.xw_dtype == GRAM_BF16) {
        // a short window does not need all the ranges: at least 8 slabs of 32 buffer rows each
        // (from the host's bound on the rows in the buffer), still a multiple of 8
        int64_t rows_bound = (other || c->dense) ? cap : (c->window_positions < cap ? c->window_positions : cap);
        if (rows_bound > row_end - row_begin) rows_bound = row_end - row_begin;
        const int64_t slabs_bound = rows_bound / WK + 1;
        int64_t want = slabs_bound / 8 / 8 * 8;
        if (want < 8) want = 8;
        if (want < S) S = (int)want;
        const bool gb = other && other->rows_bf16;
        const int64_t x_bytes = x_rows * d_in * 2, g_bytes = cap * d * (gb ? 2 : 4);
        const int tiles = ((d_in + 255) / 256) * ((d + 255) / 256);
        const WgradExport no_export = {nullptr, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
        const bool wide = x_bytes >= kBufferWindow || g_bytes >= kBufferWindow;
        const bool exporting = !wide && export_G && !other;
        int short_blocks = 0;
        const int short_tiles = ((d_in + VM - 1) / VM) * ((d + VN - 1) / VN);
        // Short windows: rows times tiles is the traffic from L2, which is what the short kernel is slower
        // at.  Kernel and reduction, short against long: 768 x 256 (24 tiles) 12.4 / 20.8 us at 2,500 rows,
        // 27.4 / 30.6 at 20,000, 45 / 40 at 40,000; 512 x 512 (32) 29.6 / 35.6 at 20,000, 48.9 / 46.6 at
        // 40,000.  With more than 32 tiles there are fewer than 8 ranges and the line lies lower: 768 x 400
        // (42) 30.4 / 31.2 at 12,000; 776 x 392 (49) 32.7 / 30.3 at 12,000, 22.9 / 25.7 at 6,400.
        const bool is_short = !wide && rows_bound * short_tiles <= (short_tiles <= 32 ? 650000 : 450000);
        if (is_short) {
            // ranges of rows: about a block per CU; a handful of slabs is one range, whose tiles go
            // straight to dW (300 rows: 8.4 us against 10.0; at 1,000 the reduction launch pays)
            int64_t ranges = c->num_cus / short_tiles;
            if (ranges > slabs_bound / VGROUPS) ranges = slabs_bound / VGROUPS;
            if (slabs_bound <= 20) ranges = 1;
            const int most = wgrad_splits_dims(d_in, d, true);      // what the partials have room for
            if (ranges > most) ranges = most;
            S = (int)(ranges >= 8 ? ranges / 8 * 8 : ranges >= 4 ? 4 : ranges >= 2 ? 2 : 1);
            short_blocks = S >= 8 ? short_tiles * S : (short_tiles * S + 7) / 8 * 8;
        }
        direct = is_short && S == 1;
        float* out = direct ? dW : c->wg_partial;
        const int add_here = direct && accumulate ? 1 : 0;
        const int waves_threads = is_short ? VTHREADS : kWgradWaves * 64;
        if (exporting) {
            WgradExport ex = no_export;
            ex.G_total = export_G;
            ex.rank_of_slot = rank_of_slot;
            if (meta) {
                int64_t mb = (rows_bound + waves_threads - 1) / waves_threads;
                ex.meta_blocks = (int)(mb < 1 ? 1 : (mb > 64 ? 64 : mb));
                ex.cnt_of_slot = c->cnt_of_slot;
                ex.slot_of = c->slot_of;
                ex.uniq_total = meta->uniq_total;
                ex.counts_total = meta->counts_total;
                ex.u_total_dev = meta->u_total_dev;
                ex.scal = c->scal;
            }
            if (is_short) {
                constexpr auto kern = k_wgrad_short<true, true>;
                ensure_dynamic_lds<kern>((int)VSMEM);
                launch_smem(c, KID_WGRAD_BF16, kern, dim3((unsigned)(short_blocks + ex.meta_blocks)), dim3(VTHREADS), VSMEM,
                            s, static_cast<const uint16_t*>(X), (uint32_t)x_bytes, ids, rows, (uint32_t)g_bytes,
                            rows_dev, d_in, d, pad_id, S, out, row_begin, row_end, add_here, ex);
            } else {
                constexpr auto kern = k_wgrad_tn_bf16<false, true>;
                ensure_dynamic_lds<kern>((int)WSMEM);
                launch_smem(c, KID_WGRAD_BF16, kern, dim3((unsigned)(tiles * S + ex.meta_blocks)), dim3(kWgradWaves * 64),
                            WSMEM, s, static_cast<const uint16_t*>(X), (uint32_t)x_bytes, ids, rows, (uint32_t)g_bytes,
                            rows_dev, d_in, d, pad_id, S, c->wg_partial, row_begin, row_end, ex);
            }
            exported = true;
        } else if (is_short) {
            auto go = [&](auto kern) {
                launch_smem(c, KID_WGRAD_BF16, kern, dim3((unsigned)short_blocks), dim3(VTHREADS), VSMEM, s,
                            static_cast<const uint16_t*>(X), (uint32_t)x_bytes, ids, rows, (uint32_t)g_bytes,
                            rows_dev, d_in, d, pad_id, S, out, row_begin, row_end, add_here, no_export);
            };
#define GRAM_GO(...) { ensure_dynamic_lds<__VA_ARGS__>((int)VSMEM); go(__VA_ARGS__); }
            if (gb && ids) GRAM_GO(k_wgrad_short<false, true, true>)
            else if (gb) GRAM_GO(k_wgrad_short<false, false, true>)
            else if (ids) GRAM_GO(k_wgrad_short<false, true>)
            else GRAM_GO(k_wgrad_short<false, false>)
#undef GRAM_GO
        } else {
            auto go = [&](auto kern, int kid, int64_t xb, int64_t gbytes) {
                launch_smem(c, kid, kern, dim3((unsigned)(tiles * S)), dim3(kWgradWaves * 64), WSMEM, s,
                            static_cast<const uint16_t*>(X), (uint32_t)xb, ids, rows, (uint32_t)gbytes,
                            rows_dev, d_in, d, pad_id, S, c->wg_partial, row_begin, row_end, no_export);
            };
#define GRAM_GO(KID, XB, GBYTES, ...) { ensure_dynamic_lds<__VA_ARGS__>((int)WSMEM); go(__VA_ARGS__, KID, XB, GBYTES); }
            // (the descriptors of the WIDE variant are not used)
            if (wide && gb) GRAM_GO(KID_WGRAD_BF16_WIDE, 0, 0, k_wgrad_tn_bf16<true, false, true>)
            else if (wide) GRAM_GO(KID_WGRAD_BF16_WIDE, 0, 0, k_wgrad_tn_bf16<true>)
            else if (gb) {
                auto rows_go = [&](auto kern) {
                    launch_smem(c, KID_WGRAD_BF16, kern, dim3((unsigned)(tiles * S)), dim3(kWgradWaves * 64), kPairLds, s,
                                static_cast<const uint16_t*>(X), (uint32_t)x_bytes, ids, reinterpret_cast<const uint16_t*>(rows),
                                (uint32_t)g_bytes, rows_dev, d_in, d, pad_id, S, c->wg_partial, row_begin, row_end);
                };
                ensure_dynamic_lds<k_wgrad_rows_bf16<true>>(kPairLds);
                ensure_dynamic_lds<k_wgrad_rows_bf16<false>>(kPairLds);
                if (ids) rows_go(k_wgrad_rows_bf16<true>);
                else rows_go(k_wgrad_rows_bf16<false>);
            }
            else GRAM_GO(KID_WGRAD_BF16, x_bytes, g_bytes, k_wgrad_tn_bf16<false>)
#undef GRAM_GO
        }
    } else {
        // a few rows are one range that goes straight to dW: the reduction launch costs more than the rows
        int64_t rows_bound = (other || c->dense) ? cap : (c->window_positions < cap ? c->window_positions : cap);
        if (rows_bound > row_end - row_begin) rows_bound = row_end - row_begin;
        direct = rows_bound <= 128;
        if (direct) S = 1;
        launch(c, KID_WGRAD_F32, k_wgrad_f32, dim3((d + 63) / 64, (d_in + 3) / 4, S), dim3(kBlock), s,
               static_cast<const float*>(X), ids, rows, rows_dev, d_in, d, pad_id, S,
               direct ? dW : c->wg_partial, row_begin, row_end, direct && accumulate ? 1 : 0);
    }
    if (direct) {
        if (loss) pseudo_loss(c, *loss, s);
        return exported;
    }
    const int64_t n4 = (int64_t)d_in * d / 4;
    const LossSum sum = loss ? *loss : LossSum{nullptr, 0, nullptr};
    launch(c, KID_WGRAD_REDUCE, k_wgrad_reduce, dim3((unsigned)((n4 + kBlock - 1) / kBlock + (loss ? 1 : 0))), dim3(kBlock), s,
           reinterpret_cast<const float4*>(c->wg_partial), n4, S, reinterpret_cast<float4*>(dW), accumulate ? 1 : 0, sum);
    return exported;
}

}  // namespace gram
