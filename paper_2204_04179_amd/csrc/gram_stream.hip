// HBM-bound kernels of the GRAM step: row gather of representations to
// interaction positions (Algorithm 1 step 1, second half; for large batches the
// contraction in gram_gemm.hip does most of it and only the copy for very
// popular items runs here), the pseudo-targets of step 3 (Eq. 6), the
// deterministic per-item reduction of dL/dH (step 3, Eq. 6) into the buffer
// that persists over a Multi-step window (Section 4.2), and the export of that
// buffer at the end of the window.
//
// No float atomics anywhere: each buffer row has exactly one writer and a
// fixed order of additions, so results are bit-identical from run to run.
#include "gram_internal.h"

namespace gram {

template <int NWAVES = kWavesPerBlock>
__device__ __forceinline__ int block_excl_scan(int v, int* total, int* sm /*[NWAVES]*/)
{
    const int incl = wave_incl_scan(v);
    if (lane_id() == kWave - 1) sm[wave_id()] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
        const int t = sm[w];
        if (w < wave_id()) base += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return base + incl - v;
}

__device__ __forceinline__ int block_sum(int v, int* sm)
{
    v = wave_sum(v);
    if (lane_id() == 0) sm[wave_id()] = v;
    __syncthreads();
    int tot = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) tot += sm[w];
    __syncthreads();
    return tot;
}

__device__ __forceinline__ float4 f4_add(float4 a, float4 b)
{
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// ---- fill ------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_fill_i32(int* __restrict__ p, int64_t n, int v)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        p[i] = v;
}

void fill_i32(int* p, int64_t n, int v, hipStream_t s)
{
    if (n <= 0) return;
    int64_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)blocks), dim3(kBlock), 0, s, p, n, v);
}

__global__ __launch_bounds__(kBlock) void k_iota_i32(int* __restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        p[i] = (int)i;
}

void iota_i32(int* p, int64_t n, hipStream_t s)
{
    if (n <= 0) return;
    int64_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_iota_i32, dim3((unsigned)blocks), dim3(kBlock), 0, s, p, n);
}

// ---- gather: H[p,:] = E[inverse[p],:] ---------------------------------------

// A block copies `rows_per_block` consecutive positions (about 32 KiB), so its
// writes to H form one contiguous stream; each thread keeps kGatherUnroll
// independent 16-byte loads in flight.  H is written once and not re-read here,
// so its stores bypass the caches; rows of E are re-read (once per occurrence)
// and keep ordinary cached loads, which measured faster than streaming ones.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kGatherUnroll = 8;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// One group of 4 columns of a row of H: float32 as it is, or rounded to bf16 (HB).
template <bool HB>
__device__ __forceinline__ void store_h4(void* __restrict__ H, int64_t group, f32x4 v)
{
    if (HB) {
        const u32x2 h = {pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
        __builtin_nontemporal_store(h, static_cast<u32x2*>(H) + group);
    } else {
        __builtin_nontemporal_store(v, static_cast<f32x4*>(H) + group);
    }
}

template <bool HB>
__global__ __launch_bounds__(kBlock) void k_gather_rows(const f32x4* __restrict__ E,
                                                        const int* __restrict__ inverse, int64_t m,
                                                        int cols4, void* __restrict__ H,
                                                        int rows_per_block)
{
    const int64_t p0 = (int64_t)blockIdx.x * rows_per_block;
    const int rows = (int)(p0 + rows_per_block < m ? rows_per_block : m - p0);
    const int total = rows * cols4;
    for (int e0 = 0; e0 < total; e0 += kBlock * kGatherUnroll) {
        if (e0 + kBlock * kGatherUnroll <= total) {
            // a whole group: nothing is conditional, so the loads go out together and every store
            // waits for its own load only (with conditions around them each store waited for all
            // memory operations before it, the earlier stores included)
            int64_t src[kGatherUnroll];
#pragma unroll
            for (int u = 0; u < kGatherUnroll; ++u) {
                const int e = e0 + u * kBlock + threadIdx.x;
                const int row = e / cols4;
                src[u] = (int64_t)inverse[p0 + row] * cols4 + (e - row * cols4);
            }
            f32x4 v[kGatherUnroll];
#pragma unroll
            for (int u = 0; u < kGatherUnroll; ++u) v[u] = E[src[u]];
#pragma unroll
            for (int u = 0; u < kGatherUnroll; ++u)
                store_h4<HB>(H, p0 * cols4 + e0 + u * kBlock + threadIdx.x, v[u]);
            continue;
        }
        int64_t src[kGatherUnroll];
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u) {
            const int e = e0 + u * kBlock + threadIdx.x;
            const int row = e / cols4;
            src[u] = e < total ? (int64_t)inverse[p0 + row] * cols4 + (e - row * cols4) : -1;
        }
        f32x4 v[kGatherUnroll];
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u)
            if (src[u] >= 0) v[u] = E[src[u]];
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u)
            if (src[u] >= 0) store_h4<HB>(H, p0 * cols4 + e0 + u * kBlock + threadIdx.x, v[u]);
    }
}

void gather_rows(Ctx* c, const float* E, const int* inverse, int64_t m, void* H, hipStream_t s)
{
    if (m == 0) return;
    const int cols4 = c->cfg.d / 4;
    int rows_per_block = (kGatherUnroll * kBlock + cols4 - 1) / cols4;
    if (rows_per_block < 1) rows_per_block = 1;
    const int64_t blocks = (m + rows_per_block - 1) / rows_per_block;
    if (c->cfg.h_dtype == GRAM_BF16)
        launch(c, KID_GATHER_ROWS, k_gather_rows<true>, dim3((unsigned)blocks), dim3(kBlock), s,
               reinterpret_cast<const f32x4*>(E), inverse, m, cols4, H, rows_per_block);
    else
        launch(c, KID_GATHER_ROWS, k_gather_rows<false>, dim3((unsigned)blocks), dim3(kBlock), s,
               reinterpret_cast<const f32x4*>(E), inverse, m, cols4, H, rows_per_block);
}

// Second half of the fused forward: items with more than kLightMax positions were written to
// E only; their rows are copied to their positions here.  Blocks walk the SORTED order (all
// positions of an item adjacent), 64 rows each, and leave at once when none of their rows
// belongs to such an item, so the row of E being copied stays in cache across many blocks.
// Bound by memory: rows written to random places, whole rows, V columns (16 bytes) per lane; a narrow row takes part of
// the block, and parts of the block share the 64 rows.  The rows of one item are a run: its row of E is loaded ahead of the run
// and waited for there, so that nothing in the run waits for memory (where the load was a condition inside the loop, every
// store waited for the store before it).  204,800 positions, Zipf 1.05, about half of them heavy, before / now in us: width 64 float32
// 15.0 / 10.6, bf16 16.2 / 8.0; 256 29.5 / 28.9, 17.3 / 16.6; 400 45.4 / 45.9, 37.4 / 35.1; 1024 104.7 / 102.0, 55.3 / 54.2 (4.8 TB/s).
constexpr int kHeavyRows = 64;
template <bool HB, int V>
__global__ __launch_bounds__(kBlock) void k_gather_heavy(const f32x4* __restrict__ E,
                                                         const int* __restrict__ seg_of_row,
                                                         const int* __restrict__ offsets,
                                                         const int* __restrict__ perm, int64_t m,
                                                         int cols, void* __restrict__ H)
{
    static_assert(V == 4 || (HB && V == 8), "16 bytes per lane at most");
    static_assert(kHeavyRows == kWave, "a row per lane");
    __shared__ int s_src[kHeavyRows], s_dst[kHeavyRows], s_first[kHeavyRows], s_n;
    if (wave_id() == 0) {
        const int64_t r = (int64_t)blockIdx.x * kHeavyRows + lane_id();
        int j = -1, p = 0;
        if (r < m) {
            j = seg_of_row[r] & kRowSeg;
            p = perm[r];
            if (offsets[j + 1] - offsets[j] <= kLightMax) j = -1;
        }
        const int before = __shfl_up(j, 1);
        const uint64_t heavy = __ballot(j >= 0);
        if (j >= 0) {
            const int at = __popcll(heavy & ((1ull << lane_id()) - 1));
            s_src[at] = j;
            s_dst[at] = p;
            s_first[at] = lane_id() == 0 || before != j;
        }
        if (lane_id() == 0) s_n = __popcll(heavy);
    }
    __syncthreads();
    const int n = s_n;
    if (n == 0) return;
    const uint64_t firsts = __ballot(lane_id() < n && s_first[lane_id()]);
    const int lanes = cols / V, parts = lanes < kBlock ? kBlock / lanes : 1;      // lanes per row, parts of the block
    const int part = parts > 1 ? (int)threadIdx.x / lanes : 0;
    if (part >= parts) return;
    const int share = (n + parts - 1) / parts, begin = part * share, end = begin + share < n ? begin + share : n;
    for (int cp = (int)threadIdx.x - part * lanes; cp < lanes; cp += parts > 1 ? lanes : kBlock) {
        for (int row = begin; row < end;) {
            const uint64_t later = row + 1 < kHeavyRows ? firsts >> (row + 1) : 0;
            int stop = later ? row + 1 + __builtin_ctzll(later) : n;
            stop = stop < end ? stop : end;
            const f32x4* src = E + ((int64_t)s_src[row] * lanes + cp) * (V / 4);
            if (V == 8) {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                const f32x4 a = src[0], b = src[1];
                u32x4 h = {pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w)};
                asm volatile("" : "+v"(h));      // in registers before the run
#pragma unroll 4
                for (int i = row; i < stop; ++i)
                    __builtin_nontemporal_store(h, static_cast<u32x4*>(H) + ((int64_t)s_dst[i] * lanes + cp));
            } else {
                f32x4 v = src[0];
                asm volatile("" : "+v"(v));
#pragma unroll 4
                for (int i = row; i < stop; ++i) store_h4<HB>(H, (int64_t)s_dst[i] * lanes + cp, v);
            }
            row = stop;
        }
    }
}

void gather_heavy(Ctx* c, const float* E, int64_t m, void* H, hipStream_t s)
{
    if (m == 0) return;
    const int d = c->cfg.d;
    const dim3 blocks((unsigned)((m + kHeavyRows - 1) / kHeavyRows));
    auto go = [&](auto kern) {
        launch(c, KID_GATHER_HEAVY, kern, blocks, dim3(kBlock), s, reinterpret_cast<const f32x4*>(E), c->seg_of_row, c->offsets, c->perm, m, d, H);
    };
    // 16 bytes per lane also where a column takes 2, if rows and H allow it
    if (c->cfg.h_dtype != GRAM_BF16) go(k_gather_heavy<false, 4>);
    else if (d % 8 == 0 && (uintptr_t)H % 16 == 0) go(k_gather_heavy<true, 8>);
    else go(k_gather_heavy<true, 4>);
}

// ---- pseudo-targets (Algorithm 1 step 3, Eq. 6) and the pseudo-loss (Eq. 7) -------------
//
// Ht[j,:] = E[j,:] - G[row of item j,:] for the unique items of the current batch, with G the
// gradient accumulated so far in the window (this batch included), and
// loss = 1/2 sum |Ht - E|^2 = 1/2 sum G^2 over those rows.  A block takes kPseudoRows items;
// its threads add their squares in double, the block adds the thread sums in a fixed tree
// and writes one partial; k_pseudo_loss adds the partials in index order: no atomics, the
// same bits on every run.  An item whose row was dropped (buffer full) keeps Ht = E.
__global__ __launch_bounds__(kBlock) void k_pseudo_target(const f32x4* __restrict__ E,
                                                          const f32x4* __restrict__ G,
                                                          const int* __restrict__ seg_slot,
                                                          const int* __restrict__ u_ws, int cols4,
                                                          f32x4* __restrict__ Ht,
                                                          double* __restrict__ partial)
{
    __shared__ double s_sum[kBlock];
    const int U = *u_ws;
    const int j0 = blockIdx.x * kPseudoRows;
    double sum = 0.0;
    if (j0 < U) {
        const int rows = U - j0 < kPseudoRows ? U - j0 : kPseudoRows;
        const int total = rows * cols4;
        for (int e = threadIdx.x; e < total; e += kBlock) {
            const int r = e / cols4, cq = e - r * cols4;
            const int code = seg_slot[j0 + r];
            f32x4 g = {0.f, 0.f, 0.f, 0.f};
            if (code >= 0) g = G[(int64_t)(code & (kSlotNew - 1)) * cols4 + cq];
            const f32x4 h = E[(int64_t)(j0 + r) * cols4 + cq];
            if (Ht) __builtin_nontemporal_store(h - g, &Ht[(int64_t)(j0 + r) * cols4 + cq]);
            sum += (double)g.x * g.x + (double)g.y * g.y + (double)g.z * g.z + (double)g.w * g.w;
        }
    }
    s_sum[threadIdx.x] = sum;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s_sum[threadIdx.x] += s_sum[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = s_sum[0];
}

__global__ __launch_bounds__(kBlock) void k_pseudo_loss(const double* __restrict__ partial,
                                                        const int* __restrict__ u_ws, int parts,
                                                        double* __restrict__ loss)
{
    half_sum_of(partial, u_ws ? (*u_ws + kPseudoRows - 1) / kPseudoRows : parts, loss);
}

void pseudo_target(Ctx* c, const float* E, float* Ht, double* loss_dev, hipStream_t s)
{
    const int64_t rows_max = c->cur_m < c->cap_u ? c->cur_m : c->cap_u;
    const int64_t blocks = (rows_max + kPseudoRows - 1) / kPseudoRows;
    if (blocks > 0)
        launch(c, KID_PSEUDO_TARGET, k_pseudo_target, dim3((unsigned)blocks), dim3(kBlock), s,
               reinterpret_cast<const f32x4*>(E), reinterpret_cast<const f32x4*>(c->G), c->seg_slot,
               c->scal + kSU, c->cfg.d / 4, reinterpret_cast<f32x4*>(Ht), c->loss_part);
    if (loss_dev)
        launch(c, KID_PSEUDO_LOSS, k_pseudo_loss, dim3(1), dim3(kBlock), s, c->loss_part, (const int*)(c->scal + kSU),
               0, loss_dev);
}

// ---- one content-encoder batch of the update (Alg. 1 step 4, Eq. 7) ---------
//
// The caller lists the items of the batch.  The IDs are copied once, checked: an ID outside
// [0, N) is replaced by a harmless one (the padding item, else item 0) and latches the range
// error, so the contraction kernels never form an address from it.
__global__ __launch_bounds__(kBlock) void k_chunk_ids(const int* __restrict__ ids, int n, int vocab_n,
                                                      int fix_id, int* __restrict__ out,
                                                      int* __restrict__ scal)
{
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j == 0) scal[kSChunkN] = n;
    if (j >= n) return;
    int id = ids[j];
    if (id < 0 || id >= vocab_n) {
        id = fix_id;
        atomicOr(&scal[kSErr], kErrBitRange);
    }
    out[j] = id;
}

void chunk_ids_prepare(Ctx* c, const int* ids, int64_t n, hipStream_t s)
{
    const int64_t blocks = n > 0 ? (n + kBlock - 1) / kBlock : 1;
    launch(c, KID_CHUNK_IDS, k_chunk_ids, dim3((unsigned)blocks), dim3(kBlock), s, ids, (int)n,
           c->cfg.vocab_n, c->cfg.pad_id >= 0 ? c->cfg.pad_id : 0, c->chunk_ids, c->scal);
}

// float32 contexts: R[j,:] holds the encoder's output for item j of the batch and becomes the regression
// miss R[j,:] - Ht[j,:] (zero for the padding item); the block's share of sum |miss|^2 goes to partial[] as
// in k_pseudo_target (double per thread, fixed tree, k_pseudo_loss adds the blocks in index order).  (The
// bf16 contractions subtract as they store, and leave such block sums themselves.)
__global__ __launch_bounds__(kBlock) void k_pseudo_miss(f32x4* __restrict__ R,
                                                        const f32x4* __restrict__ Ht,
                                                        const int* __restrict__ ids, int n, int pad_id,
                                                        int cols4, double* __restrict__ partial)
{
    __shared__ double s_sum[kBlock];
    const int j0 = blockIdx.x * kPseudoRows;
    double sum = 0.0;
    const int rows = n - j0 < kPseudoRows ? n - j0 : kPseudoRows;
    const int total = rows * cols4;
    for (int e = threadIdx.x; e < total; e += kBlock) {
        const int r = e / cols4, cq = e - r * cols4;
        const int64_t at = (int64_t)(j0 + r) * cols4 + cq;
        f32x4 m = {0.f, 0.f, 0.f, 0.f};
        if (ids[j0 + r] != pad_id) m = R[at] - __builtin_nontemporal_load(&Ht[at]);
        R[at] = m;
        sum += (double)m.x * m.x + (double)m.y * m.y + (double)m.z * m.z + (double)m.w * m.w;
    }
    s_sum[threadIdx.x] = sum;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s_sum[threadIdx.x] += s_sum[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = s_sum[0];
}

void pseudo_loss(Ctx* c, const LossSum& loss, hipStream_t s)
{
    launch(c, KID_PSEUDO_LOSS, k_pseudo_loss, dim3(1), dim3(kBlock), s, loss.part, (const int*)nullptr, loss.parts, loss.out);
}

void pseudo_miss(Ctx* c, float* R, const float* Ht, int64_t n, double* loss_dev, hipStream_t s)
{
    const int64_t blocks = (n + kPseudoRows - 1) / kPseudoRows;
    if (blocks > 0)
        launch(c, KID_PSEUDO_MISS, k_pseudo_miss, dim3((unsigned)blocks), dim3(kBlock), s,
               reinterpret_cast<f32x4*>(R), reinterpret_cast<const f32x4*>(Ht), c->chunk_ids, (int)n,
               c->cfg.pad_id, c->cfg.d / 4, c->loss_part);
    if (loss_dev) pseudo_loss(c, {c->loss_part, (int)blocks, loss_dev}, s);
}

// ---- buffer rows for the items of this batch --------------------------------
//
// An item seen for the first time in the window gets the next free row of the
// persistent buffer; new items of one batch take consecutive rows in ascending
// ID order (a scan over "is new" flags), so the row layout, and with it the
// summation order of the weight gradient, is a function of the data alone.
// The dedup kernels normally work these rows out themselves (seg_slot) and the segment
// reduction commits them; the kernels below do the same job in launches of their own when the
// slot table has changed since the dedup looked at it and for an empty batch.

__global__ __launch_bounds__(kBlock) void k_slot_count(const int* __restrict__ uniq_ws,
                                                       const int* __restrict__ slot_of,
                                                       int* __restrict__ scal,
                                                       int* __restrict__ tile_sums, int first_step)
{
    __shared__ int sm[kWavesPerBlock];
    const int u = scal[kSU];
    const int j0 = blockIdx.x * kScanTile + threadIdx.x * 4;
    int s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (j0 + i < u) s += slot_of[uniq_ws[j0 + i]] < 0 ? 1 : 0;
    const int tot = block_sum(s, sm);
    if (threadIdx.x == 0) {
        tile_sums[blockIdx.x] = tot;
        if (blockIdx.x == 0) {
            scal[kSUBase] = first_step ? 0 : scal[kSUTotal];   // a flush leaves the old count behind
            scal[kSLongCount] = 0;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_slot_emit(
    const int* __restrict__ uniq_ws, const int* __restrict__ offsets, int* __restrict__ slot_of,
    int* __restrict__ id_of_slot, long long* __restrict__ cnt_of_slot, int* __restrict__ seg_slot,
    int* __restrict__ scal, const int* __restrict__ tile_sums, int cap_total)
{
    __shared__ int sm[kWavesPerBlock];
    const int u = scal[kSU];
    const int u_base = scal[kSUBase];
    int pre = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kBlock) pre += tile_sums[t];
    pre = block_sum(pre, sm);

    const int j0 = blockIdx.x * kScanTile + threadIdx.x * 4;
    int id[4], old[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        id[i] = 0;
        old[i] = 0;
        if (j0 + i < u) {
            id[i] = uniq_ws[j0 + i];
            old[i] = slot_of[id[i]];
            s += old[i] < 0 ? 1 : 0;
        }
    }
    int total;
    int run = u_base + pre + block_excl_scan(s, &total, sm);
    bool overflow = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = j0 + i;
        if (j < u) {
            const int cnt = offsets[j + 1] - offsets[j];
            if (old[i] < 0) {
                const int slot = run++;
                if (slot < cap_total) {
                    slot_of[id[i]] = slot;
                    id_of_slot[slot] = id[i];
                    cnt_of_slot[slot] = cnt;
                    seg_slot[j] = slot | kSlotNew;
                } else {
                    seg_slot[j] = -1;      // dropped: the buffer is full
                    overflow = true;
                }
            } else {
                cnt_of_slot[old[i]] += cnt;
                seg_slot[j] = old[i];
            }
        }
    }
    if (overflow) atomicOr(&scal[kSErr], kErrBitCapacity);
    // tiles past U add nothing, so the last block of the grid sees the full count
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const int nt = u_base + pre + total;
        scal[kSUTotal] = nt < cap_total ? nt : cap_total;
    }
}

// Small batches: the same result from one block of 1024 threads that walks tiles of 4096 items in
// order (one launch, and for most small batches one pass).
constexpr int kSlotSmallThreads = 1024;
__global__ __launch_bounds__(kSlotSmallThreads) void k_slot_small(
    const int* __restrict__ uniq_ws, const int* __restrict__ offsets, int* __restrict__ slot_of,
    int* __restrict__ id_of_slot, long long* __restrict__ cnt_of_slot, int* __restrict__ seg_slot,
    int* __restrict__ scal, int cap_total, int first_step)
{
    __shared__ int sm[kSlotSmallThreads / kWave];
    const int u = scal[kSU];
    int run_base = first_step ? 0 : scal[kSUTotal];             // a flush leaves the old count behind
    bool overflow = false;
    const int t4 = (int)threadIdx.x * 4;
    for (int j0 = t4; j0 - t4 < u; j0 += kSlotSmallThreads * 4) {   // uniform trip count
        int id[4], old[4], sflag = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            id[i] = 0;
            old[i] = 0;
            if (j0 + i < u) {
                id[i] = uniq_ws[j0 + i];
                old[i] = slot_of[id[i]];
                sflag += old[i] < 0 ? 1 : 0;
            }
        }
        int total;
        int run = run_base + block_excl_scan<kSlotSmallThreads / kWave>(sflag, &total, sm);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + i;
            if (j < u) {
                const int cnt = offsets[j + 1] - offsets[j];
                if (old[i] < 0) {
                    const int slot = run++;
                    if (slot < cap_total) {
                        slot_of[id[i]] = slot;
                        id_of_slot[slot] = id[i];
                        cnt_of_slot[slot] = cnt;
                        seg_slot[j] = slot | kSlotNew;
                    } else {
                        seg_slot[j] = -1;
                        overflow = true;
                    }
                } else {
                    cnt_of_slot[old[i]] += cnt;
                    seg_slot[j] = old[i];
                }
            }
        }
        run_base += total;
    }
    if (overflow) atomicOr(&scal[kSErr], kErrBitCapacity);
    __syncthreads();      // every thread has read scal[kSUTotal] before it changes
    if (threadIdx.x == 0) {
        scal[kSUTotal] = run_base < cap_total ? run_base : cap_total;
        scal[kSLongCount] = 0;
    }
}

constexpr int64_t kSmallBatch = 8 * kScanTile;   // positions up to which one-block variants are used

// Dense-by-vocabulary buffer: the row of an item is its ID, so there is nothing to hand out (the segment
// reduction counts the items of a batch as it goes); an empty batch only has to make the rows count.
__global__ void k_slot_dense(int* __restrict__ scal, int vocab_n)
{
    if (threadIdx.x == 0) scal[kSUTotal] = vocab_n;      // rows the weight gradient contracts over: all of them
}

void assign_slots(Ctx* c, hipStream_t s)
{
    int64_t bound = c->cur_m < c->cap_u ? c->cur_m : c->cap_u;
    if (bound < 1) bound = 1;
    if (c->dense) {
        launch(c, KID_SLOT_EMIT, k_slot_dense, dim3(1), dim3(kWave), s, c->scal, c->cfg.vocab_n);
        return;
    }
    const int first_step = (c->steps_done == 0 && !c->window_imported) ? 1 : 0;
    if (bound <= kSmallBatch) {
        launch(c, KID_SLOT_EMIT, k_slot_small, dim3(1), dim3(kSlotSmallThreads), s, c->uniq_ws, c->offsets, c->slot_of,
               c->id_of_slot, c->cnt_of_slot, c->seg_slot, c->scal, (int)c->cap_total, first_step);
        return;
    }
    const int tiles = (int)((bound + kScanTile - 1) / kScanTile);
    launch(c, KID_SLOT_COUNT, k_slot_count, dim3(tiles), dim3(kBlock), s, c->uniq_ws, c->slot_of, c->scal,
                       c->tile_sums, first_step);
    launch(c, KID_SLOT_EMIT, k_slot_emit, dim3(tiles), dim3(kBlock), s, c->uniq_ws, c->offsets,
                       c->slot_of, c->id_of_slot, c->cnt_of_slot, c->seg_slot, c->scal, c->tile_sums,
                       (int)c->cap_total);
}

// ---- sorted-segment reduction -----------------------------------------------
//
// Rows of dH are visited in the sorted order of the batch (perm), where the
// occurrences of one item are adjacent and in ascending position.  The sorted
// rows are cut into tiles of TR = seg_rows_for(m) rows.
//  * A short segment (< TR rows) is summed, whole and in order, by the
//    tile that holds its first row, even where it runs past the tile's end; it
//    needs no partial result.
//  * A long segment is summed tile by tile into partial rows (seg_last for the
//    tile where it starts, seg_first for every later tile), and k_seg_combine
//    adds the partials in ascending tile order.
//
// What bounds it: HBM where the batch is large (5.3 TB/s), and on small ones the chain of dependent
// round trips to memory.  A wave holds one sorted row per lane (a tile and the end of its last segment
// are at most 2 TR - 1 <= 63 rows): the rows' segments, flags and positions come with one load each, ballots
// over the flags tell what the tile has to sum, and the rows of dH are requested next.  (Looking the
// bounds up through seg_of_row, offsets and uniq took three round trips more.)  The rows of the buffer that a step adds to
// are fetched with the rows of dH they belong to: fetched when a segment ends, each drained all loads in flight.
// A row is addressed by a descriptor of its own, built from scalars: one of zero length reads zeros and
// touches no memory, so the loads of a group are unconditional.
constexpr int kDstNone = -1;    // nothing to write (dropped item)
constexpr int kDstFirst = -2;   // partial row seg_first[tile]
constexpr int kDstLast = -3;    // partial row seg_last[tile]
constexpr int kSegPlainLoads = 16384;   // batches of at most this many positions read dH with plain loads
constexpr int kRowDescFlags = 0x00027000;   // raw buffer: 32-bit elements, no swizzle
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void write_final(float4* __restrict__ G, int cols4, int col, int code,
                                            bool is_pad, float4 acc)
{
    if (code == kDstNone) return;
    float4* dst = G + (int64_t)(code & (kSlotNew - 1)) * cols4 + col;
    if (code & kSlotNew) {
        // a row new to the window is not read again before the next step at the earliest: stored past
        // the caches, it leaves them to the forward's operands (measured: 8 us per step on the large shape)
        const float4 w = is_pad ? make_float4(0.f, 0.f, 0.f, 0.f) : acc;
        __builtin_nontemporal_store(f32x4{w.x, w.y, w.z, w.w}, reinterpret_cast<f32x4*>(dst));
    } else if (!is_pad) {
        *dst = f4_add(*dst, acc);
    }
}

// Row `row` of a matrix of cols4 float4 columns (row < 0: an empty row), lane's column offset col_off.
template <bool PLAIN>
__device__ __forceinline__ f32x4 load_row(const float4* base, int row, int cols4, uint32_t col_off)
{
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float4*>(base + (int64_t)(row < 0 ? 0 : row) * cols4), 0, row < 0 ? 0 : cols4 * 16, kRowDescFlags);
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, col_off, 0, PLAIN ? 0 : 2));
}

// TR: rows per tile.  UN: rows in flight.  PLAIN: dH read with plain instead of non-temporal loads (a row is
// read exactly once; batches of a few thousand positions often still have it in a cache).  OLD: the
// buffer may hold rows of the batch's items already (not so in the first step of a window).
template <int TR, int UN, bool PLAIN, bool OLD>
__global__ __launch_bounds__(kBlock) void k_seg_reduce(
    const float4* __restrict__ dH, const int* __restrict__ perm, const int* __restrict__ seg_of_row,
    const int* __restrict__ offsets, const int* __restrict__ uniq_ws,
    int* seg_slot, int n, int cols4, float4* __restrict__ G,
    float4* __restrict__ seg_first, float4* __restrict__ seg_last, int* __restrict__ scal,
    int4* __restrict__ long_list, int* __restrict__ slot_of, int* __restrict__ id_of_slot,
    long long* __restrict__ cnt_of_slot, long long* __restrict__ cnt64, int vocab_n)
{
    static_assert(2 * TR <= kWave, "a tile and the end of its last segment fit the lanes of a wave");
    const int t = blockIdx.x, lane = lane_id();
    const int r0 = t * TR, r = r0 + lane;
    const int info = r < n ? seg_of_row[r] : kRowHead;       // (past the end: closes the last segment)
    const int p = r < n ? perm[r] : 0;
    const int pad_seg = scal[kSPadSeg];
    // slot_of given: the buffer rows in seg_slot were worked out by the dedup and are committed
    // here, each item by the lane that holds the first row of its segment (one tile holds it)
    // cnt64 given (dense layout): the row of an item is its ID; its count grows here the same way
    const bool dense = cnt64 != nullptr;
    const bool commit = (slot_of != nullptr || dense) && blockIdx.y == 0 && threadIdx.x < kWave;
    if (commit && t == 0 && threadIdx.x == 0) scal[kSUTotal] = dense ? vocab_n : scal[kSUNext];

    const unsigned long long heads = __ballot((info & kRowHead) != 0), longs = __ballot((info & kRowLong) != 0);
    const int tile_rows = n - r0 < TR ? n - r0 : TR;         // at least 1
    const unsigned long long in_tile = (1ull << tile_rows) - 1;
    const unsigned long long starts = (heads | longs) & in_tile;
    if (starts == 0) return;      // the tile lies inside a short segment owned by an earlier tile
    // first and one-past-last lane whose row this tile sums
    const int a = __builtin_ctzll(starts);
    const int b = (longs >> (tile_rows - 1) & 1) ? tile_rows : __builtin_ctzll(heads & ~in_tile);

    const int seg = info & kRowSeg;
    const bool mine = lane >= a && lane < b, is_long = (info & kRowLong) != 0;
    const bool is_pad = seg == pad_seg, ends = lane < kWave - 1 && (heads >> (lane + 1) & 1);
    const bool begins = (info & kRowHead) != 0;
    // a long segment's part of the tile ends with the segment or the tile; it is the segment's first
    // part if the segment starts in the tile
    const bool part_ends = mine && is_long && (ends || lane == tile_rows - 1);
    const bool is_first_part = (heads & in_tile & (2ull << lane) - 1) != 0;
    const bool head_here = begins && lane < tile_rows;
    const bool need_slot = (mine && !is_long && ends) || (part_ends && is_first_part) || (commit && head_here);
    const int slot = need_slot ? (dense ? uniq_ws : seg_slot)[seg] : 0;
    int o0 = 0, o1 = 0, id = 0;
    if ((commit && head_here) || (part_ends && is_first_part)) {
        o0 = offsets[seg];
        o1 = offsets[seg + 1];
        id = uniq_ws[seg];
    }
    // per row: source (-1: padding, not read), and 0 = keep adding, else destination code + 4
    const int src = mine && !is_pad ? p : -1;
    const int col = blockIdx.y * blockDim.x + threadIdx.x;
    const uint32_t col_off = (uint32_t)col * 16u;
    const int rows = b - a;

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int code = 0;
    for (int i0 = 0; i0 < rows; i0 += UN) {
        f32x4 v[UN], g[OLD ? UN : 1];
#pragma unroll
        for (int k = 0; k < UN; ++k)
            v[k] = load_row<PLAIN>(dH, i0 + k < rows ? __builtin_amdgcn_readlane(src, (a + i0 + k) & (kWave - 1)) : -1, cols4, col_off);
        // (the rows' codes arrive behind the first group's loads)
        if (i0 == 0) code = part_ends ? (is_first_part ? kDstLast : kDstFirst) + 4 : (mine && !is_long && ends) ? slot + 4 : 0;
        if (OLD) {
#pragma unroll
            for (int k = 0; k < UN; ++k) {
                const int c = i0 + k < rows ? __builtin_amdgcn_readlane(code, (a + i0 + k) & (kWave - 1)) - 4 : -1;
                g[k] = load_row<true>(G, c >= 0 && !(c & kSlotNew) ? c : -1, cols4, col_off);
            }
        }
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            const int at = (a + i0 + k) & (kWave - 1);
            const int cd = i0 + k < rows ? __builtin_amdgcn_readlane(code, at) : 0;
            acc += v[k];
            if (cd != 0) {
                const int dst = cd - 4;
                const bool pad = __builtin_amdgcn_readlane(is_pad ? 1 : 0, at) != 0;
                if (col < cols4) {
                    if (dst == kDstFirst) {
                        reinterpret_cast<f32x4*>(seg_first)[(int64_t)t * cols4 + col] = acc;
                    } else if (dst == kDstLast) {
                        reinterpret_cast<f32x4*>(seg_last)[(int64_t)t * cols4 + col] = acc;
                    } else if (dst >= 0) {
                        f32x4* to = reinterpret_cast<f32x4*>(G) + (int64_t)(dst & (kSlotNew - 1)) * cols4 + col;
                        // a row new to the window is stored past the caches (see write_final)
                        if (dst & kSlotNew) __builtin_nontemporal_store(acc, to);       // (padding: nothing was added)
                        else if (OLD && !pad) *to = g[k] + acc;
                    }
                }
                acc = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    // long segments that start here, for k_seg_combine: everything it would otherwise look up
    if (blockIdx.y == 0 && threadIdx.x < kWave && part_ends && is_first_part)
        long_list[atomicAdd(&scal[kSLongCount], 1)] = make_int4(t, 1 + (o1 - 1) / TR - t, slot, is_pad ? 1 : 0);
    if (commit && head_here) {
        if (dense) {
            seg_slot[seg] = id;
            cnt64[id] += o1 - o0;            // distinct within a batch: no two threads meet on a count
        } else if (slot < 0) {
            atomicOr(&scal[kSErr], kErrBitCapacity);      // dropped: the buffer is full
        } else if (slot & kSlotNew) {
            const int s = slot & (kSlotNew - 1);
            slot_of[id] = s;
            id_of_slot[s] = id;
            cnt_of_slot[s] = o1 - o0;
        } else {
            cnt_of_slot[slot] += o1 - o0;
        }
    }
}

// Sum of a long segment's partial rows in ascending tile order.  A block owns
// kFixCols4 float4 columns; its kFixLanes row lanes each add every
// kFixLanes-th partial, then lane sums are added in lane order.
__global__ __launch_bounds__(kBlock) void k_seg_combine(
    int cols4, float4* __restrict__ G, const float4* __restrict__ seg_first,
    const float4* __restrict__ seg_last, const int* __restrict__ scal, const int4* __restrict__ long_list)
{
    __shared__ float4 sm[kFixLanes][kFixCols4];
    const int cl = threadIdx.x % kFixCols4;
    const int rl = threadIdx.x / kFixCols4;
    const int col = blockIdx.y * kFixCols4 + cl;
    const int count = scal[kSLongCount];
    for (int w = blockIdx.x; w < count; w += gridDim.x) {
        // partial i of the segment: i = 0 -> seg_last[t]; i >= 1 -> seg_first[t + i]
        const int4 entry = long_list[w];
        const int t = entry.x, parts = entry.y;
        const bool is_pad = entry.w != 0;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!is_pad && col < cols4) {
            // the lane's partials are fetched eight at a time (the adds keep their order): one
            // load per round trip would make the longest segment's chain the kernel's duration
            constexpr int kAhead = 8;
            for (int i0 = rl; i0 < parts; i0 += kFixLanes * kAhead) {
                float4 v[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    const int i = i0 + k * kFixLanes;
                    const float4* src = i == 0 ? seg_last + (int64_t)t * cols4
                                               : seg_first + (int64_t)(t + i) * cols4;
                    v[k] = i < parts ? src[col] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int k = 0; k < kAhead; ++k)
                    if (i0 + k * kFixLanes < parts) acc = f4_add(acc, v[k]);
            }
        }
        sm[rl][cl] = acc;
        __syncthreads();
        if (rl == 0 && col < cols4) {
            float4 tot = sm[0][cl];
#pragma unroll
            for (int k = 1; k < kFixLanes; ++k) tot = f4_add(tot, sm[k][cl]);
            write_final(G, cols4, col, entry.z, is_pad, tot);
        }
        __syncthreads();
    }
}

// commit: seg_slot holds rows worked out by the dedup; the reduction writes them into the slot table
void segment_reduce(Ctx* c, const float* dH, int64_t m, hipStream_t s, bool commit)
{
    if (m == 0) return;
    const int n = (int)m;
    const int cols4 = c->cfg.d / 4;
    int threads = ((cols4 + kWave - 1) / kWave) * kWave;
    if (threads > kBlock) threads = kBlock;
    const int slabs = (cols4 + threads - 1) / threads;
    const int tile_rows = seg_rows_for(n);
    const int tiles = (n + tile_rows - 1) / tile_rows;
    // in the first step of a window every row is new
    const bool old = c->dense || !commit || c->steps_done > 0 || c->window_imported;
    const dim3 grid(tiles, slabs);
    auto go = [&](auto kern) {
        launch(c, KID_SEG_REDUCE, kern, grid, dim3(threads), s, reinterpret_cast<const float4*>(dH), c->perm,
               c->seg_of_row, c->offsets, c->uniq_ws, c->seg_slot, n, cols4, reinterpret_cast<float4*>(c->G),
               reinterpret_cast<float4*>(c->seg_first), reinterpret_cast<float4*>(c->seg_last), c->scal, c->long_list,
               commit && !c->dense ? c->slot_of : (int*)nullptr, c->id_of_slot, c->cnt_of_slot,
               c->dense ? c->cnt64 : (long long*)nullptr, c->cfg.vocab_n);
    };
    static_assert(kSegPlainLoads == kSegSmallBatch, "the two lines of the dispatch below coincide");
    if (n <= kSegSmallBatch) {
        if (old) go(k_seg_reduce<kSegRowsSmall, 16, true, true>);
        else go(k_seg_reduce<kSegRowsSmall, 32, true, false>);
    } else {
        if (old) go(k_seg_reduce<kSegRows, 16, false, true>);
        else go(k_seg_reduce<kSegRows, 16, false, false>);
    }
    int fix_blocks = tiles;                          // upper bound of long segments: one starts per tile
    if (fix_blocks > 1024) fix_blocks = 1024;        // a block per long segment for all but extreme batches
    launch(c, KID_SEG_COMBINE, k_seg_combine, dim3(fix_blocks, (cols4 + kFixCols4 - 1) / kFixCols4),
           dim3(kBlock), s, cols4, reinterpret_cast<float4*>(c->G), reinterpret_cast<const float4*>(c->seg_first),
           reinterpret_cast<const float4*>(c->seg_last), c->scal, c->long_list);
}

// ---- end of the window: export in ascending ID order, then empty ------------
//
// One launch: rows of G are copied out in ascending ID order while a few extra blocks export the
// IDs and counts and clear the items' entries of the slot map.
// The count of buffer rows (scal[kSUTotal]) is left as it is: every block reads it here, and
// the first step of the next window starts from zero by itself.  `n_zero`: the window is empty.

// rank_of_slot (nullable, needs sorted_slots): receives, for every buffer row, its place in
// ascending-ID order, for a weight-gradient kernel that writes the rows out itself.
__global__ __launch_bounds__(kBlock) void k_flush_meta(
    const int* __restrict__ sorted_ids, const int* __restrict__ sorted_slots,
    const long long* __restrict__ cnt_of_slot, int* __restrict__ slot_of, int* __restrict__ uniq_total,
    int* __restrict__ counts_total, long long* __restrict__ counts64_total, int* __restrict__ scal,
    int* __restrict__ u_total_dev, int n_zero, int* __restrict__ rank_of_slot)
{
    const int n = n_zero ? 0 : scal[kSUTotal];
    for (int r = blockIdx.x * kBlock + threadIdx.x; r < n; r += gridDim.x * kBlock) {
        flush_meta_row(r, sorted_ids, sorted_slots, cnt_of_slot, slot_of, uniq_total, counts_total,
                       counts64_total);
        if (rank_of_slot) rank_of_slot[sorted_slots[r]] = r;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (u_total_dev) *u_total_dev = n;
        scal[kSFlushN] = n;
    }
}

// Blocks [0, copy_blocks) copy rows; the blocks after them export IDs and counts and clear the
// slot map (kept out of the copy loop: their scattered accesses would stall the copying waves).
__global__ __launch_bounds__(kBlock) void k_flush_rows(
    const int* __restrict__ sorted_ids, const int* __restrict__ sorted_slots,
    const long long* __restrict__ cnt_of_slot, int* __restrict__ slot_of, int* __restrict__ uniq_total,
    int* __restrict__ counts_total, long long* __restrict__ counts64_total,
    const float4* __restrict__ G, int cols4, float4* __restrict__ G_total, int* __restrict__ scal,
    int* __restrict__ u_total_dev, int copy_blocks)
{
    const int n = scal[kSUTotal];
    if ((int)blockIdx.x >= copy_blocks) {
        const int mb = blockIdx.x - copy_blocks, nmb = gridDim.x - copy_blocks;
        for (int r = mb * kBlock + threadIdx.x; r < n; r += nmb * kBlock)
            flush_meta_row(r, sorted_ids, sorted_slots, cnt_of_slot, slot_of, uniq_total, counts_total,
                           counts64_total);
        if (mb == 0 && threadIdx.x == 0) {
            if (u_total_dev) *u_total_dev = n;
            scal[kSFlushN] = n;
        }
        return;
    }
    const int64_t total = (int64_t)n * cols4;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total;
         i += (int64_t)copy_blocks * kBlock) {
        const int64_t r = i / cols4;
        const int cc = (int)(i % cols4);
        const f32x4 t = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4*>(G) + (int64_t)(sorted_slots ? sorted_slots[r] : (int)r) * cols4 + cc);
        __builtin_nontemporal_store(t, reinterpret_cast<f32x4*>(G_total) + i);
    }
}

void flush_export(Ctx* c, int* uniq_total, int* counts_total, long long* counts64_total, float* G_total,
                  int* u_total_dev, hipStream_t s)
{
    if (c->steps_done == 0 && !c->window_imported) {       // nothing accumulated since the last flush
        launch(c, KID_FLUSH_META, k_flush_meta, dim3(1), dim3(kBlock), s, c->id_of_slot, (const int*)nullptr,
               c->cnt_of_slot, c->slot_of, uniq_total, counts_total, counts64_total, c->scal, u_total_dev, 1,
               (int*)nullptr);
        return;
    }
    // After one step the buffer rows are already in ascending ID order (rows are handed out in
    // that order within a step); only later steps append out of order.
    const int* sorted_ids = c->id_of_slot;
    const int* sorted_slots = nullptr;
    if (c->steps_done > 1 || c->window_imported) {
        const int r = radix_sort_pairs(c, c->id_of_slot, nullptr, 0, c->scal + kSUTotal, c->cap_total,
                                       false, 0, s);
        sorted_ids = c->keys[r];
        sorted_slots = c->vals[r];
    }
    if (G_total) {
        int64_t blocks = (c->cap_total * (c->cfg.d / 4) + kBlock - 1) / kBlock;
        if (blocks > 2048) blocks = 2048;
        int64_t meta_blocks = (c->cap_total + kBlock - 1) / kBlock;
        if (meta_blocks > 64) meta_blocks = 64;
        launch(c, KID_FLUSH_ROWS, k_flush_rows, dim3((unsigned)(blocks + meta_blocks)), dim3(kBlock), s, sorted_ids,
               sorted_slots, c->cnt_of_slot, c->slot_of, uniq_total, counts_total, counts64_total,
               reinterpret_cast<const float4*>(c->G), c->cfg.d / 4, reinterpret_cast<float4*>(G_total), c->scal,
               u_total_dev, (int)blocks);
    } else {
        int64_t blocks = (c->cap_total + kBlock - 1) / kBlock;
        if (blocks > 1024) blocks = 1024;
        launch(c, KID_FLUSH_META, k_flush_meta, dim3((unsigned)blocks), dim3(kBlock), s, sorted_ids,
               sorted_slots, c->cnt_of_slot, c->slot_of, uniq_total, counts_total, counts64_total, c->scal,
               u_total_dev, 0, (int*)nullptr);
    }
}

// The export without the rows: IDs and counts in ascending-ID order, slot map cleared, and the
// place of every buffer row in that order (returned; NULL: the rows are in that order already).
// The caller's weight-gradient kernel then writes the rows themselves.  Needs a non-empty window.
// *left_to_caller: nothing was launched (a one-step window); the caller's kernel does this part too.
const int* flush_meta_and_ranks(Ctx* c, int* uniq_total, int* counts_total, int* u_total_dev, hipStream_t s,
                                bool* left_to_caller)
{
    const int* sorted_ids = c->id_of_slot;
    const int* sorted_slots = nullptr;
    int* ranks = nullptr;
    *left_to_caller = false;
    if (c->steps_done <= 1 && !c->window_imported) {
        // one step: the rows are in order already and nothing has to be ranked; a few extra blocks
        // of the caller's weight-gradient launch export the IDs and counts
        *left_to_caller = true;
        return nullptr;
    }
    {
        const int r = radix_sort_pairs(c, c->id_of_slot, nullptr, 0, c->scal + kSUTotal, c->cap_total,
                                       false, 0, s);
        sorted_ids = c->keys[r];
        sorted_slots = c->vals[r];
        ranks = c->chunk_ids;          // [cap_chunk >= cap_total]: free between content-encoder batches
    }
    int64_t blocks = (c->cap_total + kBlock - 1) / kBlock;
    if (blocks > 1024) blocks = 1024;
    launch(c, KID_FLUSH_META, k_flush_meta, dim3((unsigned)blocks), dim3(kBlock), s, sorted_ids, sorted_slots,
           c->cnt_of_slot, c->slot_of, uniq_total, counts_total, (long long*)nullptr, c->scal, u_total_dev, 0,
           ranks);
    return ranks;
}

// ---- slot table: a saved window state merged into the buffer ----------------------------
//
// One block walks the listed items in tiles of 4096 exactly as k_slot_small walks the items of a
// batch: an item the window has not met takes the next free row (in list order), an item it has
// met keeps its row; the saved count is added (64-bit counts, as in the dense layout).
// code[j] receives the row (kSlotNew set for a fresh row, -1 when the buffer is full or the ID is
// outside [0, N)); k_import_rows then writes or adds the saved gradient rows.
__global__ __launch_bounds__(kSlotSmallThreads) void k_slot_import(
    const int* __restrict__ ids, const long long* __restrict__ counts, int n, int vocab_n,
    int* __restrict__ slot_of, int* __restrict__ id_of_slot, long long* __restrict__ cnt_of_slot,
    int* __restrict__ code, int* __restrict__ scal, int cap_total, int first_touch)
{
    __shared__ int sm[kSlotSmallThreads / kWave];
    int run_base = first_touch ? 0 : scal[kSUTotal];
    int err = 0;
    const int t4 = (int)threadIdx.x * 4;
    for (int j0 = t4; j0 - t4 < n; j0 += kSlotSmallThreads * 4) {   // uniform trip count
        int id[4], old[4], sflag = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            id[i] = -1;
            old[i] = 0;
            if (j0 + i < n) {
                const int v = ids[j0 + i];
                if (v >= 0 && v < vocab_n) {
                    id[i] = v;
                    old[i] = slot_of[v];
                    sflag += old[i] < 0 ? 1 : 0;
                } else {
                    err |= kErrBitRange;
                }
            }
        }
        int total;
        int run = run_base + block_excl_scan<kSlotSmallThreads / kWave>(sflag, &total, sm);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + i;
            if (j >= n) continue;
            if (id[i] < 0) {
                code[j] = -1;
                continue;
            }
            const long long c64 = counts[j];
            if (old[i] < 0) {
                const int slot = run++;
                if (slot < cap_total) {
                    slot_of[id[i]] = slot;
                    id_of_slot[slot] = id[i];
                    cnt_of_slot[slot] = c64;
                    code[j] = slot | kSlotNew;
                } else {
                    code[j] = -1;
                    err |= kErrBitCapacity;
                }
            } else {
                cnt_of_slot[old[i]] += c64;
                code[j] = old[i];
            }
        }
        run_base += total;
    }
    if (err) atomicOr(&scal[kSErr], err);
    if (threadIdx.x == 0) scal[kSUTotal] = run_base < cap_total ? run_base : cap_total;
}

__global__ __launch_bounds__(kBlock) void k_import_rows(const int* __restrict__ code,
                                                        const f32x4* __restrict__ rows, int n,
                                                        int cols4, f32x4* __restrict__ G)
{
    const int64_t total = (int64_t)n * cols4;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t r = i / cols4;
        const int cc = (int)(i % cols4);
        const int cd = code[r];
        if (cd < 0) continue;
        f32x4* dst = G + (int64_t)(cd & (kSlotNew - 1)) * cols4 + cc;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (rows) v = rows[i];
        *dst = (cd & kSlotNew) ? v : *dst + v;
    }
}

void import_slots(Ctx* c, const int* ids, const long long* counts, const float* rows, int64_t n,
                  hipStream_t s)
{
    const int first_touch = (c->steps_done == 0 && !c->window_imported) ? 1 : 0;
    launch(c, KID_SLOT_EMIT, k_slot_import, dim3(1), dim3(kSlotSmallThreads), s, ids, counts, (int)n,
           c->cfg.vocab_n, c->slot_of, c->id_of_slot, c->cnt_of_slot, c->chunk_ids, c->scal,
           (int)c->cap_total, first_touch);
    if (n == 0) return;
    int64_t blocks = (n * (c->cfg.d / 4) + kBlock - 1) / kBlock;
    if (blocks > 2048) blocks = 2048;
    launch(c, KID_FLUSH_ROWS, k_import_rows, dim3((unsigned)blocks), dim3(kBlock), s, c->chunk_ids,
           reinterpret_cast<const f32x4*>(rows), (int)n, c->cfg.d / 4, reinterpret_cast<f32x4*>(c->G));
}

// ---- dense-by-vocabulary buffer: end of the window, and resuming one --------------------
//
// The items of the window are those with a non-zero count.  Tiles of kScanTile IDs are counted,
// then every tile finds its place from the counts of the tiles before it and writes its items'
// IDs (ascending by construction) and counts, clearing the counts; a third kernel copies the
// items' rows out and zeroes them, which is what makes "always add" correct in the next window.

__global__ __launch_bounds__(kBlock) void k_dense_count(const long long* __restrict__ cnt64,
                                                        int vocab_n, int* __restrict__ tile_sums)
{
    __shared__ int sm[kWavesPerBlock];
    const int i0 = blockIdx.x * kScanTile + threadIdx.x * 4;
    int s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i0 + i < vocab_n) s += cnt64[i0 + i] != 0 ? 1 : 0;
    const int tot = block_sum(s, sm);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kBlock) void k_dense_emit(
    long long* __restrict__ cnt64, int vocab_n, const int* __restrict__ tile_sums,
    int* __restrict__ list, int* __restrict__ uniq_total, int* __restrict__ counts_total,
    long long* __restrict__ counts64_total, int* __restrict__ scal, int* __restrict__ u_total_dev)
{
    __shared__ int sm[kWavesPerBlock];
    int pre = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kBlock) pre += tile_sums[t];
    pre = block_sum(pre, sm);
    const int i0 = blockIdx.x * kScanTile + threadIdx.x * 4;
    long long cnt[4];
    int s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        cnt[i] = i0 + i < vocab_n ? cnt64[i0 + i] : 0;
        s += cnt[i] != 0 ? 1 : 0;
    }
    int total;
    int at = pre + block_excl_scan(s, &total, sm);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (cnt[i] != 0) {
            list[at] = i0 + i;
            if (uniq_total) uniq_total[at] = i0 + i;
            if (counts_total) counts_total[at] = cnt[i] > 0x7fffffffLL ? 0x7fffffff : (int)cnt[i];
            if (counts64_total) counts64_total[at] = cnt[i];
            cnt64[i0 + i] = 0;
            ++at;
        }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        if (u_total_dev) *u_total_dev = pre + total;
        scal[kSFlushN] = pre + total;
    }
}

__global__ __launch_bounds__(kBlock) void k_dense_rows(const int* __restrict__ list,
                                                       const int* __restrict__ scal,
                                                       f32x4* __restrict__ G, int cols4,
                                                       f32x4* __restrict__ G_total)
{
    const int64_t total = (int64_t)scal[kSFlushN] * cols4;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t r = i / cols4;
        const int cc = (int)(i % cols4);
        f32x4* src = G + (int64_t)list[r] * cols4 + cc;
        if (G_total) __builtin_nontemporal_store(*src, G_total + i);
        *src = zero;
    }
}

void flush_dense(Ctx* c, int* uniq_total, int* counts_total, long long* counts64_total, float* G_total,
                 int* u_total_dev, hipStream_t s)
{
    const int n = c->cfg.vocab_n;
    const int tiles = (n + kScanTile - 1) / kScanTile;
    int* list = c->keys[0];
    launch(c, KID_FLUSH_META, k_dense_count, dim3(tiles), dim3(kBlock), s, c->cnt64, n, c->dense_sums);
    launch(c, KID_FLUSH_META, k_dense_emit, dim3(tiles), dim3(kBlock), s, c->cnt64, n, c->dense_sums, list,
           uniq_total, counts_total, counts64_total, c->scal, u_total_dev);
    int64_t blocks = ((int64_t)n * (c->cfg.d / 4) + kBlock - 1) / kBlock;
    if (blocks > 2048) blocks = 2048;
    launch(c, KID_FLUSH_ROWS, k_dense_rows, dim3((unsigned)blocks), dim3(kBlock), s, list, c->scal,
           reinterpret_cast<f32x4*>(c->G), c->cfg.d / 4, reinterpret_cast<f32x4*>(G_total));
}

// A saved window state merged into the buffer: counts and rows of the listed (distinct) items are
// added.  An ID outside [0, N) latches the range error and is skipped.
__global__ __launch_bounds__(kBlock) void k_dense_import(const int* __restrict__ ids,
                                                         const long long* __restrict__ counts,
                                                         const f32x4* __restrict__ rows, int n,
                                                         int vocab_n, int cols4,
                                                         long long* __restrict__ cnt64,
                                                         f32x4* __restrict__ G, int* __restrict__ scal)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[kSUTotal] = vocab_n;
    const int64_t total = (int64_t)n * cols4;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t r = i / cols4;
        const int cc = (int)(i % cols4);
        const int id = ids[r];
        if (id < 0 || id >= vocab_n) {
            if (cc == 0) atomicOr(&scal[kSErr], kErrBitRange);
            continue;
        }
        if (cc == 0) cnt64[id] += counts[r];
        if (rows) {
            f32x4* dst = G + (int64_t)id * cols4 + cc;
            *dst = *dst + rows[i];
        }
    }
}

void import_dense(Ctx* c, const int* ids, const long long* counts, const float* rows, int64_t n,
                  hipStream_t s)
{
    int64_t blocks = (n * (c->cfg.d / 4) + kBlock - 1) / kBlock;
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    launch(c, KID_FLUSH_ROWS, k_dense_import, dim3((unsigned)blocks), dim3(kBlock), s, ids, counts,
           reinterpret_cast<const f32x4*>(rows), (int)n, c->cfg.vocab_n, c->cfg.d / 4, c->cnt64,
           reinterpret_cast<f32x4*>(c->G), c->scal);
}

}  // namespace gram
