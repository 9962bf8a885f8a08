// Dedup of a batch of item IDs: the set B_I of unique items (Table 1 of the
// paper; Algorithm 1 ranges over it), its inverse index and multiplicities.
//
// Method: stable LSD radix sort of (id, position) pairs over only the
// ceil(log2 N) significant key bits, in digits of up to 10 bits (at most two
// passes for a vocabulary of a million items), followed by head-flag scan and
// compaction.  Each 64-lane wave owns a contiguous chunk of keys; ranks inside
// a wave come from ballot-based digit matching, ranks across blocks from a
// per-block digit table that is prefix-summed down its columns.  Small batches
// are ranked by counting comparisons instead (k_rank_small).
// All counters are integer (LDS atomics are order independent), so the result
// is exact.
#include "gram_internal.h"

namespace gram {

// Counters that a wave re-reads from LDS after its own lanes have written them are accessed
// through volatile pointers IN THE LDS ADDRESS SPACE: a volatile pointer without an address
// space is compiled to flat, system-coherent accesses, each followed by a wait for every
// outstanding memory operation of the wave (its scattered global stores included).
typedef __attribute__((address_space(3))) int lds_i32;

// Exclusive scan of one value per thread over a 256-thread block; *total gets the block sum.
__device__ __forceinline__ int block_excl_scan(int v, int* total, int* sm /*[kWavesPerBlock]*/)
{
    const int incl = wave_incl_scan(v);
    if (lane_id() == kWave - 1) sm[wave_id()] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
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

constexpr int kSortBatch = 16;   // rounds whose keys are loaded ahead

// A block of 4 waves owns items * 256 consecutive keys; wave w of the block owns
// the w-th quarter of them.
SortPlan make_sort_plan(int key_bits, int64_t n_max)
{
    SortPlan p{};
    if (key_bits < 1) key_bits = 1;
    p.passes = (key_bits + kMaxDigitBits - 1) / kMaxDigitBits;
    int left = key_bits;
    for (int i = 0; i < p.passes; ++i) {
        int b = (left + (p.passes - i) - 1) / (p.passes - i);
        p.digit_bits[i] = b;
        left -= b;
    }
    // about 256 blocks (one per CU): the scatter pass issues two 4-byte stores per key to
    // unrelated addresses, and the rate of such stores per CU is what bounds it
    int64_t items = (n_max + (int64_t)kBlock * 256 - 1) / ((int64_t)kBlock * 256);
    if (items < 4) items = 4;
    if (items > 64) items = 64;
    p.items = (int)items;
    const int64_t kpb = (int64_t)kBlock * p.items;
    int64_t nb = (n_max + kpb - 1) / kpb;
    if (nb < 1) nb = 1;
    p.blocks = (int)nb;
    return p;
}

// The keys of one wave's chunk are walked kSortBatch rounds of 64 keys at a time; the keys of a
// batch (and the values that travel with them: the expression VLOAD of the index idx_) are
// fetched together, because the rounds are short and otherwise each would wait for its own
// global load.  BODY sees the key k, its index idx, `valid` and the value vv.
#define GRAM_LOAD_BATCH(IT0, KB, VB, VLOAD)                                                         \
    _Pragma("unroll") for (int u = 0; u < kSortBatch; ++u) {                                        \
        const int64_t idx_ = base + (int64_t)((IT0) + u) * kWave + lane;                            \
        const bool in_ = (IT0) + u < items && idx_ < n;                                             \
        KB[u] = in_ ? keys_in[idx_] : 0;                                                            \
        VB[u] = in_ ? (VLOAD) : 0;                                                                  \
    }
#define GRAM_RUN_BATCH(IT0, KB, VB, BODY)                                                           \
    _Pragma("unroll") for (int u = 0; u < kSortBatch; ++u) {                                        \
        if ((IT0) + u >= items) break; /* wave-uniform */                                           \
        const int64_t idx = base + (int64_t)((IT0) + u) * kWave + lane;                             \
        const bool valid = idx < n;                                                                 \
        int k = KB[u];                                                                              \
        const int vv = VB[u];                                                                       \
        (void)vv;                                                                                   \
        BODY                                                                                        \
    }
#define GRAM_FOR_WAVE_KEYS(BODY)                                                                    \
    for (int it0 = 0; it0 < items; it0 += kSortBatch) {                                             \
        int kb_[kSortBatch], vb_[kSortBatch];                                                       \
        GRAM_LOAD_BATCH(it0, kb_, vb_, 0)                                                           \
        GRAM_RUN_BATCH(it0, kb_, vb_, BODY)                                                         \
    }
// The same walk with the first batch already in registers (KB0, VB0).
#define GRAM_FOR_WAVE_KEYS_FROM(KB0, VB0, VLOAD, BODY)                                              \
    for (int it0 = 0; it0 < items; it0 += kSortBatch) {                                             \
        int kb_[kSortBatch], vb_[kSortBatch];                                                       \
        if (it0 == 0) {                                                                             \
            _Pragma("unroll") for (int u = 0; u < kSortBatch; ++u) {                                \
                kb_[u] = KB0[u];                                                                    \
                vb_[u] = VB0[u];                                                                    \
            }                                                                                       \
        } else {                                                                                    \
            GRAM_LOAD_BATCH(it0, kb_, vb_, VLOAD)                                                   \
        }                                                                                           \
        GRAM_RUN_BATCH(it0, kb_, vb_, BODY)                                                         \
    }

// Digit histogram of one pass per block.  table[block * bins + digit] = count: a block stores, and in the
// scatter reads, one row of it (a column cost 1024 separate cache lines each way).
template <bool CHECK>
__global__ __launch_bounds__(kBlock) void k_radix_hist(const int* __restrict__ keys_in, int n_host,
                                                       const int* __restrict__ n_dev, int shift,
                                                       int dbits, int items,
                                                       int* __restrict__ table, int vocab_n,
                                                       int fix_key, int* __restrict__ err)
{
    __shared__ int cnt[1 << kMaxDigitBits];
    const int n = n_dev ? *n_dev : n_host;
    const int wave = wave_id(), lane = lane_id();
    const int bins = 1 << dbits;
    for (int b = threadIdx.x; b < bins; b += kBlock) cnt[b] = 0;
    __syncthreads();
    const int64_t base = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * items * kWave;
    bool bad = false;
    GRAM_FOR_WAVE_KEYS(
        if (valid) {
            if (CHECK && (k < 0 || k >= vocab_n)) { bad = true; k = fix_key; }
            atomicAdd(&cnt[(k >> shift) & (bins - 1)], 1);
        })
    if (CHECK && bad) atomicOr(err, kErrBitRange);
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += kBlock) table[(int64_t)blockIdx.x * bins + b] = cnt[b];
}

// Exclusive prefix over the blocks' counts of every digit (in place), digit totals to gtot.  A block
// takes 64 digits, one per lane; its 16 waves share the rows of the table, and up to 16 rows each are
// fetched together (256 blocks in all, i.e. batches of up to 4 million keys; beyond that in several turns).
constexpr int kScanWaves = 16;
__global__ __launch_bounds__(kScanWaves * kWave) void k_radix_scan(int* __restrict__ table, int nb, int bins,
                                                                   int* __restrict__ gtot)
{
    __shared__ int part[kScanWaves][kWave];
    constexpr int kPer = 16;
    const int lane = lane_id(), g = wave_id();
    const int b = blockIdx.x * kWave + lane;
    const bool ok = b < bins;
    int carry = 0;
    for (int row0 = 0; row0 < nb; row0 += kScanWaves * kPer) {
        const int rows = nb - row0 < kScanWaves * kPer ? nb - row0 : kScanWaves * kPer;
        const int per = (rows + kScanWaves - 1) / kScanWaves;
        const int r0 = g * per, r1 = r0 + per < rows ? r0 + per : rows;
        int* col = table + (int64_t)row0 * bins + b;
        int v[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) v[i] = ok && r0 + i < r1 ? col[(int64_t)(r0 + i) * bins] : 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) sum += v[i];
        __syncthreads();
        part[g][lane] = sum;
        __syncthreads();
        int run = carry;
#pragma unroll
        for (int w = 0; w < kScanWaves; ++w) {
            const int s = part[w][lane];
            if (w < g) run += s;
            carry += s;
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (ok && r0 + i < r1) {
                col[(int64_t)(r0 + i) * bins] = run;
                run += v[i];
            }
    }
    if (ok && g == 0) gtot[b] = carry;
}

// Stable scatter of one pass.  The block recounts its keys per wave, turns the counts into the
// first output slot of every (wave, digit), then each wave walks its chunk in rounds of 64 keys:
// lanes holding the same digit find each other with one ballot per digit bit and take consecutive
// slots in lane order.
template <bool CHECK>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const int* __restrict__ keys_in, const int* __restrict__ vals_in, int n_host,
    const int* __restrict__ n_dev, int shift, int dbits, int items,
    const int* __restrict__ table, const int* __restrict__ gtot, int* __restrict__ keys_out,
    int* __restrict__ vals_out, int vocab_n, int fix_key)
{
    __shared__ int digit_base[1 << kMaxDigitBits];
    __shared__ int cnt_s[kWavesPerBlock][1 << kMaxDigitBits];
    __shared__ int sm[kWavesPerBlock];
    const int n = n_dev ? *n_dev : n_host;
    const int wave = wave_id(), lane = lane_id();
    const int bins = 1 << dbits;
    const int64_t base = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * items * kWave;

    // Everything this block reads that does not depend on its own work is fetched first, in one
    // round trip: the first batch of its keys and values (kept for both walks below), its row
    // of the block table and the digit totals.
    int kb0[kSortBatch], vb0[kSortBatch];
    GRAM_LOAD_BATCH(0, kb0, vb0, (vals_in ? vals_in[idx_] : (int)idx_))
    static_assert((1 << kMaxDigitBits) <= 4 * kBlock, "a thread holds at most 4 digits of the block table");
    int tb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = threadIdx.x + i * kBlock;
        tb[i] = b < bins ? table[(int64_t)blockIdx.x * bins + b] : 0;
    }

    for (int b = threadIdx.x; b < bins; b += kBlock)
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) cnt_s[w][b] = 0;
    {   // exclusive scan of the digit totals, 4 digits per thread
        int v[4], s = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = threadIdx.x * 4 + i;
            v[i] = b < bins ? gtot[b] : 0;
            s += v[i];
        }
        int total;
        int run = block_excl_scan(s, &total, sm);      // contains barriers: cnt_s is zero after it
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = threadIdx.x * 4 + i;
            if (b < bins) digit_base[b] = run;
            run += v[i];
        }
    }
    GRAM_FOR_WAVE_KEYS_FROM(kb0, vb0, 0,
        if (valid) {
            if (CHECK && (k < 0 || k >= vocab_n)) k = fix_key;
            atomicAdd(&cnt_s[wave][(k >> shift) & (bins - 1)], 1);
        })
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = threadIdx.x + i * kBlock;
        if (b < bins) {
            int o = digit_base[b] + tb[i];
#pragma unroll
            for (int w = 0; w < kWavesPerBlock; ++w) {
                const int cw = cnt_s[w][b];
                cnt_s[w][b] = o;
                o += cw;
            }
        }
    }
    __syncthreads();

    volatile lds_i32* cnt = (volatile lds_i32*)cnt_s[wave];
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    GRAM_FOR_WAVE_KEYS_FROM(kb0, vb0, (vals_in ? vals_in[idx_] : (int)idx_),
        if (CHECK && valid && (k < 0 || k >= vocab_n)) k = fix_key;
        const int v = vv;
        const int dg = (k >> shift) & (bins - 1);
        unsigned long long peers = __ballot(valid);
        for (int bit = 0; bit < dbits; ++bit) {
            const bool one = (dg >> bit) & 1;
            const unsigned long long mm = __ballot(one);
            peers &= one ? mm : ~mm;
        }
        const int below = __popcll(peers & lt_mask);
        int pos = 0;
        if (valid) pos = cnt[dg] + below;
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) cnt[dg] = pos + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
        if (valid && (unsigned)pos < (unsigned)n) {     // pos < n always holds; the test keeps a
            keys_out[pos] = k;                           // logic error from becoming a stray store
            vals_out[pos] = v;
        })
}
#undef GRAM_FOR_WAVE_KEYS
#undef GRAM_FOR_WAVE_KEYS_FROM
#undef GRAM_LOAD_BATCH
#undef GRAM_RUN_BATCH

int radix_sort_pairs(Ctx* c, const int* keys_in, const int* vals_in, int n_host, const int* n_dev,
                     int64_t n_max, bool check_range, int fix_key, hipStream_t s)
{
    const SortPlan p = make_sort_plan(c->key_bits, n_max);
    const int* kin = keys_in;
    const int* vin = vals_in;
    int shift = 0, dst = 0;
    for (int pass = 0; pass < p.passes; ++pass) {
        const int db = p.digit_bits[pass];
        const int bins = 1 << db;
        const bool chk = check_range && pass == 0;
        if (chk)
            launch(c, KID_RADIX_HIST, k_radix_hist<true>, dim3(p.blocks), dim3(kBlock), s, kin, n_host,
                               n_dev, shift, db, p.items, c->table, c->cfg.vocab_n, fix_key,
                               c->scal + kSErr);
        else
            launch(c, KID_RADIX_HIST, k_radix_hist<false>, dim3(p.blocks), dim3(kBlock), s, kin, n_host,
                               n_dev, shift, db, p.items, c->table, 0, 0, c->scal + kSErr);
        launch(c, KID_RADIX_SCAN, k_radix_scan, dim3((bins + kWave - 1) / kWave), dim3(kScanWaves * kWave), s, c->table,
               p.blocks, bins, c->gtot);
        if (chk)
            launch(c, KID_RADIX_SCATTER, k_radix_scatter<true>, dim3(p.blocks), dim3(kBlock), s, kin, vin,
                               n_host, n_dev, shift, db, p.items, c->table, c->gtot,
                               c->keys[dst], c->vals[dst], c->cfg.vocab_n, fix_key);
        else
            launch(c, KID_RADIX_SCATTER, k_radix_scatter<false>, dim3(p.blocks), dim3(kBlock), s, kin, vin,
                               n_host, n_dev, shift, db, p.items, c->table, c->gtot,
                               c->keys[dst], c->vals[dst], 0, 0);
        kin = c->keys[dst];
        vin = c->vals[dst];
        shift += db;
        dst ^= 1;
    }
    return dst ^ 1;
}

// ---- head flags -> uniq / inverse / offsets / counts / prospective buffer rows ----

__device__ __forceinline__ bool is_head(const int* __restrict__ sk, int r)
{
    return r == 0 || sk[r] != sk[r - 1];
}

// Two launches over tiles of kScanTile sorted rows.  The first leaves four figures per tile
// (tile_info[t], [T + t], [2 T + t], [3 T + t] with T tiles): the number of segment heads in the tile,
// how many of those items have no row in the window's buffer yet, and the rows of the tile's first and
// last head (-1: none).  The second turns them into everything that is known per unique item:
// uniq, offsets, counts (a head's segment ends at the next head, which may lie tiles ahead: the
// third figure finds it), the inverse index, per sorted row its segment with the flags of the segment
// reduction (the segment of a tile's first rows may have started tiles before: the fourth figure), and - when the context keeps a slot table - the
// buffer row each item WOULD get from the next gram_grad_accumulate (seg_slot: its row, or for
// an item new to the window the next free row with kSlotNew set, in ascending-ID order, or -1
// when the buffer is full).  Nothing of the slot table is written here: the accumulate step
// commits those rows, provided the table has not changed in between.
__device__ __forceinline__ int block_min(int v, int* sm)
{
    v = wave_min(v);
    if (lane_id() == 0) sm[wave_id()] = v;
    __syncthreads();
    int m = sm[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) m = sm[w] < m ? sm[w] : m;
    __syncthreads();
    return m;
}

constexpr int kNoRow = 0x7fffffff;

__global__ __launch_bounds__(kBlock) void k_heads_count(const int* __restrict__ sk, int n,
                                                        const int* __restrict__ slot_of,
                                                        int* __restrict__ tile_info, int first_step,
                                                        int* __restrict__ scal)
{
    __shared__ int sm[kWavesPerBlock];
    const int r0 = blockIdx.x * kScanTile + threadIdx.x * 4;
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[kSPadSeg] = -1;      // the emit launch sets it if there is padding
    int s = 0, fresh = 0, first = kNoRow, last = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (r0 + i < n && is_head(sk, r0 + i)) {
            ++s;
            if (first == kNoRow) first = r0 + i;
            last = r0 + i;
            // (in the first step of a window the buffer holds nothing: every item is new)
            if (slot_of && (first_step || slot_of[sk[r0 + i]] < 0)) ++fresh;
        }
    const int tot = block_sum(s | fresh << 16, sm);        // (at most kScanTile each)
    const int row = block_min(first, sm), end_row = -block_min(-last, sm);
    if (threadIdx.x == 0) {
        tile_info[blockIdx.x] = tot & 0xffff;
        tile_info[gridDim.x + blockIdx.x] = tot >> 16;
        tile_info[2 * gridDim.x + blockIdx.x] = row == kNoRow ? -1 : row;
        tile_info[3 * gridDim.x + blockIdx.x] = end_row;
    }
}

__global__ __launch_bounds__(kBlock) void k_heads_emit(
    const int* __restrict__ sk, const int* __restrict__ sv, int n, const int* __restrict__ tile_info,
    int* __restrict__ uniq, int* __restrict__ inverse, int* __restrict__ counts,
    int* __restrict__ offsets, int* __restrict__ seg_of_row, int* __restrict__ uniq_ws,
    int* __restrict__ u_out, const int* __restrict__ slot_of, int* __restrict__ seg_slot,
    int* __restrict__ scal, int first_step, int cap_total, int pad_id)
{
    __shared__ int sm[kWavesPerBlock];
    __shared__ int s_rows[kScanTile + 1];     // rows of the tile's heads, then the next head's row
    __shared__ int s_next;
    const int T = gridDim.x;
    // Everything that does not depend on this block's own work is fetched before the first
    // barrier, in one round trip: the thread's 4 sorted keys and positions, the key before them,
    // the figures of the tiles before and (a first look) after this one, the buffer's row count.
    const int r0 = blockIdx.x * kScanTile + threadIdx.x * 4;
    int key[4] = {0, 0, 0, 0}, posn[4] = {0, 0, 0, 0};
    if (r0 + 3 < n) {           // whole groups of 4: 16-byte loads (the arrays are 256-byte aligned)
        const int4 k4 = *reinterpret_cast<const int4*>(sk + r0);
        const int4 p4 = *reinterpret_cast<const int4*>(sv + r0);
        key[0] = k4.x; key[1] = k4.y; key[2] = k4.z; key[3] = k4.w;
        posn[0] = p4.x; posn[1] = p4.y; posn[2] = p4.z; posn[3] = p4.w;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (r0 + i < n) {
                key[i] = sk[r0 + i];
                posn[i] = sv[r0 + i];
            }
    }
    const int prev = (r0 > 0 && r0 < n) ? sk[r0 - 1] : -1;
    const int u_base = (slot_of && !first_step) ? scal[kSUTotal] : 0;   // a flush leaves the old count behind
    const int ahead0 = (int)blockIdx.x + 1 + (int)threadIdx.x < T ? tile_info[2 * T + blockIdx.x + 1 + threadIdx.x] : -1;
    int pre = 0, pre_fresh = 0, before = -1;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kBlock) {
        pre += tile_info[t];
        pre_fresh += tile_info[T + t];
        const int h = tile_info[3 * T + t];
        before = h > before ? h : before;
    }
    bool f[4];
    int old[4];
    int s = 0, fresh = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[i] = (r0 + i < n) && (r0 + i == 0 || key[i] != (i ? key[i - 1] : prev));
        old[i] = 0;
        s += f[i] ? 1 : 0;
        if (f[i] && slot_of) {
            old[i] = first_step ? -1 : slot_of[key[i]];
            fresh += old[i] < 0 ? 1 : 0;
        }
    }
    pre = block_sum(pre, sm);
    pre_fresh = block_sum(pre_fresh, sm);
    before = -block_min(-before, sm);        // the last head before this tile (head rows ascend)
    const int long_rows = seg_rows_for(n);
    if (threadIdx.x == 0) s_next = kNoRow;
    int total;      // both counts in one scan: at most kScanTile each
    int local = block_excl_scan(s | fresh << 16, &total, sm);
    const int local_fresh = local >> 16, total_fresh = total >> 16;
    local &= 0xffff;
    total &= 0xffff;
    {
        int li = local;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (f[i]) s_rows[li++] = r0 + i;
    }
    // the first head after this tile: the tiles ahead are looked at kBlock at a time (their first
    // heads ascend with the tile index, so the minimum is the nearest)
    for (int base = blockIdx.x + 1; base < T; base += kBlock) {
        const int t = base + threadIdx.x;
        const int row = base == (int)blockIdx.x + 1 ? ahead0 : (t < T ? tile_info[2 * T + t] : -1);
        if (row >= 0) atomicMin(&s_next, row);
        __syncthreads();
        if (s_next != kNoRow) break;           // the same value for every thread
        __syncthreads();
    }
    __syncthreads();
    if (threadIdx.x == 0) s_rows[total] = s_next == kNoRow ? n : s_next;
    __syncthreads();

    int run = pre + local, li = local, next_slot = u_base + pre_fresh + local_fresh;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = r0 + i;
        if (r < n) {
            run += f[i] ? 1 : 0;
            const int seg = run - 1;
            // li heads of the tile lie before row r: s_rows[li - 1] (this row, if it is one) starts its
            // segment, s_rows[li] the next one
            const int li_in = li + (f[i] ? 1 : 0);
            const int start = li_in > 0 ? s_rows[li_in - 1] : before;
            seg_of_row[r] = seg | (f[i] ? kRowHead : 0) | (s_rows[li_in] - start >= long_rows ? kRowLong : 0);
            inverse[posn[i]] = seg;
            if (f[i]) {
                if (key[i] == pad_id) scal[kSPadSeg] = seg;
                uniq[seg] = key[i];
                uniq_ws[seg] = key[i];
                offsets[seg] = r;
                counts[seg] = s_rows[li + 1] - r;
                ++li;
                if (slot_of) {
                    int code = old[i];
                    if (code < 0) {
                        const int slot = next_slot++;
                        code = slot < cap_total ? (slot | kSlotNew) : -1;
                    }
                    seg_slot[seg] = code;
                }
            }
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const int u = pre + total;
        scal[kSU] = u;
        if (u_out) *u_out = u;
        offsets[u] = n;
        scal[kSLongCount] = 0;
        if (slot_of) {
            const int nt = u_base + pre_fresh + total_fresh;
            scal[kSUNext] = nt < cap_total ? nt : cap_total;
        }
    }
}

__global__ void k_unique_empty(int* u_ws, int* u_out, int* offsets)
{
    if (threadIdx.x == 0) {
        *u_ws = 0;
        if (u_out) *u_out = 0;
        offsets[0] = 0;
    }
}

// ---- small batches: ranks by comparison ----------------------------------------------
//
// Up to kSmallMaxN positions (12,000: 26 us against 32 to 35 us for the radix sort; 16,384: 34 against 32 to
// 36).  The sorted place of a position is the number of positions whose
// (id, position) pair is smaller, and that number is counted outright: every position against every
// other, two VALU instructions per pair.  n^2 comparisons spread over the whole chip are cheaper at
// these sizes than sorting on one CU (a radix sort in the LDS of one block: 21 us at n = 6,400 with 14
// key bits, 28 us at n = 7,040 with 17; here 14.7 us for both) and than a radix sort over many blocks (8
// launches, about 36 us).  What bounds k_rank_small is the VALU: 4.7 of its 10 us at n = 6,400 are
// comparisons, the rest is the launch and the loads of the IDs.  Two launches:
//   k_rank_small  kRankP positions per block, 1024 threads: thread (p, slice) compares position p
//                 with the 16-byte groups slice, slice + S, ... of all IDs, which the block holds in
//                 LDS; the counts of the slices are added and (id, position) goes to its place;
//   k_emit_small  head flags of the sorted IDs, their scan, and everything that is known per
//                 position and per unique item; every block works out the flags of all rows and
//                 writes its own 1024 rows and items.
// Batches of at most kFusedMaxN positions do both in one block and one launch (3.9 us at n = 64, where the
// LDS radix sort took 7.3; at 512 the two launches take as long as the one).
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kFusedMaxN = 512;
constexpr int kRankP = 32;

// Exclusive scan of one value per thread over the 1024-thread block.
__device__ __forceinline__ int block1024_excl_scan(int v, int* total, int* wsum /*[kSmallWaves]*/)
{
    const int incl = wave_incl_scan(v);
    if (lane_id() == kWave - 1) wsum[wave_id()] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
        const int t = wsum[w];
        if (w < wave_id()) base += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return base + incl - v;
}

// IDs of the batch into LDS (checked; a multiple of 4 entries, the rest larger than any ID).  FRESH: the error
// word is written, not added to (contains a barrier).
template <bool FRESH>
__device__ __forceinline__ void load_small_ids(const int* __restrict__ ids, int n, int vocab_n, int fix_key,
                                               int* __restrict__ err, bool report, int* keys)
{
    const int n4 = (n + 3) & ~3;
    bool bad = false;
    for (int i0 = 0; i0 < n4; i0 += 8 * kSmallThreads) {
        int k[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kSmallThreads + threadIdx.x;
            k[u] = i < n ? ids[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * kSmallThreads + threadIdx.x;
            if (i >= n4) break;
            if (i >= n) k[u] = 0x7fffffff;
            else if (k[u] < 0 || k[u] >= vocab_n) { bad = true; k[u] = fix_key; }
            keys[i] = k[u];
        }
    }
    if (FRESH) {
        const int any = __syncthreads_or(bad);
        if (report && threadIdx.x == 0) *err = any ? kErrBitRange : 0;
    } else if (report && bad) {
        atomicOr(err, kErrBitRange);
    }
}

// Rank of position p0 + (tid % P) of the n keys in LDS, P = 1 << log2p positions per block; valid in
// threads tid < P.  red: kSmallThreads ints of LDS.  Contains barriers.
__device__ __forceinline__ int rank_by_comparison(const int* keys, int n, int p0, int log2p, int* red)
{
    const int tid = threadIdx.x, P = 1 << log2p, S = kSmallThreads >> log2p;
    const int p = p0 + (tid & (P - 1)), slice = tid >> log2p;
    const int groups = (n + 3) >> 2, own = p >> 2;
    const int key = keys[p < n ? p : n - 1];
    const int4* k4 = reinterpret_cast<const int4*>(keys);
    int cnt = 0;
    // an equal ID counts if its position is smaller: groups before the position's own are compared
    // with key + 1 (IDs are below 2^31 - 1), later ones with key
#pragma unroll 4
    for (int g = slice; g < groups; g += S) {
        const int4 q = k4[g];
        const int t = key + (g < own ? 1 : 0);
        cnt += (q.x < t ? 1 : 0) + (q.y < t ? 1 : 0) + (q.z < t ? 1 : 0) + (q.w < t ? 1 : 0);
    }
    red[tid] = cnt;
    __syncthreads();
    int rank = 0;
    if (tid < P) {
#pragma unroll 8
        for (int s = 0; s < S; ++s) rank += red[(s << log2p) + tid];
        for (int q = own << 2; q < p && q < n; ++q) rank += keys[q] == key ? 1 : 0;
    }
    return rank;
}

template <bool FRESH>
__global__ __launch_bounds__(kSmallThreads) void k_rank_small(const int* __restrict__ ids, int n, int vocab_n,
                                                              int fix_key, int* __restrict__ scal,
                                                              int* __restrict__ sorted_keys, int* __restrict__ perm)
{
    extern __shared__ __attribute__((aligned(16))) int lds[];
    __shared__ int red[kSmallThreads];
    constexpr int kLog2P = 5;
    static_assert(1 << kLog2P == kRankP, "positions per block");
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[kSPadSeg] = -1;      // the emit launch sets it if there is padding
    load_small_ids<FRESH>(ids, n, vocab_n, fix_key, scal + kSErr, blockIdx.x == 0, lds);
    __syncthreads();
    const int p0 = blockIdx.x * kRankP;
    const int rank = rank_by_comparison(lds, n, p0, kLog2P, red);
    const int p = p0 + (int)threadIdx.x;
    if ((int)threadIdx.x < kRankP && p < n && (unsigned)rank < (unsigned)n) {   // rank < n always holds;
        sorted_keys[rank] = lds[p];                                             // the test keeps a logic error
        perm[rank] = p;                                                         // from becoming a stray store
    }
}

// R sorted rows per thread (n <= 1024 R).  FUSED: the ranks are worked out here too (one block).
template <int R, bool FUSED, bool FRESH>
__global__ __launch_bounds__(kSmallThreads) void k_emit_small(
    const int* __restrict__ ids, int n, int log2p, int vocab_n, int fix_key, int* __restrict__ err,
    const int* __restrict__ sorted_keys, int* __restrict__ perm, int* __restrict__ uniq,
    int* __restrict__ inverse, int* __restrict__ counts, int* __restrict__ offsets,
    int* __restrict__ seg_of_row, int* __restrict__ uniq_ws, int* __restrict__ u_ws,
    int* __restrict__ u_out, const int* __restrict__ slot_of, int* __restrict__ seg_slot,
    int* __restrict__ scal, int first_step, int cap_total, int pad_id)
{
    constexpr int NR = kSmallThreads * R;
    // sorted IDs | segment of every row (16-bit) | first row of every segment (16-bit)
    extern __shared__ __attribute__((aligned(16))) int sk[];
    __shared__ int wsum[kSmallWaves];
    uint16_t* lseg = reinterpret_cast<uint16_t*>(sk + NR);
    uint16_t* loff = lseg + NR;
    const int tid = threadIdx.x;
    const int r0 = tid * R;
    const int row = blockIdx.x * kSmallThreads + tid;       // the row and the item this thread writes
    int key[R], posn = 0;
    if constexpr (FUSED) {
        static_assert(R == 1, "one row per thread");
        __shared__ __attribute__((aligned(16))) int kin[kFusedMaxN];
        __shared__ int red[kSmallThreads], pos_of[kFusedMaxN];
        load_small_ids<FRESH>(ids, n, vocab_n, fix_key, err, true, kin);
        if (tid == 0) scal[kSPadSeg] = -1;
        __syncthreads();
        const int rank = rank_by_comparison(kin, n, 0, log2p, red);
        if (tid < n && (unsigned)rank < (unsigned)n) {
            sk[rank] = kin[tid];
            pos_of[rank] = tid;
        }
        __syncthreads();
        key[0] = tid < n ? sk[tid] : 0;
        if (tid < n) {
            posn = pos_of[tid];
            perm[tid] = posn;
        }
    } else {
        if (r0 + R <= n) {
#pragma unroll
            for (int i = 0; i < R / 4; ++i) {
                const int4 k = *reinterpret_cast<const int4*>(sorted_keys + r0 + 4 * i);
                key[4 * i] = k.x; key[4 * i + 1] = k.y; key[4 * i + 2] = k.z; key[4 * i + 3] = k.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) key[i] = r0 + i < n ? sorted_keys[r0 + i] : 0;
        }
        if (row < n) posn = perm[row];
#pragma unroll
        for (int i = 0; i < R / 4; ++i)
            *reinterpret_cast<int4*>(sk + r0 + 4 * i) = make_int4(key[4 * i], key[4 * i + 1], key[4 * i + 2], key[4 * i + 3]);
        __syncthreads();
    }
    const int u_base = (slot_of && !first_step) ? scal[kSUTotal] : 0;    // a flush leaves the old count behind
    const int prev = r0 > 0 && r0 < n ? sk[r0 - 1] : -1;
    bool f[R];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int r = r0 + i;
        f[i] = r < n && (r == 0 || key[i] != (i ? key[i - 1] : prev));
        sum += f[i] ? 1 : 0;
    }
    int total;
    int run = block1024_excl_scan(sum, &total, wsum);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        run += f[i] ? 1 : 0;
        lseg[r0 + i] = (uint16_t)(run - 1);
        if (f[i]) loff[run - 1] = (uint16_t)(r0 + i);
    }
    __syncthreads();
    if (row < n) {
        const int seg = lseg[row], start = loff[seg], end = seg + 1 < total ? (int)loff[seg + 1] : n;
        seg_of_row[row] = seg | (row == start ? kRowHead : 0) | (end - start >= seg_rows_for(n) ? kRowLong : 0);
        inverse[posn] = seg;
    }
    if (row < total) {
        const int r = loff[row];
        const int k = sk[r];
        uniq[row] = k;
        uniq_ws[row] = k;
        if (k == pad_id) scal[kSPadSeg] = row;
        offsets[row] = r;
        counts[row] = (row + 1 < total ? (int)loff[row + 1] : n) - r;
    }
    if (blockIdx.x == 0 && tid == 0) {
        *u_ws = total;
        if (u_out) *u_out = total;
        offsets[total] = n;
        scal[kSLongCount] = 0;
    }
    // the buffer rows the items would get from the next gram_grad_accumulate (see k_heads_emit).  In
    // the first step of a window the buffer holds nothing: item j gets row j.  Later thread t looks up
    // items R t .. R t + R - 1, one scan ranks the items new to the window.
    if (!slot_of) return;
    int nt = total;
    if (first_step) {
        if (row < total) seg_slot[row] = row < cap_total ? (row | kSlotNew) : -1;
    } else {
        int old[R], fresh = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) old[i] = r0 + i < total ? slot_of[sk[loff[r0 + i]]] : 0;
#pragma unroll
        for (int i = 0; i < R; ++i) fresh += old[i] < 0 ? 1 : 0;
        int total_fresh;
        int next_slot = u_base + block1024_excl_scan(fresh, &total_fresh, wsum);
        nt = u_base + total_fresh;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            int code = old[i];
            if (code < 0) {
                const int slot = next_slot++;
                code = slot < cap_total ? (slot | kSlotNew) : -1;
            }
            // (each block writes the codes of its own items)
            if (r0 + i < total && (unsigned)(r0 + i - (int)blockIdx.x * kSmallThreads) < (unsigned)kSmallThreads)
                seg_slot[r0 + i] = code;
        }
    }
    if (blockIdx.x == 0 && tid == 0) scal[kSUNext] = nt < cap_total ? nt : cap_total;
}

// ---- small and mid-sized batches: one launch -----------------------------------------------
//
// The two launches of the comparison ranks and the three of the counting dedup below are short ones, each a chain of
// a few round trips.  Up to kOnceMaxM positions one launch does it all, because every block can afford to read all IDs
// (held in registers): it counts them by key in LDS, those of the positions before its own slice first, then its slice
// (whose positions' places among their ID's positions are thereby known), then the rest.  A scan over the keys gives
// every key its first row and its number among the items; each thread of the slice writes what is known of its position
// and, if it is its ID's first, of the item.  Nothing passes between blocks.
//   BITS = false: the key is the ID (16-bit counts of all IDs in LDS: up to about 56,000, less for small batches).
//   BITS = true:  a bitmap of the IDs that occur is made first and the key is the ID's number among them: any
//                 vocabulary whose bitmap and its prefix fit (0.19 bytes per ID: 524,288), up to kOnceBitsM positions.
// What bounds it is the LDS atomic per ID, about 30 to 45 cycles per wave (lanes of a wave that meet on a bank): nothing at
// 6,400 positions, most of the time at 50,000.  Lanes that meet on one counter wait for each other, about 130 cycles where all 64
// do, so the first of a thread's four positions that hold one ID counts them all.  16,384 positions over 13,000 IDs, first step, an
// atomic per position / four equal ones together / any equal ones together (three launches): one item 20.1 / 10.0 / 9.9 us (10.9),
// half of them one item 13.7 / 13.1 / 10.2 (11.5), two items 14.3 / 13.6 / 10.4 (11.0), Zipf 1.2 10.0 / 9.9 / 9.4 (11.6), uniform 7.9 / 8.1 / 8.5
// (12.7).  (Finding equal lanes of a wave by ballots costs every batch 0.3 to 1 us.)
// Whole call, ranks or counting dedup / one launch: 1,000 positions 8.1 / 6.3 us, 6,400 over 13,000 IDs 13.3 / 6.6, 7,040 over 100,000 14.0 / 9.8, 12,000 over 300,000 26.7 / 12.9, 16,000 over 20,000
// 12.3 / 10.6, 25,600 12.7 / 14.1 (padded histories 12.9 / 10.8), 51,200 13.8 / 23.3: the line lies at 16,384.
// Small batches over large vocabularies go by the bitmap, which passes over IDs that do not occur sooner, in later steps all
// the more (by ID, every block looks at every ID's slot): 520 positions over 50,000 IDs, by ID / by bitmap, first step 7.5 / 6.7,
// later 10.8 / 7.8 (in two launches 8.3); later, 2,048 over 20,000 8.5 / 8.1, 4,000 over 50,000 11.1 / 9.2; 4,000 in a first step
// 7.9 / 7.8, with many equal IDs 9.1 / 9.6.
// Later steps of what the counting dedup takes too (from 8,193 positions) are left to it where the look-ups cost more than its two
// launches: one launch / counting, 10,000 positions over 50,000 IDs Zipf 0.9 to 1.2 12.3 to 13.4 / 12.4, over 100,000 uniform
// 16.7 / 14.5, 12,000 19.4 / 14.8; over 30,000 10.5 to 11.7 / 11.4, 16,384 over 13,000 9.8 to 11.8 / 11.2.
// The outputs must not overlap the IDs (other blocks still read those): such calls take the ways below.
// (constants of the counting dedup)
constexpr int kCountThreads = 1024;
constexpr int kCountIds = 65536;             // IDs per part: 128 KiB of 16-bit counters
constexpr int kCountTile = 128;              // IDs per block of k_ids_scan
constexpr int kCountTilesMax = kCountMaxVocab / kCountTile;

constexpr int kOnceThreads = 1024, kOnceWaves = kOnceThreads / kWave;
constexpr int kOnceMaxM = 16384, kOnceBitsM = 12288;
constexpr int kOnceLaterIds = 40960;         // in later steps, where the counting dedup takes the batch too
constexpr int kOnceSlice = 256;              // positions per block, at most
constexpr int kOnceRounds = 8;               // groups of 8 keys per thread, at most
constexpr size_t kOnceLds = 156 * 1024;      // dynamic; beside it 3 KiB

struct OnceLayout {              // byte offsets of the arrays in LDS; groups of 8 keys, words of the bitmap
    int groups, words, dummy, base, base_f, mask, bits, bits_pre;
    size_t bytes;
    __host__ __device__ OnceLayout(bool by_bits, bool slots, int n, int vocab_n)
    {
        groups = ((by_bits ? n : vocab_n) + 7) / 8;
        words = by_bits ? (int)((vocab_n + 127ll) / 128 * 4) : 0;
        dummy = groups * 16;                                 // [64] words that count padding, one per lane
        base = dummy + kWave * 4;                            // [groups] first row | items before << 16
        base_f = base + groups * 4;                          // [groups] new items before
        mask = base_f + (slots ? (groups * 2 + 3) / 4 * 4 : 0);      // [groups] a bit per key: a new item
        bits = (mask + (slots ? groups : 0) + 15) / 16 * 16;
        bits_pre = bits + words * 4;                         // [words] items before
        bytes = (size_t)bits_pre + (size_t)words * 2;
    }
};

// Exclusive scan over rounds of one value per thread (round r before round r + 1, threads in order): v[r] becomes the sum
// ahead of it; returns the total.  sm: [kOnceRounds * kOnceWaves].  Contains barriers.
template <int ROUNDS>
__device__ __forceinline__ uint32_t once_scan(uint32_t (&v)[ROUNDS], uint32_t* sm)
{
    static_assert(ROUNDS * kOnceWaves <= 2 * kWave, "two values per lane");
    const int lane = lane_id(), wave = wave_id();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t incl = (uint32_t)wave_incl_scan((int)v[r]);
        if (lane == kWave - 1) sm[r * kOnceWaves + wave] = incl;
        v[r] = incl - v[r];
    }
    __syncthreads();
    const int a = lane < ROUNDS * kOnceWaves ? (int)sm[lane] : 0;
    const int b = lane + kWave < ROUNDS * kOnceWaves ? (int)sm[lane + kWave] : 0;
    const int ia = wave_incl_scan(a), ta = __builtin_amdgcn_readlane(ia, kWave - 1), ib = wave_incl_scan(b) + ta;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int at = __builtin_amdgcn_readfirstlane(r * kOnceWaves + wave);
        v[r] += (uint32_t)(at == 0 ? 0 : at <= kWave ? __builtin_amdgcn_readlane(ia, at - 1) : __builtin_amdgcn_readlane(ib, at - 1 - kWave));
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(ib, kWave - 1);
    __syncthreads();
    return total;
}

// R: groups of 4 positions per thread.  SLOTS: the buffer may hold items already (slot_of is looked at; else, where it is
// given, item j gets row j).  fresh_err: the error word is written, not added to.
template <int R, bool BITS, bool SLOTS>
__global__ __launch_bounds__(kOnceThreads) void k_ids_once(
    const int* __restrict__ ids, int n, int slice, int key_bits, int vocab_n, int fix_key, int fresh_err, int* __restrict__ perm, int* __restrict__ uniq,
    int* __restrict__ inverse, int* __restrict__ counts, int* __restrict__ offsets, int* __restrict__ seg_of_row,
    int* __restrict__ uniq_ws, int* __restrict__ u_out, const int* __restrict__ slot_of, int* __restrict__ seg_slot,
    int* __restrict__ scal, int cap_total, int pad_id)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char once_lds[];
    __shared__ __attribute__((aligned(16))) int own[kOnceSlice];
    __shared__ uint32_t sm[kOnceRounds * kOnceWaves];
    typedef int v4a __attribute__((ext_vector_type(4), aligned(4)));
    const OnceLayout lo(BITS, SLOTS, n, vocab_n);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(once_lds);
    uint32_t* base = reinterpret_cast<uint32_t*>(once_lds + lo.base);
    uint16_t* base_f = reinterpret_cast<uint16_t*>(once_lds + lo.base_f);
    unsigned char* mask = once_lds + lo.mask;
    uint32_t* bits = reinterpret_cast<uint32_t*>(once_lds + lo.bits);
    uint16_t* bits_pre = reinterpret_cast<uint16_t*>(once_lds + lo.bits_pre);
    const int tid = threadIdx.x, lane = lane_id();
    const int p_lo = blockIdx.x * slice, p_hi = p_lo + slice < n ? p_lo + slice : n;      // slice: a multiple of 4
    const int g_lo = p_lo >> 2, g_hi = (p_hi + 3) >> 2;

    // the IDs, checked: thread t holds groups t, t + 1024, ... of 4 positions
    int k[R][4];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = (tid + r * kOnceThreads) * 4;
        if (p + 3 < n) {
            const v4a q = *reinterpret_cast<const v4a*>(ids + p);
            k[r][0] = q.x; k[r][1] = q.y; k[r][2] = q.z; k[r][3] = q.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) k[r][c] = p + c < n ? ids[p + c] : 0;      // (checked, then marked: -1)
        }
    }
    const int u_base = SLOTS ? scal[kSUTotal] : 0;
    for (int i = tid; i < lo.base / 16; i += kOnceThreads) reinterpret_cast<uint4*>(cnt)[i] = make_uint4(0, 0, 0, 0);
    if (BITS) {
        for (int i = tid; i < lo.words / 4; i += kOnceThreads) reinterpret_cast<uint4*>(bits)[i] = make_uint4(0, 0, 0, 0);
        if (SLOTS)
            for (int i = tid; i < (lo.groups + 3) / 4; i += kOnceThreads) reinterpret_cast<uint32_t*>(mask)[i] = 0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if ((unsigned)k[r][c] >= (unsigned)vocab_n) {
                k[r][c] = fix_key;
                bad = true;
            }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if ((tid + r * kOnceThreads) * 4 + 3 >= n)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if ((tid + r * kOnceThreads) * 4 + c >= n) k[r][c] = -1;       // (no position)
    if (blockIdx.x == 0) {              // (it has seen all of them)
        if (fresh_err) {
            const int any = __syncthreads_or(bad);
            if (tid == 0) scal[kSErr] = any ? kErrBitRange : 0;
        } else if (bad) {
            atomicOr(&scal[kSErr], kErrBitRange);
        }
    }
    if (!BITS && SLOTS) {
        // which of a group's 8 IDs have no row in the buffer
        for (int g = tid; g < lo.groups; g += kOnceThreads) {
            uint32_t m = 0;
            if (8 * g + 7 < vocab_n) {
                const int4 a = *reinterpret_cast<const int4*>(slot_of + 8 * g), b = *reinterpret_cast<const int4*>(slot_of + 8 * g + 4);
                m = (uint32_t)a.x >> 31 | (uint32_t)a.y >> 31 << 1 | (uint32_t)a.z >> 31 << 2 | (uint32_t)a.w >> 31 << 3 |
                    (uint32_t)b.x >> 31 << 4 | (uint32_t)b.y >> 31 << 5 | (uint32_t)b.z >> 31 << 6 | (uint32_t)b.w >> 31 << 7;
            } else {
                for (int i = 0; i < 8; ++i)
                    if (8 * g + i < vocab_n && slot_of[8 * g + i] < 0) m |= 1u << i;
            }
            mask[g] = (unsigned char)m;
        }
    }
    // the slice's IDs (tid < p_hi - p_lo: one position per thread)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int g = tid + r * kOnceThreads;
        if (g >= g_lo && g < g_hi) *reinterpret_cast<int4*>(own + 4 * (g - g_lo)) = make_int4(k[r][0], k[r][1], k[r][2], k[r][3]);
    }
    __syncthreads();
    const int p = p_lo + tid;
    const bool mine = p < p_hi;
    int id = mine ? own[tid] : 0, key = id, pad_key = pad_id;
    if (BITS) {
        // the bitmap, the number of IDs before each of its words, and every ID's number
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int v = k[r][c], first = __builtin_amdgcn_readfirstlane(v);
                const unsigned long long pads = __ballot(v == pad_id);
                const bool same = __ballot(v == first) == ~0ull;
                if (v >= 0 && (v == pad_id ? lane == __builtin_ctzll(pads) : !same || lane == 0)) atomicOr(&bits[v >> 5], 1u << (v & 31));
            }
        __syncthreads();
        constexpr int kWordRounds = 4;
        uint32_t pre[kWordRounds];
#pragma unroll
        for (int r = 0; r < kWordRounds; ++r) {
            const int w = tid + r * kOnceThreads;
            uint4 q = make_uint4(0, 0, 0, 0);
            if (w < lo.words / 4) q = reinterpret_cast<const uint4*>(bits)[w];
            pre[r] = __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
        }
        once_scan(pre, sm);
#pragma unroll
        for (int r = 0; r < kWordRounds; ++r) {
            const int w = tid + r * kOnceThreads;
            if (w < lo.words / 4) {
                const uint4 q = reinterpret_cast<const uint4*>(bits)[w];
                const uint32_t b1 = pre[r] + __popc(q.x), b2 = b1 + __popc(q.y), b3 = b2 + __popc(q.z);
                reinterpret_cast<uint2*>(bits_pre)[w] = make_uint2(pre[r] | b1 << 16, b2 | b3 << 16);
            }
        }
        __syncthreads();
        auto number = [&](int v) { return (int)(bits_pre[v >> 5] + __popc(bits[v >> 5] & ((1u << (v & 31)) - 1u))); };
        if (pad_id >= 0) pad_key = bits[pad_id >> 5] >> (pad_id & 31) & 1 ? number(pad_id) : -1;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int v = k[r][c];
                if (v < 0) continue;
                k[r][c] = number(v);
                if (SLOTS && slot_of[v] < 0) atomicOr(reinterpret_cast<uint32_t*>(mask) + (k[r][c] >> 5), 1u << (k[r][c] & 31));
            }
        key = number(id);
    }

    // Padding, and what is no position, goes to a counter per lane: on one word its many positions would wait for each other.
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (k[r][c] == pad_key || k[r][c] < 0) k[r][c] = lo.groups * 8 + lane * 2;
    auto count_groups = [&](int from, int to) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int g = tid + r * kOnceThreads;
            if (g < from || g >= to) continue;
            // (the first of a thread's equal keys adds for all of them)
            const int k0 = k[r][0], k1 = k[r][1], k2 = k[r][2], k3 = k[r][3];
            const bool e01 = k0 == k1, e02 = k0 == k2, e03 = k0 == k3, e12 = k1 == k2, e13 = k1 == k3, e23 = k2 == k3;
            const uint32_t add[4] = {1u + e01 + e02 + e03, e01 ? 0u : 1u + e12 + e13, e02 || e12 ? 0u : 1u + e23, e03 || e13 || e23 ? 0u : 1u};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (add[c]) atomicAdd(&cnt[k[r][c] >> 1], add[c] << ((uint32_t)k[r][c] << 4 & 31u));
        }
    };
    count_groups(0, g_lo);
    __syncthreads();
    // The slice: lanes of a wave with the same key find each other by ballots, the waves take turns at the counters in
    // position order.
    typedef __attribute__((address_space(3))) uint16_t lds_u16;
    volatile lds_u16* cnt16 = (volatile lds_u16*)(lds_u16*)once_lds;
    unsigned long long peers = __ballot(mine);
    int at = 0;
    if (tid < kOnceSlice)
        for (int bit = 0; bit < key_bits; ++bit) {
            const bool one = (key >> bit) & 1;
            const unsigned long long mm = __ballot(one);
            peers &= one ? mm : ~mm;
        }
    const int below = __popcll(peers & ((1ull << lane) - 1ull));
    const int pads_ahead = wave_sum((int)cnt[lo.dummy / 4 + lane]);
    if (tid == 0 && pad_key >= 0 && pads_ahead) cnt16[pad_key] = (uint16_t)pads_ahead;
    for (int w = 0; w * kWave < slice; ++w) {
        if (w == wave_id() && mine) {
            at = cnt16[key];
            __builtin_amdgcn_wave_barrier();
            if (below == 0) cnt16[key] = (uint16_t)(at + (int)__popcll(peers));
        }
        __syncthreads();
    }
    at += below;
    count_groups(g_hi, (n + 3) >> 2);
    __syncthreads();
    const int pads_behind = wave_sum((int)cnt[lo.dummy / 4 + lane]) - pads_ahead - (g_hi << 2 < n ? -n & 3 : 0);

    // first row, number among the items and among the new items of every group of 8 keys
    constexpr int kRounds = BITS ? 2 : kOnceRounds;
    auto occurring = [](uint4 q) {          // a bit per key of the group that occurs
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) m |= (w[i] & 0xffffu ? 1u << (2 * i) : 0u) | (w[i] >> 16 ? 2u << (2 * i) : 0u);
        return m;
    };
    uint32_t sum[kRounds], fresh[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int g = tid + r * kOnceThreads;
        sum[r] = fresh[r] = 0;
        if (g < lo.groups) {
            uint4 q = reinterpret_cast<const uint4*>(cnt)[g];
            if (pad_key >= 0 && g == pad_key >> 3) {
                const uint32_t add = (uint32_t)pads_behind << ((pad_key & 1) * 16);
                const int w = pad_key >> 1 & 3;
                q.x += w == 0 ? add : 0u; q.y += w == 1 ? add : 0u; q.z += w == 2 ? add : 0u; q.w += w == 3 ? add : 0u;
                reinterpret_cast<uint4*>(cnt)[g] = q;
            }
            const uint32_t occ = occurring(q), c2 = q.x + q.y + q.z + q.w;      // (two 16-bit sums: at most 65,535 in all)
            sum[r] = (c2 & 0xffffu) + (c2 >> 16) + ((uint32_t)__popc(occ) << 16);
            if (SLOTS) fresh[r] = __popc(occ & mask[g]);
        }
    }
    const int items = (int)(once_scan(sum, sm) >> 16);
    int fresh_all = 0;
    if (SLOTS) fresh_all = (int)once_scan(fresh, sm);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int g = tid + r * kOnceThreads;
        if (g < lo.groups) {
            base[g] = sum[r];
            if (SLOTS) base_f[g] = (uint16_t)fresh[r];
        }
    }
    __syncthreads();

    if (mine) {
        const int g = key >> 3, i = key & 7;
        const uint4 q = reinterpret_cast<const uint4*>(cnt)[g];
        const uint32_t w[4] = {q.x, q.y, q.z, q.w}, below_i = occurring(q) & ((1u << i) - 1u);
        int first_row = (int)(base[g] & 0xffffu), count = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int c = (int)(w[j >> 1] >> ((j & 1) * 16) & 0xffffu);
            first_row += j < i ? c : 0;
            count = j == i ? c : count;
        }
        const int seg = (int)(base[g] >> 16) + __popc(below_i), pos = first_row + at;
        inverse[p] = seg;
        if ((unsigned)pos < (unsigned)n) {      // pos < n always holds; the test keeps a logic error from
            perm[pos] = p;                       // becoming a stray store
            seg_of_row[pos] = seg | (at == 0 ? kRowHead : 0) | (count >= seg_rows_for(n) ? kRowLong : 0);
        }
        if (at == 0) {
            uniq[seg] = id;
            uniq_ws[seg] = id;
            if (id == pad_id) scal[kSPadSeg] = seg;
            offsets[seg] = first_row;
            counts[seg] = count;
            if (slot_of) {
                int slot = SLOTS ? slot_of[id] : -1;
                if (slot < 0) {
                    const int s = SLOTS ? u_base + base_f[g] + __popc(below_i & mask[g]) : seg;
                    slot = s < cap_total ? (s | kSlotNew) : -1;
                }
                seg_slot[seg] = slot;
            }
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
        scal[kSU] = items;
        if (u_out) *u_out = items;
        offsets[items] = n;
        scal[kSLongCount] = 0;
        if (pad_id < 0 || (BITS ? pad_key < 0 : cnt16[pad_id] == 0)) scal[kSPadSeg] = -1;     // (else its first position sets it)
        if (slot_of) {
            const int nt = SLOTS ? u_base + fresh_all : items;
            scal[kSUNext] = nt < cap_total ? nt : cap_total;
        }
    }
}

static bool overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return a && b && x < y + (uintptr_t)b_bytes && y < x + (uintptr_t)a_bytes;
}

static bool counting_takes(const Ctx* c, int n)
{
    const int64_t N = c->cfg.vocab_n;
    if (!c->cnt_table || n < kCountMinM || n > kCountMaxM || N > kCountMaxVocab) return false;
    const int64_t rows = (n + kCountThreads - 1) / kCountThreads, pitch = (N + kCountTile - 1) / kCountTile * kCountTile;
    return rows * pitch / 2 <= kCountMaxWords;
}

// Returns false where the one-launch dedup does not apply.
bool unique_once(Ctx* c, const int* ids, int n, int fix_key, int* uniq, int* inverse, int* counts, int* u_out,
                 hipStream_t s, bool prospect, int first_step)
{
    if (n <= kFusedMaxN || n > kOnceMaxM) return false;
    const int N = c->cfg.vocab_n;
    const bool slots = prospect && !first_step;
    if (slots && N > kOnceLaterIds && counting_takes(c, n)) return false;
    const int most_by_id = n > (slots ? 4096 : 2048) ? 8 * kOnceRounds * kOnceThreads : slots && n <= 2048 ? 16384 : 32768;
    const bool by_id = N <= most_by_id && OnceLayout(false, slots, n, N).bytes <= kOnceLds;
    const bool by_bits = !by_id && n <= kOnceBitsM && N <= 128 * 4 * kOnceThreads && OnceLayout(true, slots, n, N).bytes <= kOnceLds;
    if (!by_id && !by_bits) return false;
    const int64_t ids_bytes = (int64_t)n * 4, items_bytes = (int64_t)(n < N ? n : N) * 4;
    if (overlap(ids, ids_bytes, uniq, items_bytes) || overlap(ids, ids_bytes, counts, items_bytes) || overlap(ids, ids_bytes, inverse, ids_bytes) ||
        overlap(ids, ids_bytes, u_out, 4))
        return false;
    c->sorted_keys = nullptr;
    c->perm = c->vals[0];
    int slice = ((n + c->num_cus - 1) / c->num_cus + 3) & ~3;
    slice = slice < kWave ? kWave : slice > kOnceSlice ? kOnceSlice : slice;
    const OnceLayout lo(by_bits, slots, n, N);
    int key_bits = 1;
    while (((by_bits ? n : N) - 1) >> key_bits) ++key_bits;
    auto go = [&](auto kern) {
        launch_smem(c, KID_IDS_ONCE, kern, dim3((unsigned)((n + slice - 1) / slice)), dim3(kOnceThreads), lo.bytes, s, ids, n, slice,
                    key_bits, N, fix_key, c->fresh_err ? 1 : 0, c->perm, uniq, inverse, counts, c->offsets, c->seg_of_row, c->uniq_ws, u_out,
                    prospect ? c->slot_of : (const int*)nullptr, c->seg_slot, c->scal, (int)c->cap_total, c->cfg.pad_id);
    };
#define GRAM_GO(R, BITS)                                                                            \
    {                                                                                               \
        ensure_dynamic_lds<k_ids_once<R, BITS, true>>((int)kOnceLds);                               \
        ensure_dynamic_lds<k_ids_once<R, BITS, false>>((int)kOnceLds);                              \
        if (slots) go(k_ids_once<R, BITS, true>);                                                   \
        else go(k_ids_once<R, BITS, false>);                                                        \
    }
    constexpr int kPer = 4 * kOnceThreads;
    static_assert(kOnceBitsM <= 3 * kPer && kOnceMaxM <= 4 * kPer, "positions per thread");
    if (by_bits && n <= 2 * kPer) GRAM_GO(2, true)
    else if (by_bits) GRAM_GO(3, true)
    else if (n <= 2 * kPer) GRAM_GO(2, false)
    else GRAM_GO(4, false)
#undef GRAM_GO
    return true;
}

// ---- mid-sized batches over small vocabularies: counting by ID -------------------------
//
// A sort of such a batch is bound by its eight short launches (two radix passes of three, two for the
// head flags: 33 to 37 us from 12,000 to 65,000 positions whatever the vocabulary).  Where a counter
// per ID fits in LDS, three launches do it all:
//   k_ids_count  a block counts the IDs of its 1024 positions in LDS (16-bit counters) and leaves them
//                as one row of table[block][id], every position's rank among its block's positions of the ID, and the
//                checked IDs where k_ids_emit reads them (the caller's buffer of IDs may be one of the outputs: a launch
//                that writes those does not read it);
//   k_ids_scan   exclusive prefix down every column of the table (a block takes 128 IDs), and per ID
//                its count and its place among the positions, items and new items of its 128 IDs;
//   k_ids_emit   position blocks: place of a position = first row of its ID + the column prefix + its rank;
//                ID blocks: everything per unique item.  The first launch has the counters in LDS anyway; with the ranks worked out
//                here, in blocks of 1024, this one took 7.9 us at 51,200 positions over 20,000 IDs, now 4.8.
// Vocabularies beyond kCountIds are cut into parts: a block then takes (1024 positions, one part).
// 16-bit counts and prefixes hold because a batch has fewer than 65,536 positions.  Batches below kCountMinM
// are as fast ranked by comparison, in a launch less (whole call, 50,000 IDs: 8,192 positions 14.7 us ranked,
// 14.3 counted; 6,400 positions 13.5 and 14.2; 4,096 11.1 and 14.0; 12,000 26 and 14.5); up to 16,384 positions both are left
// with what the one launch above does not take.
static_assert(kCountTilesMax % kBlock == 0, "tiles per thread in the scan of k_ids_emit");
static_assert(kCountMaxM < 65536, "16-bit prefixes");

int64_t count_table_words(int64_t vocab_n, int64_t max_positions)
{
    if (vocab_n > kCountMaxVocab || max_positions < kCountMinM) return 0;
    const int64_t m = max_positions < kCountMaxM ? max_positions : kCountMaxM;
    const int64_t rows = (m + kCountThreads - 1) / kCountThreads, pitch = (vocab_n + kCountTile - 1) / kCountTile * kCountTile;
    int64_t words = rows * pitch / 2;
    return words > kCountMaxWords ? kCountMaxWords : words;
}

// A position's ID; one outside [0, vocab_n) is replaced and reported.
__device__ __forceinline__ int count_id(int raw, int vocab_n, int fix_key, bool* bad)
{
    if (raw < 0 || raw >= vocab_n) {
        *bad = true;
        return fix_key;
    }
    return raw;
}

__global__ __launch_bounds__(kCountThreads) void k_ids_count(const int* __restrict__ ids, int n, int key_bits, int vocab_n,
                                                             int fix_key, int pitch, int* __restrict__ scal,
                                                             uint32_t* __restrict__ table, int* __restrict__ checked, int* __restrict__ ranks)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t cnt[];
    const int tid = threadIdx.x, lane = lane_id(), lo = blockIdx.y * kCountIds;
    const int words = (pitch - lo < kCountIds ? pitch - lo : kCountIds) / 2;      // a multiple of 64
    const int p = blockIdx.x * kCountThreads + tid;
    const int raw = p < n ? ids[p] : 0;
    for (int i = tid * 4; i < words; i += kCountThreads * 4) *reinterpret_cast<uint4*>(cnt + i) = make_uint4(0, 0, 0, 0);
    bool bad = false;
    const int key = count_id(raw, vocab_n, fix_key, &bad), id = key - lo;
    if (blockIdx.y == 0 && p < n) checked[p] = key;
    const bool mine = p < n && (unsigned)id < (unsigned)(2 * words);
    if (bad && p < n) atomicOr(scal + kSErr, kErrBitRange);
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) scal[kSPadSeg] = -1;    // k_ids_emit sets it if there is padding
    // rank among the block's positions of the same ID: lanes of a wave find each other by ballots, the waves take
    // turns at the counters in position order
    unsigned long long peers = __ballot(mine);
    for (int bit = 0; bit < key_bits; ++bit) {
        const bool one = (key >> bit) & 1;
        const unsigned long long mm = __ballot(one);
        peers &= one ? mm : ~mm;
    }
    const int below = __popcll(peers & ((1ull << lane) - 1ull));
    typedef __attribute__((address_space(3))) uint16_t lds_u16;
    volatile lds_u16* cnt16 = (volatile lds_u16*)(lds_u16*)cnt;
    int before = 0;
    __syncthreads();
    for (int w = 0; w < kCountThreads / kWave; ++w) {
        if (w == wave_id() && mine) {
            before = cnt16[id];
            __builtin_amdgcn_wave_barrier();
            if (below == 0) cnt16[id] = (uint16_t)(before + (int)__popcll(peers));
        }
        __syncthreads();
    }
    if (mine) ranks[p] = before + below;
    uint32_t* row = table + ((int64_t)blockIdx.x * pitch + lo) / 2;
    for (int i = tid * 4; i < words; i += kCountThreads * 4)
        *reinterpret_cast<uint4*>(row + i) = *reinterpret_cast<const uint4*>(cnt + i);
}

// Per ID: x = first row within the tile (16 bits) | items before it in the tile (8) | new items before
// it (8); y = its count.  tile_info[t], [T + t], [2 T + t]: positions, items, new items of tile t.
__global__ __launch_bounds__(kBlock) void k_ids_scan(uint32_t* __restrict__ table, int rows, int pitch,
                                                     const int* __restrict__ slot_of, int first_step, int vocab_n,
                                                     uint2* __restrict__ id_info, int* __restrict__ tile_info)
{
    constexpr int kGroups = kBlock / (kCountTile / 2);       // 4 groups of threads share the rows of a column
    constexpr int kRowsMax = (kCountMaxM + kCountThreads - 1) / kCountThreads;
    constexpr int kPer = (kRowsMax + kGroups - 1) / kGroups;
    __shared__ uint32_t part[kGroups][kCountTile / 2];
    const int w = threadIdx.x & (kCountTile / 2 - 1), g = threadIdx.x / (kCountTile / 2);
    const int word = blockIdx.x * (kCountTile / 2) + w;
    uint32_t* col = table + word;
    const int64_t step = pitch / 2;
    const int per = (rows + kGroups - 1) / kGroups;
    const int b0 = g * per, b1 = b0 + per < rows ? b0 + per : rows;
    const int id = 2 * word;
    int slot0 = -1, slot1 = -1;
    if (g == 0 && slot_of && !first_step) {
        if (id < vocab_n) slot0 = slot_of[id];
        if (id + 1 < vocab_n) slot1 = slot_of[id + 1];
    }
    // all of a thread's counts are fetched together; two 16-bit sums per word never carry into each other
    uint32_t v[kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) v[i] = b0 + i < b1 ? col[(b0 + i) * step] : 0u;
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum += v[i];
    part[g][w] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const uint32_t t = part[i][w];
        if (i < g) run += t;
        tot += t;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        if (b0 + i < b1) {
            col[(b0 + i) * step] = run;
            run += v[i];
        }
    if (g != 0) return;
    // the first wave: 2 IDs per lane
    static_assert(kCountTile == 2 * kWave, "the tile's IDs sit in one wave");
    const int c0 = (int)(tot & 0xffffu), c1 = (int)(tot >> 16);
    const int h0 = c0 > 0, h1 = c1 > 0, n0 = h0 && slot0 < 0, n1 = h1 && slot1 < 0;
    const int pos = wave_incl_scan(c0 + c1);
    const int hn = wave_incl_scan((h0 + h1) | (n0 + n1) << 16);
    const int pos0 = pos - c0 - c1, hd0 = (hn & 0xffff) - h0 - h1, nw0 = (hn >> 16) - n0 - n1;
    uint2* out = id_info + id;          // two entries as one 16-byte store (id is even)
    *reinterpret_cast<uint4*>(out) =
        make_uint4((uint32_t)pos0 | (uint32_t)hd0 << 16 | (uint32_t)nw0 << 24, (uint32_t)c0,
                   (uint32_t)((pos0 + c0) & 0xffff) | (uint32_t)(hd0 + h0) << 16 | (uint32_t)(nw0 + n0) << 24, (uint32_t)c1);
    if (w == kWave - 1) {
        const int T = gridDim.x;
        tile_info[blockIdx.x] = pos;
        tile_info[T + blockIdx.x] = hn & 0xffff;
        tile_info[2 * T + blockIdx.x] = hn >> 16;
    }
}

constexpr int kEmitTiles = kCountTilesMax / kBlock;      // tiles per thread in the scan of k_ids_emit

__global__ __launch_bounds__(kBlock) void k_ids_emit(
    const int* __restrict__ checked, const int* __restrict__ ranks, int n, int vocab_n, int pitch, int pos_blocks,
    const uint16_t* __restrict__ table, const uint2* __restrict__ id_info, const int* __restrict__ tile_info, int T,
    int* __restrict__ perm, int* __restrict__ uniq, int* __restrict__ inverse, int* __restrict__ counts,
    int* __restrict__ offsets, int* __restrict__ seg_of_row, int* __restrict__ uniq_ws, int* __restrict__ u_out,
    const int* __restrict__ slot_of, int* __restrict__ seg_slot, int* __restrict__ scal, int first_step,
    int cap_total, int pad_id)
{
    __shared__ int s_pos[kCountTilesMax], s_item[kCountTilesMax], s_new[kCountTilesMax];
    __shared__ unsigned long long s_wave[kWavesPerBlock];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const bool per_id = (int)blockIdx.x >= pos_blocks;

    // what does not depend on the scan of the tiles is fetched first
    const int p = blockIdx.x * kBlock + tid;                       // position blocks
    const int j = ((int)blockIdx.x - pos_blocks) * kBlock + tid;   // ID blocks
    const bool mine = per_id ? j < vocab_n : p < n;
    int id = 0, at = 0, slot = -1;
    uint2 info = make_uint2(0, 0);
    if (mine) {
        id = per_id ? j : checked[p];
        if (!per_id) at = ranks[p];
        info = id_info[id];
        if (per_id && slot_of && !first_step) slot = slot_of[j];
        if (!per_id) at += table[(int64_t)(p / kCountThreads) * pitch + id];
    }
    const int u_base = (slot_of && !first_step) ? scal[kSUTotal] : 0;     // a flush leaves the old count behind
    // exclusive prefix over the tiles, three figures of at most 17 bits in one 64-bit sum
    unsigned long long tv[kEmitTiles], sum = 0;
#pragma unroll
    for (int i = 0; i < kEmitTiles; ++i) {
        const int t = tid * kEmitTiles + i;
        tv[i] = t < T ? (unsigned long long)tile_info[t] | (unsigned long long)tile_info[T + t] << 20 |
                            (unsigned long long)tile_info[2 * T + t] << 40 : 0ull;
        sum += tv[i];
    }
    const unsigned long long incl = (unsigned long long)(unsigned)wave_incl_scan((int)(sum & 0xfffff)) |
                                    (unsigned long long)(unsigned)wave_incl_scan((int)(sum >> 20 & 0xfffff)) << 20 |
                                    (unsigned long long)(unsigned)wave_incl_scan((int)(sum >> 40)) << 40;
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    unsigned long long base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
        const unsigned long long t = s_wave[w];
        if (w < wave) base += t;
        all += t;
    }
    base += incl - sum;
#pragma unroll
    for (int i = 0; i < kEmitTiles; ++i) {
        const int t = tid * kEmitTiles + i;
        if (t < T) {
            s_pos[t] = (int)(base & 0xfffff);
            s_item[t] = (int)(base >> 20 & 0xfffff);
            s_new[t] = (int)(base >> 40);
        }
        base += tv[i];
    }
    __syncthreads();
    const int tile = id / kCountTile;
    const int first_row = s_pos[tile] + (int)(info.x & 0xffff), seg = s_item[tile] + (int)(info.x >> 16 & 0xff);

    if (per_id) {
        if (info.y > 0) {                                                 // the ID occurs
            uniq[seg] = id;
            uniq_ws[seg] = id;
            if (id == pad_id) scal[kSPadSeg] = seg;
            offsets[seg] = first_row;
            counts[seg] = (int)info.y;
            if (slot_of) {
                if (slot < 0) {
                    const int s = u_base + s_new[tile] + (int)(info.x >> 24);
                    slot = s < cap_total ? (s | kSlotNew) : -1;
                }
                seg_slot[seg] = slot;
            }
        }
        if (j == 0) {
            const int u = (int)(all >> 20 & 0xfffff);
            scal[kSU] = u;
            if (u_out) *u_out = u;
            offsets[u] = n;
            scal[kSLongCount] = 0;
            if (slot_of) {
                const int nt = u_base + (int)(all >> 40);
                scal[kSUNext] = nt < cap_total ? nt : cap_total;
            }
        }
    } else if (mine) {
        const int pos = first_row + at;
        inverse[p] = seg;
        if ((unsigned)pos < (unsigned)n) {      // pos < n always holds; the test keeps a logic error from
            perm[pos] = p;                       // becoming a stray store
            seg_of_row[pos] = seg | (at == 0 ? kRowHead : 0) | ((int)info.y >= seg_rows_for(n) ? kRowLong : 0);
        }
    }
}

// Returns false where the counting dedup does not apply: a vocabulary or batch beyond its counters, or
// a table larger than kCountMaxWords (its four trips through memory then cost more than the launches saved).
bool unique_by_count(Ctx* c, const int* ids, int n, int fix_key, int* uniq, int* inverse, int* counts, int* u_out,
                     hipStream_t s, bool prospect, int first_step)
{
    if (!counting_takes(c, n)) return false;
    const int64_t N = c->cfg.vocab_n;
    const int pitch = (int)((N + kCountTile - 1) / kCountTile * kCountTile);
    const int rows = (n + kCountThreads - 1) / kCountThreads;
    const int parts = (pitch + kCountIds - 1) / kCountIds, T = pitch / kCountTile;
    const size_t lds = (size_t)(pitch < kCountIds ? pitch : kCountIds) * 2;
    ensure_dynamic_lds<k_ids_count>(kCountIds * 2);
    const int* slot_of = prospect ? c->slot_of : nullptr;
    c->sorted_keys = nullptr;
    c->perm = c->vals[0];
    launch_smem(c, KID_IDS_COUNT, k_ids_count, dim3(rows, parts), dim3(kCountThreads), lds, s, ids, n, c->key_bits, c->cfg.vocab_n,
                fix_key, pitch, c->scal, c->cnt_table, c->keys[0], c->keys[1]);
    launch(c, KID_IDS_SCAN, k_ids_scan, dim3(T), dim3(kBlock), s, c->cnt_table, rows, pitch, slot_of, first_step,
           c->cfg.vocab_n, c->id_info, c->id_tiles);
    const int pos_blocks = (n + kBlock - 1) / kBlock, id_blocks = (int)((N + kBlock - 1) / kBlock);
    launch(c, KID_IDS_EMIT, k_ids_emit, dim3(pos_blocks + id_blocks), dim3(kBlock), s, c->keys[0], c->keys[1], n,
           c->cfg.vocab_n, pitch, pos_blocks, reinterpret_cast<const uint16_t*>(c->cnt_table), c->id_info,
           c->id_tiles, T, c->perm, uniq, inverse, counts, c->offsets, c->seg_of_row, c->uniq_ws, u_out, slot_of,
           c->seg_slot, c->scal, first_step, (int)c->cap_total, c->cfg.pad_id);
    return true;
}

// prospect: also work out the buffer rows the items would get (slot-table contexts only);
// first_step: the window's buffer holds nothing yet.
void unique_from_sorted(Ctx* c, int n, int* uniq, int* inverse, int* counts, int* u_out,
                        hipStream_t s, bool prospect, int first_step)
{
    if (n == 0) {
        launch(c, KID_UNIQUE_EMPTY, k_unique_empty, dim3(1), dim3(kWave), s, c->scal + kSU, u_out, c->offsets);
        return;
    }
    const int tiles = (n + kScanTile - 1) / kScanTile;
    const int* slot_of = prospect ? c->slot_of : nullptr;
    launch(c, KID_HEADS_COUNT, k_heads_count, dim3(tiles), dim3(kBlock), s, c->sorted_keys, n, slot_of,
           c->tile_sums, first_step, c->scal);
    launch(c, KID_HEADS_EMIT, k_heads_emit, dim3(tiles), dim3(kBlock), s, c->sorted_keys, c->perm, n,
           c->tile_sums, uniq, inverse, counts, c->offsets, c->seg_of_row, c->uniq_ws, u_out, slot_of,
           c->seg_slot, c->scal, first_step, (int)c->cap_total, c->cfg.pad_id);
}

template <int R, bool FUSED, bool FRESH = false>
static void launch_emit_small(Ctx* c, const int* ids, int n, int log2p, int fix_key, int* uniq, int* inverse,
                              int* counts, int* u_out, hipStream_t s, bool prospect, int first_step)
{
    constexpr size_t lds = (size_t)kSmallThreads * R * 8;
    constexpr auto kern = k_emit_small<R, FUSED, FRESH>;
    ensure_dynamic_lds<kern>((int)lds);
    const unsigned blocks = (unsigned)((n + kSmallThreads - 1) / kSmallThreads);
    launch_smem(c, KID_UNIQUE_SMALL, kern, dim3(blocks), dim3(kSmallThreads), lds, s, ids, n, log2p, c->cfg.vocab_n,
                fix_key, c->scal + kSErr, c->sorted_keys, c->perm, uniq, inverse, counts, c->offsets, c->seg_of_row,
                c->uniq_ws, c->scal + kSU, u_out, prospect ? c->slot_of : nullptr, c->seg_slot, c->scal, first_step,
                (int)c->cap_total, c->cfg.pad_id);
}

bool unique_small(Ctx* c, const int* ids, int n, int fix_key, int* uniq, int* inverse, int* counts,
                  int* u_out, hipStream_t s, bool prospect, int first_step)
{
    if (n <= 0 || n > kSmallMaxN) return false;
    c->sorted_keys = c->keys[0];
    c->perm = c->vals[0];
    if (n <= kFusedMaxN) {
        int log2p = 6;
        while ((1 << log2p) < n) ++log2p;
        if (c->fresh_err) launch_emit_small<1, true, true>(c, ids, n, log2p, fix_key, uniq, inverse, counts, u_out, s, prospect, first_step);
        else launch_emit_small<1, true>(c, ids, n, log2p, fix_key, uniq, inverse, counts, u_out, s, prospect, first_step);
        return true;
    }
    const size_t lds = (size_t)((n + 3) & ~3) * sizeof(int);
    auto rank = [&](auto kern) {
        launch_smem(c, KID_RANK_SMALL, kern, dim3((unsigned)((n + kRankP - 1) / kRankP)), dim3(kSmallThreads), lds, s,
                    ids, n, c->cfg.vocab_n, fix_key, c->scal, c->sorted_keys, c->perm);
    };
    ensure_dynamic_lds<k_rank_small<false>>(kSmallMaxN * (int)sizeof(int));
    ensure_dynamic_lds<k_rank_small<true>>(kSmallMaxN * (int)sizeof(int));
    if (c->fresh_err) rank(k_rank_small<true>);
    else rank(k_rank_small<false>);
    if (n <= 8 * kSmallThreads)
        launch_emit_small<8, false>(c, ids, n, 0, fix_key, uniq, inverse, counts, u_out, s, prospect, first_step);
    else
        launch_emit_small<kSmallMaxN / kSmallThreads, false>(c, ids, n, 0, fix_key, uniq, inverse, counts, u_out, s, prospect, first_step);
    return true;
}

}  // namespace gram
