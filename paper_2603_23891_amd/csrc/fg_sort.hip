// Gaussian-tile key emission, (tile, depth) ordering and per-tile ranges.
//
// The required order is ascending (tile id, depth bits, splat index). It is
// reached with two stable sorts instead of one sort of 64-bit keys:
//
//   1. the splats that cover at least one tile (splats whose shrunk
//      rectangle is empty emit nothing) are radix-sorted by their 32-bit
//      depth key, so ties keep ascending splat index; the first pass reads
//      the selections in (view, index) order and skips the others, which
//      packs the tile-covering splats as it sorts;
//   2. an exclusive prefix scan of their tile counts, taken in that depth
//      order, gives each splat its output offset, and the splat emits one
//      (tile id, splat index) pair per tile of its rectangle;
//   3. the pairs are radix-sorted by tile id only (ceil(log2 tiles) bits),
//      stably, so pairs of one tile keep the depth order of step 1.
//
// Pair traffic drops from ~6 passes over 12-byte (u64 key, u32 value)
// records to 2 passes over 8-byte records at 1080p.
//
// Radix pass (LSD, one digit of BITS bits, stable), up to three kernels:
//   k_hist      per 1024-item tile: digit histogram (LDS atomics) -> hist[digit][tile]
//   k_rowscan   one workgroup per digit: exclusive scan over the tiles,
//               digit totals (few tiles: the scatter sums the rows itself)
//   k_scatter   per tile: stable local ranks (wave ballot match on the digit
//               bits for all of a wave's rounds, then one pass per digit over
//               the per-(round, wave) counts in item order), items staged
//               through LDS in locally sorted order, then written out so that
//               consecutive lanes write consecutive addresses.
// What bounds a pass at a few million items is the latency of its steps and the
// scattered writes (a tile's run of one digit is a few items), so items travel
// as 8-byte {key, value} pairs, one store each, and a digit's output base is
// loaded while the ranks are computed: 15.6 -> 12.4 us per 8-bit depth pass of
// 1.5M splats and 13.6 -> 12.6 per 7-bit tile pass of 1.9M pairs against
// separate key and value stores, 10.5 for the last depth pass, which writes
// values alone.
//
// Block offsets of the emission step are exclusive sums over the per-block
// counts of all earlier blocks. Up to 8192 blocks every block adds them up
// itself (a few thousand L2-resident words), so no scan launch sits between
// counting and writing; larger batches scan the counts in one workgroup
// first. The first blocks in depth order hold the nearest and so the largest
// splats, whose pairs are shared among workgroups in slices.
#include "fg_device.h"
#include "fg_slices.h"

#include <algorithm>

namespace {

constexpr int kThreads = 256;
constexpr int kIPT = 4;
constexpr int kTileItems = kThreads * kIPT;  // 1024
constexpr int kWaves = kThreads / fgd::kWave;
constexpr int kEmitIPT = 4;
constexpr int kEmitItems = kThreads * kEmitIPT;  // 1024
constexpr int kEmitRun = 4;                       // consecutive pairs per thread
constexpr uint32_t kEmitSlice = 2048;             // pairs a workgroup emits at a time

__device__ __forceinline__ int64_t count_of(const uint32_t* p, int64_t cap)
{
    const int64_t n = (int64_t)*p;
    return n < cap ? n : cap;
}

// Exclusive scan of one value per thread over a 256-thread block.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s_wave, uint32_t& total)
{
    const int lane = fgd::lane_id();
    const int wave = threadIdx.x / fgd::kWave;
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < fgd::kWave; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, fgd::kWave);
        if (lane >= d) x += y;
    }
    if (lane == fgd::kWave - 1) s_wave[wave] = x;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
        const uint32_t t = s_wave[w];
        if (w < wave) before += t;
        total += t;
    }
    __syncthreads();
    return before + x - v;
}

// Sum of v[0 .. k) over the workgroup (every thread gets it).
__device__ __forceinline__ unsigned long long block_prefix(const uint32_t* __restrict__ v, int64_t k,
                                                           unsigned long long* s_red)
{
    unsigned long long x = 0;
    for (int64_t i0 = threadIdx.x; i0 < k; i0 += 4 * kThreads) {  // 4 independent loads per step
        uint32_t a[4];
#pragma unroll
        for (int u = 0; u < 4; u++) a[u] = i0 + u * kThreads < k ? v[i0 + u * kThreads] : 0u;
#pragma unroll
        for (int u = 0; u < 4; u++) x += a[u];
    }
#pragma unroll
    for (int d = fgd::kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, fgd::kWave);
    if (fgd::lane_id() == 0) s_red[threadIdx.x / fgd::kWave] = x;
    __syncthreads();
    unsigned long long t = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) t += s_red[w];
    __syncthreads();
    return t;
}

// Block offsets of the emission kernel: either read from counts
// that k_block_scan turned into exclusive offsets, or, when the blocks are few
// enough (kInlineBlocks), summed by every block from the raw counts of the
// blocks before it (L2-resident words), which saves the scan launch; then
// block 0 also stores the total and flags an overflow of cap.
struct BlockOffsets {
    const uint32_t* cnt;
    bool inline_sum;
    uint32_t* total;
    int64_t cap;
    uint32_t* status;
    uint32_t overflow_bit;
};

__device__ __forceinline__ unsigned long long block_offset(const BlockOffsets& o, int64_t blk,
                                                           unsigned long long* s_red)
{
    return o.inline_sum ? block_prefix(o.cnt, blk, s_red) : (unsigned long long)o.cnt[blk];
}

__device__ __forceinline__ void block_total(const BlockOffsets& o, int64_t nblk, unsigned long long* s_red)
{
    if (!o.inline_sum || blockIdx.x != 0) return;
    const unsigned long long t = block_prefix(o.cnt, nblk, s_red);
    if (threadIdx.x == 0) {
        *o.total = (uint32_t)(t < 0xFFFFFFFFull ? t : 0xFFFFFFFFull);
        if ((long long)t > o.cap) atomicOr(o.status, o.overflow_bit);
    }
}

// The views of one call: their splats lie at stride cap_sel in the splat
// planes (view v's splat j is global splat v * cap_sel + j), and their tiles
// have the consecutive global ids tile_base[v] + ty * Wt[v] + tx.
constexpr int kMaxViews = 64;
struct SortViews {
    int n;
    uint32_t cap_sel;
    uint32_t Wt[kMaxViews];
    uint32_t tile_base[kMaxViews];
};

// s_seg[v] = sum over views u < v of min(n_sel[u], cap_sel) (v = 0 .. n): the
// position of view v's first splat among the concatenated selections. Read by
// the first wave; ends with a barrier.
__device__ __forceinline__ void load_segments(const uint32_t* __restrict__ n_sel, const SortViews& V,
                                              uint32_t* s_seg)
{
    if (threadIdx.x < fgd::kWave) {
        const int lane = fgd::lane_id();
        uint32_t c = 0;
        if (lane < V.n) {
            c = n_sel[lane];
            c = c < V.cap_sel ? c : V.cap_sel;
        }
        uint32_t x = c;
#pragma unroll
        for (int d = 1; d < fgd::kWave; d <<= 1) {
            const uint32_t y = __shfl_up(x, d, fgd::kWave);
            if (lane >= d) x += y;
        }
        if (lane == 0) s_seg[0] = 0u;
        if (lane < V.n) s_seg[lane + 1] = x;
    }
    __syncthreads();
}

// Global splat index of concatenated selection item i (i < s_seg[n]).
__device__ __forceinline__ uint32_t item_splat(uint32_t i, const uint32_t* s_seg, const SortViews& V)
{
    int lo = 0, hi = V.n;  // the last view v with s_seg[v] <= i
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_seg[mid] <= i) lo = mid; else hi = mid;
    }
    return (uint32_t)lo * V.cap_sel + (i - s_seg[lo]);
}

// Words of a histogram row: rows start 16-byte aligned.
__device__ __forceinline__ int64_t row_words(int64_t n_tiles) { return (n_tiles + 3) & ~(int64_t)3; }

template <int BITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; b++) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

// Input of the first depth pass: the concatenated selections themselves.
// Item i is global splat g = item_splat(i); it takes part when its rectangle
// covers a tile (tiles[g] != 0), with key = the bits of its depth and value
// g. So the pass also packs the tile-covering splats, in (view, index) order
// within each digit. The histogram kernel clears the tile ranges and stores
// the item count; the scatter stores the packed count and flags an overflow
// of cap_out.
struct SelInput {
    const float4* rgb_depth;
    const uint32_t* tiles;
    const uint32_t* n_sel;
    uint32_t* n_items;  // selection items (written by k_hist)
    unsigned long long* n_slices;  // cleared by k_hist
    uint32_t* n_out;    // packed items (written by k_scatter)
    int64_t cap_out;
    uint32_t* status;
    uint32_t* ranges;
    int64_t n_range_words;
};

// Items of a pass: the selections (the first depth pass), {key, value} pairs,
// or separate key and value arrays; results are pairs, separate arrays, or
// values alone.
enum Form { kSel, kPairs, kSplit, kValues };
struct Items {
    uint2* kv;      // kPairs
    uint32_t* key;  // kSplit
    uint32_t* val;  // kSplit, kValues
};

// Key and value of item idx of a pass (valid: the item takes part).
template <int IN>
__device__ __forceinline__ void pass_item(const Items& in, const SelInput& si, const SortViews& V, const uint32_t* s_seg,
                                          int64_t idx, int64_t n, bool want_val, bool& valid, uint32_t& k,
                                          uint32_t& v)
{
    valid = idx < n;
    k = 0xFFFFFFFFu;
    v = 0u;
    if (!valid) return;
    if constexpr (IN == kSel) {
        const uint32_t g = item_splat((uint32_t)idx, s_seg, V);
        valid = si.tiles[g] != 0u;
        if (valid) {
            k = __float_as_uint(si.rgb_depth[g].w);
            v = g;
        }
    } else if constexpr (IN == kPairs) {
        if (want_val) {
            const uint2 e = in.kv[idx];
            k = e.x;
            v = e.y;
        } else {
            k = in.kv[idx].x;
        }
    } else {
        k = in.key[idx];
        if (want_val) v = in.val[idx];
    }
}

template <int BITS, int IPT, int IN>
__global__ __launch_bounds__(kThreads) void k_hist(Items in, const uint32_t* __restrict__ n_p, int64_t cap, int shift,
                                                   uint32_t* __restrict__ hist, SelInput si, SortViews V)
{
    constexpr int R = 1 << BITS;
    constexpr bool SEL = IN == kSel;
    __shared__ uint32_t h[R];
    __shared__ uint32_t s_seg[SEL ? kMaxViews + 1 : 1];
    int64_t n;
    if constexpr (SEL) {
        for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < si.n_range_words;
             t += (int64_t)gridDim.x * kThreads)
            si.ranges[t] = 0u;
        load_segments(si.n_sel, V, s_seg);
        n = s_seg[V.n];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            *si.n_items = (uint32_t)n;
            *si.n_slices = 0ull;
        }
    } else {
        n = count_of(n_p, cap);
    }
    const int64_t n_tiles = (n + (kThreads * IPT) - 1) / (kThreads * IPT);
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        for (int d = threadIdx.x; d < R; d += kThreads) h[d] = 0;
        __syncthreads();
        // all items are loaded before the first is counted, so that a thread waits
        // once: 12.4 -> 10.1 us for the three 8-bit passes over 176k splats, 6.0 ->
        // 5.2 for the first over 425k selections, 32.0 -> 31.4 and 28.1 -> 26.3 for
        // 2.1M and 4.9M
        uint32_t k[IPT];
        bool valid[IPT];
#pragma unroll
        for (int r = 0; r < IPT; r++) {
            const int64_t idx = tile * (kThreads * IPT) + r * kThreads + threadIdx.x;
            uint32_t v;
            pass_item<IN>(in, si, V, s_seg, idx, n, false, valid[r], k[r], v);
        }
#pragma unroll
        for (int r = 0; r < IPT; r++)
            if (valid[r]) atomicAdd(&h[(k[r] >> shift) & (R - 1)], 1u);
        __syncthreads();
        for (int d = threadIdx.x; d < R; d += kThreads) hist[(int64_t)d * row_words(n_tiles) + tile] = h[d];
        __syncthreads();
    }
}

// One workgroup per digit: exclusive scan of hist[digit][0..n_tiles) in place.
template <int IPT>
__global__ __launch_bounds__(kThreads) void k_rowscan(const uint32_t* __restrict__ n_p, int64_t cap,
                                                      uint32_t* __restrict__ hist, uint32_t* __restrict__ digit_total)
{
    __shared__ uint32_t s_wave[kWaves];
    const int64_t n = count_of(n_p, cap);
    const int64_t n_tiles = (n + (kThreads * IPT) - 1) / (kThreads * IPT);
    uint32_t* row = hist + (int64_t)blockIdx.x * row_words(n_tiles);
    // 8 consecutive words per thread and round, loaded as two vectors (a row is
    // 16-byte aligned and padded; its padding is not counted). Rows of 4200 words:
    // 12.6 us with a contiguous part of the row per thread, 5.9 us this way.
    uint32_t carry = 0;
    for (int64_t base = 0; base < n_tiles; base += 8 * kThreads) {
        uint32_t c[8], s = 0;
        const int64_t i0 = base + 8 * (int64_t)threadIdx.x;
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const int64_t i = i0 + 4 * q;
            const uint4 v = i < n_tiles ? *reinterpret_cast<const uint4*>(row + i) : make_uint4(0u, 0u, 0u, 0u);
            c[4 * q] = v.x;
            c[4 * q + 1] = i + 1 < n_tiles ? v.y : 0u;
            c[4 * q + 2] = i + 2 < n_tiles ? v.z : 0u;
            c[4 * q + 3] = i + 3 < n_tiles ? v.w : 0u;
        }
#pragma unroll
        for (int k = 0; k < 8; k++) s += c[k];
        uint32_t total;
        uint32_t run = carry + block_excl_scan(s, s_wave, total);
#pragma unroll
        for (int q = 0; q < 2; q++) {
            uint4 o;
            o.x = run;
            o.y = o.x + c[4 * q];
            o.z = o.y + c[4 * q + 1];
            o.w = o.z + c[4 * q + 2];
            run = o.w + c[4 * q + 3];
            if (i0 + 4 * q < n_tiles) *reinterpret_cast<uint4*>(row + i0 + 4 * q) = o;
        }
        carry += total;
    }
    if (threadIdx.x == 0) digit_total[blockIdx.x] = carry;
}

template <int BITS, int IPT, int IN, int OUT, bool SUM>
__global__ __launch_bounds__(kThreads) void k_scatter(Items in, Items out, const uint32_t* __restrict__ n_p,
                                                      int64_t cap, int shift, const uint32_t* __restrict__ hist,
                                                      const uint32_t* __restrict__ digit_total, SelInput si,
                                                      SortViews V)
{
    constexpr int R = 1 << BITS;
    constexpr bool SEL = IN == kSel;
    static_assert(R <= kThreads, "one thread per digit");
    __shared__ uint32_t s_dst[R];    // output index of the digit's first item of this tile, less s_start
    __shared__ uint32_t s_start[R];
    // per (round, wave, digit): the group's count, then its exclusive offset
    // among the tile's items of that digit (at most (kThreads * IPT): fits 16 bits)
    __shared__ uint16_t s_cnt[IPT][kWaves][R];
    __shared__ uint2 s_kv[(kThreads * IPT)];
    __shared__ uint32_t s_wave[kWaves];
    __shared__ uint32_t s_seg[SEL ? kMaxViews + 1 : 1];
    const int64_t n = count_of(n_p, cap);
    const int64_t n_tiles = (n + (kThreads * IPT) - 1) / (kThreads * IPT);
    const int tid = threadIdx.x;
    const int wave = tid / fgd::kWave;
    const uint32_t* row = hist + (int64_t)(tid < R ? tid : 0) * row_words(n_tiles);
    if constexpr (SEL) load_segments(si.n_sel, V, s_seg);
    uint32_t base = 0;  // output index of the digit's first item
    auto set_base = [&](uint32_t v) {
        uint32_t tot;
        base = block_excl_scan(tid < R ? v : 0u, s_wave, tot);
        if (SEL && blockIdx.x == 0 && tid == 0) {
            *si.n_out = tot;
            if ((int64_t)tot > si.cap_out) atomicOr(si.status, FG_STATUS_ITEM_OVERFLOW);
        }
    };
    if constexpr (!SUM) set_base(tid < R ? digit_total[tid] : 0u);
    else if (n_tiles == 0) set_base(0u);
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        uint32_t k[IPT], v[IPT], below[IPT];
        bool ok[IPT];
#pragma unroll
        for (int r = 0; r < IPT; r++) {
            const int64_t idx = tile * (kThreads * IPT) + r * kThreads + tid;
            pass_item<IN>(in, si, V, s_seg, idx, n, true, ok[r], k[r], v[r]);
        }
        // the digit's items in earlier tiles
        uint32_t before = 0;
        if constexpr (!SUM) {
            if (tid < R) before = row[tile];
        } else {
            uint32_t all = 0;
            if (tid < R) {
                for (int64_t t = 0; t < n_tiles; t += 4) {
                    const uint4 c4 = *reinterpret_cast<const uint4*>(row + t);
                    const uint32_t c[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        all += t + u < n_tiles ? c[u] : 0u;
                        before += t + u < tile ? c[u] : 0u;
                    }
                }
            }
            set_base(all);
        }
        {
            uint32_t* c32 = reinterpret_cast<uint32_t*>(&s_cnt[0][0][0]);
            for (int i = tid; i < IPT * kWaves * R / 2; i += kThreads) c32[i] = 0u;
        }
        __syncthreads();
        // every wave ranks its items of every round among equal digits
        // (ballot match), with no barrier between rounds
#pragma unroll
        for (int r = 0; r < IPT; r++) {
            const uint32_t d = (k[r] >> shift) & (R - 1);
            const uint64_t m = match_digit<BITS>(d, ok[r]);
            below[r] = (uint32_t)__popcll(m & fgd::lanemask_lt());
            if (ok[r] && below[r] == 0) s_cnt[r][wave][d] = (uint16_t)__popcll(m);
        }
        __syncthreads();
        // per digit, groups in item order (round-major, then wave)
        uint32_t run = 0;
        if (tid < R) {
#pragma unroll
            for (int r = 0; r < IPT; r++)
#pragma unroll
                for (int w = 0; w < kWaves; w++) {
                    const uint32_t c = s_cnt[r][w][tid];
                    s_cnt[r][w][tid] = (uint16_t)run;
                    run += c;
                }
        }
        uint32_t cnt;  // items of this tile that take part
        {
            const uint32_t e = block_excl_scan(run, s_wave, cnt);
            if (tid < R) {
                s_start[tid] = e;
                s_dst[tid] = base + before - e;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; r++) {
            if (ok[r]) {
                const uint32_t d = (k[r] >> shift) & (R - 1);
                const uint32_t pos = s_start[d] + s_cnt[r][wave][d] + below[r];
                s_kv[pos] = make_uint2(k[r], v[r]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; r++) {
            const int p = r * kThreads + tid;
            if ((uint32_t)p < cnt) {
                const uint2 e = s_kv[p];
                const int64_t g = (int64_t)(s_dst[(e.x >> shift) & (R - 1)] + (uint32_t)p);
                if (!SEL || g < si.cap_out) {
                    if constexpr (OUT == kPairs) {
                        out.kv[g] = e;
                    } else {
                        if constexpr (OUT == kSplit) out.key[g] = e.x;
                        out.val[g] = e.y;
                    }
                }
            }
        }
        __syncthreads();
    }
}

// One workgroup: cnt[0 .. *nblk_items / per) becomes its exclusive prefix sum
// in place, *total the sum (and *total_out, when given, a copy of it clamped
// to 32 bits; overflow of cap sets status bit). The number of blocks is
// derived from the item count that the previous kernel counted over.
__global__ __launch_bounds__(kThreads) void k_block_scan(uint32_t* __restrict__ cnt, const uint32_t* __restrict__ n_items,
                                                         int64_t per, int64_t cap_items, uint32_t* __restrict__ total,
                                                         uint32_t* __restrict__ total_out, int64_t cap_total,
                                                         uint32_t* __restrict__ status, uint32_t overflow_bit)
{
    __shared__ uint32_t s_wave[kWaves];
    const int64_t n = count_of(n_items, cap_items);
    const int64_t nblk = (n + per - 1) / per;
    const int tid = threadIdx.x;
    unsigned long long carry = 0;
    for (int64_t base = 0; base < nblk; base += (int64_t)kThreads * 8) {
        uint32_t c[8];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int64_t i = base + (int64_t)tid * 8 + k;
            c[k] = i < nblk ? cnt[i] : 0u;
            sum += c[k];
        }
        uint32_t tot;
        unsigned long long run = carry + block_excl_scan(sum, s_wave, tot);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int64_t i = base + (int64_t)tid * 8 + k;
            if (i < nblk) cnt[i] = (uint32_t)run;
            run += c[k];
        }
        carry += tot;
    }
    if (tid == 0) {
        const uint32_t t32 = (uint32_t)(carry < 0xFFFFFFFFull ? carry : 0xFFFFFFFFull);
        *total = t32;
        if (total_out) *total_out = t32;
        if ((long long)carry > cap_total) atomicOr(status, overflow_bit);
    }
}

// The blocks with more than kEmitSlice pairs are emitted by several workgroups:
// the first takes their first kEmitSlice pairs, and their further slices
// {block, slice} are listed. A block whose slices do not fit the list keeps all
// its pairs (shared[block] = 0); that takes more pairs than cap_pairs, an
// overflow that the call reports. See fg_slices.h for the list's rule. One workgroup per block took 67 us per view of the
// 20M-node scene at 3 sigma (a block of near splats holds 100 times the mean)
// and 21 us for 100k large splats; slices of 2048 take 21 and 9 us, of 4096 23
// and 13; where the counts are even it makes no difference.
constexpr uint32_t kNoBlock = 0xFFFFFFFFu;  // an empty entry

struct EmitSlices {
    unsigned long long* n;  // slices asked for
    uint2* list;
    uint32_t* shared;
    int64_t cap;
};

// Per 1024 splats in depth order: the sum of their tile counts (the areas of
// their rectangles). The rectangles are gathered here once and stored in depth
// order, so that the emission reads them contiguously.
__global__ __launch_bounds__(kThreads) void k_count_reduce(const uint32_t* __restrict__ order,
                                                           const ushort4* __restrict__ rect,
                                                           const uint32_t* __restrict__ n_p, int64_t cap,
                                                           uint32_t* __restrict__ bsum, ushort4* __restrict__ rect_d,
                                                           EmitSlices sl)
{
    __shared__ uint32_t s_wave[kWaves];
    __shared__ unsigned long long s_at;
    const int64_t n = count_of(n_p, cap);
    const int64_t nblk = (n + kEmitItems - 1) / kEmitItems;
    for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        uint32_t s = 0;
#pragma unroll
        for (int r = 0; r < kEmitIPT; r++) {
            const int64_t j = blk * kEmitItems + r * kThreads + threadIdx.x;
            if (j < n) {
                const ushort4 q = rect[order[j]];
                rect_d[j] = q;
                s += (uint32_t)(q.z - q.x) * (uint32_t)(q.w - q.y);
            }
        }
        uint32_t total;
        block_excl_scan(s, s_wave, total);
        uint32_t share = 0u;  // the block's first workgroup emits all of it
        if (total > kEmitSlice) {
            const uint32_t more = (total - 1) / kEmitSlice;
            if (threadIdx.x == 0) s_at = atomicAdd(sl.n, (unsigned long long)more);
            __syncthreads();
            const fgs::Claim c = fgs::claim(s_at, more, (uint64_t)sl.cap);
            for (uint64_t k = c.first + threadIdx.x; k < c.last; k += kThreads)
                sl.list[k] = c.listed ? make_uint2((uint32_t)blk, (uint32_t)(k - c.first) + 1u) : make_uint2(kNoBlock, 0u);
            share = c.listed ? 1u : 0u;
        }
        if (threadIdx.x == 0) {
            bsum[blk] = total;
            sl.shared[blk] = share;
        }
    }
}

// Per 1024 splats in depth order: every splat's output offset (the block's
// offset from the scanned block sums, plus an exclusive scan within the
// block), then the block's pairs are written with thread k taking output
// positions k, k + 256, ...: a binary search over the offsets finds the
// splat, and the position within its rectangle (rows, then columns) gives
// the tile, numbered in its view's global tile ids.
template <int OUT>
__global__ __launch_bounds__(kThreads) void k_emit(const uint32_t* __restrict__ order,
                                                   const ushort4* __restrict__ rect_d, const uint32_t* __restrict__ n_p,
                                                   int64_t cap, BlockOffsets boff, int64_t cap_pairs,
                                                   SortViews V, EmitSlices sl, Items out)
{
    __shared__ uint32_t s_wave[kWaves];
    __shared__ unsigned long long s_red[kWaves];
    __shared__ uint32_t s_off[kEmitItems + 1];
    __shared__ uint32_t s_g[kEmitItems];
    __shared__ ushort4 s_rect[kEmitItems];
    const int64_t n = count_of(n_p, cap);
    const int64_t nblk = (n + kEmitItems - 1) / kEmitItems;
    const int tid = threadIdx.x;
    const int64_t n_items = nblk + (int64_t)fgs::entries(*sl.n, (uint64_t)sl.cap);
    for (int64_t it = blockIdx.x; it < n_items; it += gridDim.x) {
        int64_t blk = it;
        uint32_t first = 0, most = 0xFFFFFFFFu;  // of the block's pairs
        if (it >= nblk) {
            const uint2 e = sl.list[it - nblk];
            if ((int64_t)e.x >= nblk) continue;  // an empty entry
            blk = e.x;
            first = e.y * kEmitSlice;
            most = kEmitSlice;
        } else if (sl.shared[blk]) {
            most = kEmitSlice;
        }
        const unsigned long long base = block_offset(boff, blk, s_red);
        const int64_t j0 = blk * kEmitItems + (int64_t)tid * kEmitIPT;
        uint32_t c[kEmitIPT];
        uint32_t sum = 0;
#pragma unroll
        for (int r = 0; r < kEmitIPT; r++) {
            const int64_t j = j0 + r;
            const uint32_t g = j < n ? order[j] : 0u;
            const ushort4 q = j < n ? rect_d[j] : make_ushort4(0, 0, 0, 0);
            c[r] = (uint32_t)(q.z - q.x) * (uint32_t)(q.w - q.y);
            s_g[tid * kEmitIPT + r] = g;
            s_rect[tid * kEmitIPT + r] = q;
            sum += c[r];
        }
        uint32_t total;
        uint32_t run = block_excl_scan(sum, s_wave, total);
#pragma unroll
        for (int r = 0; r < kEmitIPT; r++) {
            s_off[tid * kEmitIPT + r] = run;
            run += c[r];
        }
        if (tid == 0) s_off[kEmitItems] = total;
        __syncthreads();
        // runs of kEmitRun consecutive outputs per thread: one binary search
        // per run (the last splat k with s_off[k] <= o; splats with no tile
        // share their successor's offset and are passed over), then step
        // through the rectangle, rows then columns
        const uint32_t last = total - first < most ? total : first + most;
        for (uint32_t o0 = first + (uint32_t)tid * kEmitRun; o0 < last; o0 += (uint32_t)kThreads * kEmitRun) {
            int lo = 0, hi = kEmitItems;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_off[mid] <= o0) lo = mid; else hi = mid;
            }
            ushort4 q = s_rect[lo];
            uint32_t w = (uint32_t)(q.z - q.x);
            uint32_t gv = s_g[lo] / V.cap_sel;
            const uint32_t local = o0 - s_off[lo];
            uint32_t ty = q.y + local / w, tx = q.x + local % w;
            const int m = last - o0 < (uint32_t)kEmitRun ? (int)(last - o0) : kEmitRun;
            for (int r = 0; r < m; r++) {
                const unsigned long long dst = base + o0 + (uint32_t)r;
                if (dst < (unsigned long long)cap_pairs) {
                    const uint2 e = make_uint2(V.tile_base[gv] + ty * V.Wt[gv] + tx, s_g[lo]);
                    if constexpr (OUT == kPairs) {
                        out.kv[dst] = e;
                    } else {
                        out.key[dst] = e.x;
                        out.val[dst] = e.y;
                    }
                }
                if (r + 1 < m && ++tx == q.z) {
                    tx = q.x;
                    if (++ty == q.w) {  // next splat with a tile (one exists: r + 1 < m)
                        do {
                            ++lo;
                        } while (s_off[lo + 1] == s_off[lo]);
                        q = s_rect[lo];
                        w = (uint32_t)(q.z - q.x);
                        gv = s_g[lo] / V.cap_sel;
                        tx = q.x;
                        ty = q.y;
                    }
                }
            }
        }
        __syncthreads();
    }
    block_total(boff, nblk, s_red);
}

__global__ void k_ranges(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ n_p, int64_t cap,
                         uint32_t tile_base, int64_t n_tiles, uint32_t* __restrict__ ranges)
{
    const int64_t n = count_of(n_p, cap);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = keys[i];
        const uint32_t t = k - tile_base;
        if ((int64_t)t >= n_tiles) continue;
        if (i == 0 || keys[i - 1] != k) ranges[2 * (int64_t)t] = (uint32_t)i;
        if (i == n - 1 || keys[i + 1] != k) ranges[2 * (int64_t)t + 1] = (uint32_t)(i + 1);
    }
}

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int64_t tiles_for(int64_t n) { return (n + kTileItems - 1) / kTileItems; }

// Depth keys and splat ids ping-pong between buffers 0 and 1 as pairs; the last
// of the four passes leaves the splat ids alone in buffer 0, after which buffer
// 1 (8 bytes per splat) holds the rectangles in depth order.
struct SortWs {
    uint2 *d0, *d1, *alt;
    uint32_t *bsum, *hist, *digit_total, *counts;
    ushort4* rect_d;
    EmitSlices slices;
};
// counts[0]: concatenated selection items, [1]: tile-covering splats packed,
// [2, 3]: emission slices asked for (64 bits)

size_t carve(void* base, int64_t sel_items, int64_t cap_items, int64_t cap_pairs, SortWs* w)
{
    int64_t most = cap_items > cap_pairs ? cap_items : cap_pairs;
    if (sel_items > most) most = sel_items;
    const int64_t ht = tiles_for(most);
    const size_t nblk_emit = (size_t)((cap_items + kEmitItems - 1) / kEmitItems + 1);
    w->slices.cap = cap_pairs / kEmitSlice + 1;
    const size_t sizes[9] = {(size_t)cap_items * 8, (size_t)cap_items * 8, (size_t)cap_pairs * 8, nblk_emit * 4,
                             (size_t)256 * (size_t)(ht + 4) * 4, (size_t)256 * 4, 16, (size_t)w->slices.cap * 8,
                             nblk_emit * 4};
    void** dst[9] = {(void**)&w->d0, (void**)&w->d1, (void**)&w->alt, (void**)&w->bsum, (void**)&w->hist,
                     (void**)&w->digit_total, (void**)&w->counts, (void**)&w->slices.list, (void**)&w->slices.shared};
    size_t off = 0;
    for (int i = 0; i < 9; i++) {
        if (base) *dst[i] = (char*)base + off;
        off += align_up(sizes[i] + 4);
    }
    if (base) {
        w->rect_d = reinterpret_cast<ushort4*>(w->d1);
        // 8-byte aligned for its atomics, whatever the workspace's own alignment
        w->slices.n = reinterpret_cast<unsigned long long*>(((uintptr_t)(w->counts + 2) + 7) & ~(uintptr_t)7);
    }
    return off;
}

// Items per thread of a radix pass: 4 (1024-item tiles) for one view, whose
// counts are a few million; 8 (2048-item tiles) for a batch of views with a
// capacity of tens of millions, where a scatter tile's 256 digit runs average 8
// items (64-byte writes). Eight views of the 20M-node scene, all passes: 4 items
// 1062 us, 8 items 893 us, 16 items (two workgroups per CU by LDS) 1031 us; one
// view of 1.5M splats and 1.9M pairs: 4 and 8 items within 1 %.
// Chosen from the call's shape on the host (the counts stay on the device).
constexpr int kBigIPT = 8;
constexpr int64_t kBigSort = (int64_t)4 << 20;

// Block counts up to which the emission kernel sums its block offsets itself
// (see BlockOffsets): up to 8M splats at 1024 per block.
constexpr int64_t kInlineBlocks = 8192;

// Histogram tiles up to which the scatter sums each digit's row itself instead of
// having it scanned first: every workgroup reads all rows (up to 256 KiB,
// L2-resident), which grows with the square of the tiles, but saves a launch of
// 3 us and its gap per pass. 15k splats, depth passes: 19 us of scatters and 12 of
// scans before, 25 us with the sums inside (first frame pass included).
constexpr int64_t kSumTiles = 256;

template <int BITS, int IPT, int IN, int OUT>
void radix_pass_ipt(const Items& in, const Items& out, const uint32_t* n_p, int64_t cap, int shift, const SortWs& w,
                    const SelInput& si, const SortViews& V, hipStream_t s)
{
    const int64_t tiles = (cap + kThreads * IPT - 1) / (kThreads * IPT);
    const unsigned grid = (unsigned)(tiles > 4096 ? 4096 : (tiles < 1 ? 1 : tiles));
    hipLaunchKernelGGL((k_hist<BITS, IPT, IN>), dim3(grid), dim3(kThreads), 0, s, in, n_p, cap, shift, w.hist, si, V);
    if (IPT == kIPT && tiles <= kSumTiles) {
        hipLaunchKernelGGL((k_scatter<BITS, IPT, IN, OUT, IPT == kIPT>), dim3(grid), dim3(kThreads), 0, s, in, out, n_p,
                           cap, shift, w.hist, w.digit_total, si, V);
        return;
    }
    hipLaunchKernelGGL(k_rowscan<IPT>, dim3(1u << BITS), dim3(kThreads), 0, s, n_p, cap, w.hist, w.digit_total);
    hipLaunchKernelGGL((k_scatter<BITS, IPT, IN, OUT, false>), dim3(grid), dim3(kThreads), 0, s, in, out, n_p, cap,
                       shift, w.hist, w.digit_total, si, V);
}

template <int BITS, int IN, int OUT>
void radix_pass(const Items& in, const Items& out, const uint32_t* n_p, int64_t cap, int shift, bool big,
                const SortWs& w, const SelInput& si, const SortViews& V, hipStream_t s)
{
    if (big) radix_pass_ipt<BITS, kBigIPT, IN, OUT>(in, out, n_p, cap, shift, w, si, V, s);
    else radix_pass_ipt<BITS, kIPT, IN, OUT>(in, out, n_p, cap, shift, w, si, V, s);
}

// A pass over the Gaussian-tile pairs: the last one and every second before it
// write the separate output arrays, the others the pair buffer.
template <int BITS>
void tile_pass(bool to_split, const Items& split, const Items& alt, const uint32_t* n_p, int64_t cap, int shift,
               bool big, const SortWs& w, const SortViews& V, hipStream_t s)
{
    const SelInput none{};
    if (to_split) radix_pass<BITS, kPairs, kSplit>(alt, split, n_p, cap, shift, big, w, none, V, s);
    else radix_pass<BITS, kSplit, kPairs>(split, alt, n_p, cap, shift, big, w, none, V, s);
}

void tile_pass_bits(int bits, bool to_split, const Items& split, const Items& alt, const uint32_t* n_p, int64_t cap,
                    int shift, bool big, const SortWs& w, const SortViews& V, hipStream_t s)
{
    switch (bits) {
        case 4: tile_pass<4>(to_split, split, alt, n_p, cap, shift, big, w, V, s); break;
        case 5: tile_pass<5>(to_split, split, alt, n_p, cap, shift, big, w, V, s); break;
        case 6: tile_pass<6>(to_split, split, alt, n_p, cap, shift, big, w, V, s); break;
        case 7: tile_pass<7>(to_split, split, alt, n_p, cap, shift, big, w, V, s); break;
        default: tile_pass<8>(to_split, split, alt, n_p, cap, shift, big, w, V, s); break;
    }
}

// Validates the views of a sort or render call: sizes, consecutive global
// tile ids (view v's first tile follows view v-1's last). Returns the total
// tile count, or -1.
int64_t views_tiles(const fg_camera* cams, int32_t n_views)
{
    if (!cams || n_views < 1 || n_views > kMaxViews) return -1;
    int64_t total = 0;
    for (int v = 0; v < n_views; v++) {
        if (cams[v].width <= 0 || cams[v].height <= 0) return -1;
        const int64_t nt = (int64_t)((cams[v].width + 15) / 16) * ((cams[v].height + 15) / 16);
        if ((int64_t)cams[v].tile_base != (int64_t)cams[0].tile_base + total) return -1;
        total += nt;
    }
    if ((uint64_t)cams[0].tile_base + (uint64_t)total - 1 > 0xFFFFFFFFull) return -1;
    return total;
}

}  // namespace

extern "C" size_t fg_sort_workspace_size(int64_t cap_sel, int32_t n_views, int64_t cap_items, int64_t cap_pairs)
{
    if (cap_sel < 0 || n_views < 1 || cap_items < 0 || cap_pairs < 0) return 0;
    SortWs w;
    return carve(nullptr, cap_sel * n_views, cap_items, cap_pairs, &w);
}

extern "C" int fg_sort(const fg_splats* splats, const uint32_t* n_sel, int64_t cap_sel, const fg_camera* cams,
                       int32_t n_views, int64_t cap_items, uint32_t* tile_keys, uint32_t* vals, int64_t cap_pairs,
                       uint32_t* n_pairs, uint32_t* ranges, uint32_t* status, void* ws, size_t ws_bytes,
                       const fg_tune* tune, void* stream)
{
    if (!splats || !n_sel || !cams || !n_pairs || !ranges || !status || cap_sel < 0 || cap_pairs < 0 ||
        cap_items < 0 || n_views < 1)
        return FG_ERR_INVALID_ARG;
    if (n_views > kMaxViews || cap_sel * n_views >= ((int64_t)1 << 32) || cap_items >= ((int64_t)1 << 31) ||
        cap_pairs >= ((int64_t)1 << 32) - 1)
        return FG_ERR_UNSUPPORTED;
    if (cap_pairs > 0 && (!tile_keys || !vals)) return FG_ERR_INVALID_ARG;
    if (cap_sel > 0 && (!splats->rgb_depth || !splats->rect || !splats->tiles)) return FG_ERR_INVALID_ARG;
    const int64_t n_tiles = views_tiles(cams, n_views);
    if (n_tiles < 0) return FG_ERR_INVALID_ARG;
    int bits = 0;  // 0: the narrowest digit that needs no more passes than 8-bit digits
    if (tune && tune->radix_bits) {
        if (tune->radix_bits < 4 || tune->radix_bits > 8) return FG_ERR_INVALID_ARG;
        bits = tune->radix_bits;
    }
    SortWs w;
    const size_t need = carve(nullptr, cap_sel * n_views, cap_items, cap_pairs, &w);
    if (!ws || ws_bytes < need) return FG_ERR_WORKSPACE;
    carve(ws, cap_sel * n_views, cap_items, cap_pairs, &w);
    SortViews V;
    V.n = n_views;
    V.cap_sel = (uint32_t)cap_sel;
    for (int v = 0; v < kMaxViews; v++) {
        V.Wt[v] = v < n_views ? (uint32_t)((cams[v].width + 15) / 16) : 0u;
        V.tile_base[v] = v < n_views ? cams[v].tile_base : 0u;
    }
    hipStream_t s = (hipStream_t)stream;
    const uint64_t max_tile = (uint64_t)cams[0].tile_base + (uint64_t)n_tiles - 1;

    // 1. the splats that cover a tile, in depth order: the first 8-bit pass
    //    reads the selections and packs them (into buffer 1), three more
    //    passes end in buffer 0
    auto grid_for = [](int64_t items, int64_t per) {
        int64_t g = (items + per - 1) / per;
        return (unsigned)(g > 4096 ? 4096 : (g < 1 ? 1 : g));
    };
    const int64_t sel_items = cap_sel * n_views;
    const bool big_depth = n_views > 1 && cap_items >= kBigSort;
    const SelInput sel{(const float4*)splats->rgb_depth, splats->tiles, n_sel, w.counts, w.slices.n, w.counts + 1, cap_items,
                       status, ranges, 2 * n_tiles};
    const SelInput none{};
    const Items d0{w.d0, nullptr, nullptr}, d1{w.d1, nullptr, nullptr};
    const Items order{nullptr, nullptr, reinterpret_cast<uint32_t*>(w.d0)};
    radix_pass<8, kSel, kPairs>(Items{}, d1, w.counts, sel_items, 0, big_depth, w, sel, V, s);
    const uint32_t* n_vis = w.counts + 1;
    radix_pass<8, kPairs, kPairs>(d1, d0, n_vis, cap_items, 8, big_depth, w, none, V, s);
    radix_pass<8, kPairs, kPairs>(d0, d1, n_vis, cap_items, 16, big_depth, w, none, V, s);
    radix_pass<8, kPairs, kValues>(d1, order, n_vis, cap_items, 24, big_depth, w, none, V, s);
    // 2. tile counts in depth order and key emission
    const unsigned gv = grid_for(cap_items, kEmitItems);
    hipLaunchKernelGGL(k_count_reduce, dim3(gv), dim3(kThreads), 0, s, order.val, (const ushort4*)splats->rect, n_vis,
                       cap_items, w.bsum, w.rect_d, w.slices);
    const BlockOffsets boff{w.bsum, (cap_items + kEmitItems - 1) / kEmitItems <= kInlineBlocks, n_pairs, cap_pairs,
                            status, FG_STATUS_PAIR_OVERFLOW};
    if (!boff.inline_sum)
        hipLaunchKernelGGL(k_block_scan, dim3(1), dim3(kThreads), 0, s, w.bsum, n_vis, (int64_t)kEmitItems, cap_items,
                           n_pairs, (uint32_t*)nullptr, cap_pairs, status, FG_STATUS_PAIR_OVERFLOW);
    int tile_bits = 1;
    while (tile_bits < 32 && (max_tile >> tile_bits) != 0) ++tile_bits;
    if (bits == 0) {
        const int p8 = (tile_bits + 7) / 8;
        bits = (tile_bits + p8 - 1) / p8;  // e.g. 13 bits: two passes of 7
        if (bits < 4) bits = 4;
    }
    const int passes = (tile_bits + bits - 1) / bits;
    // emit into the buffer that the first pass reads
    const Items split{nullptr, tile_keys, vals}, alt{w.alt, nullptr, nullptr};
    const unsigned ge = gv + grid_for(w.slices.cap, 4);
    if (passes % 2)
        hipLaunchKernelGGL(k_emit<kPairs>, dim3(ge), dim3(kThreads), 0, s, order.val, w.rect_d, n_vis, cap_items, boff,
                           cap_pairs, V, w.slices, alt);
    else
        hipLaunchKernelGGL(k_emit<kSplit>, dim3(ge), dim3(kThreads), 0, s, order.val, w.rect_d, n_vis, cap_items, boff,
                           cap_pairs, V, w.slices, split);
    if (cap_pairs > 0) {
        // 3. stable sort of the pairs by tile id
        for (int p = 0; p < passes; p++)
            tile_pass_bits(bits, (passes - p) % 2 != 0, split, alt, n_pairs, cap_pairs, bits * p,
                           n_views > 1 && cap_pairs >= kBigSort, w, V, s);
        hipLaunchKernelGGL(k_ranges, dim3(grid_for(cap_pairs, 256)), dim3(256), 0, s, tile_keys, n_pairs, cap_pairs,
                           cams[0].tile_base, n_tiles, ranges);
    }
    return hipGetLastError() == hipSuccess ? FG_OK : FG_ERR_HIP;
}
