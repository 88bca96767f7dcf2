// Per-tile front-to-back alpha blending, Eq. (2).
//
// In Eq. (2) the per-fragment opacity alpha_i and the skip decisions
// (power > 0, alpha < 1/255) depend only on the splat and the pixel, not on
// the transmittance; only the product T_i = prod (1 - alpha_j), the early
// stop (T < 1e-4) and the colour sum run sequentially. Tiles near a horizon
// can hold ~10^4 splats whose pixels seldom saturate, so one workgroup that
// tests every (pixel, splat) of such a tile would leave the frame waiting on
// it. Tiles are therefore told apart (see init_counters for the line):
//
//   "long" tiles have pass masks (per pixel, the splats that pass the skip
//   tests) made for all their chunks of CHUNK splats in parallel; then each
//   pixel walks the tile's splats in list order, chunk by chunk, visiting
//   only the marked ones and recomputing alpha with the same expressions, two
//   lanes per pixel sharing the alphas (k_render_long);
//
//   the others are blended by one workgroup each, 256 splats at a time, every
//   8 lanes visiting the splats that can reach their own 4 x 2 pixel block
//   (fg_blocks.h): each alpha is evaluated once, where it is used, with no
//   masks and no atomics.
//
// k_render makes the masks and blends the tiles that are not long, in one
// launch; k_render_long follows. Every value and decision is bit-identical to
// one sequential pass.
//
// Before them, k_schedule counts each tile's chunks and orders the tiles that
// hold splats ("heavy" ones, of more than one chunk, first), and k_tile_prep
// writes the pixels of the others (background, T = 1) and maps chunk items to
// their tiles. The launch boundaries order all writes before their reads; no
// workgroup ever waits for another.
#include "fg_blocks.h"
#include "fg_device.h"
#include "fg_render_ws.h"

namespace {

constexpr int kThreads = 256;
constexpr int kScanThreads = 1024;

struct RenderWs {
    uint32_t* nch;        // [n_tiles] chunks per tile (0: no splats)
    uint32_t* mfirst;     // [n_tiles] first chunk item of a heavy tile
    uint32_t* order;      // [n_tiles] tiles in processing order, heavy first
    uint32_t* mitem;      // [max_items] chunk item -> tile
    uint32_t* counters;   // see the kCnt* indices
    uint32_t* masks;      // [max_items][CHUNK/32][256] pass masks of the long tiles' chunks
    float* state;         // with save_state: [max_items][4][256] T, C0, C1, C2 after each chunk; else null
    uint32_t* sched;      // [tile blocks][4] block totals of the many-tile schedule
};

// counters[]: heavy tiles, chunk items (clamped to max_items), tiles with
// splats, chunks from which a tile is long.
enum { kCntHeavy, kCntItems, kCntTiles, kCntLongChunks };

// From how many chunks on a tile is long. Walking a tile's batches one after
// another costs 10 to 20 us per 256 splats on the tile's own (the crowded pixel
// rows of a horizon keep few lanes busy), but about half the work of masks
// and a second walk. So what counts is whether the heavy tiles fill the chip
// by themselves (k_render + k_render_long, us, long from 2 chunks on and by the
// batches):
//  - many of much the same length (items^2 over the sum of squares, the number
//    of equal tiles that they amount to, is 900 or more and at least three
//    quarters of the heavy tiles): only tiles of 12 x 256 splats, or of a
//    thousandth of all chunks, whose own walk takes about as long as all of
//    them together. Training views: 1000 and 343 for 2M Gaussians at 1080p, 625
//    and 333 at 720p, 359 and 255 for 1M at 960 x 540; lists of 3 to 6 chunks
//    on 8000 tiles 2757 and 1187 (128-splat chunks 3822 and 1306). At 640 x 360
//    (766 equal tiles) it is 204 and 252;
//  - of four chunks or more on average (a horizon), or all chunks together too
//    few to fill the chip: from two chunks on. 1M-leaf city (842 chunks on 184
//    tiles) 97 and 290; 20M nodes at 1440p (1017 equal tiles of 1982) 381 and 416;
//  - otherwise only tiles of 12 chunks.
constexpr float kAlikeTiles = 900.0f, kAlikeShare = 0.75f;

__device__ __forceinline__ uint32_t long_chunks(uint32_t heavy, uint32_t items, float squares, int chunk)
{
    const float equal = (float)heavy >= kAlikeTiles ? (float)items * (float)items / squares : 0.0f;
    if (equal >= kAlikeTiles && equal >= kAlikeShare * (float)heavy) {
        const uint32_t least = 12u * 256u / (uint32_t)chunk, share = items / 1000u;
        return share > least ? share : least;
    }
    return items >= 4u * heavy || items < 1024u ? 2u : 12u;
}

__device__ __forceinline__ void init_counters(uint32_t* __restrict__ counters, uint32_t heavy, uint32_t items,
                                              uint32_t tiles, float squares, int chunk, int64_t max_items)
{
    counters[kCntHeavy] = heavy;
    counters[kCntItems] = (int64_t)items < max_items ? items : (uint32_t)max_items;
    counters[kCntTiles] = tiles;
    counters[kCntLongChunks] = long_chunks(heavy, items, squares, chunk);
}

struct Frag {
    unsigned n_eval, n_exp, n_pass, n_blend;
};

// The views of one call. Their tiles are numbered consecutively (view v owns
// tiles tile0[v] .. tile0[v+1] of the call, in the order of its global tile
// ids); view v's image is [3][H][W] at image + 3 * pix0[v], its final T and
// contributor counts at + pix0[v].
constexpr int kMaxViews = 64;
struct RenderViews {
    int n;
    uint32_t tile0[kMaxViews + 1];
    int W[kMaxViews], H[kMaxViews], Wt[kMaxViews];
    int64_t pix0[kMaxViews];
};

// One tile's view and geometry.
struct TileGeom {
    int tx, ty, W, H;
    int64_t pix0;
};

__device__ __forceinline__ TileGeom tile_geom(const RenderViews& V, uint32_t t)
{
    int lo = 0, hi = V.n;  // the view v with tile0[v] <= t < tile0[v+1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (V.tile0[mid] <= t) lo = mid; else hi = mid;
    }
    const uint32_t lt = t - V.tile0[lo];
    TileGeom g;
    g.tx = (int)(lt % (uint32_t)V.Wt[lo]);
    g.ty = (int)(lt / (uint32_t)V.Wt[lo]);
    g.W = V.W[lo];
    g.H = V.H[lo];
    g.pix0 = V.pix0[lo];
    return g;
}

// Whether a heavy tile of nch chunks (first item mf) is long: its chunks' pass
// masks are made by the first workgroups of k_render. Every item must have a
// place in the mask store.
__device__ __forceinline__ bool is_long(const RenderWs& ws, uint32_t nch, uint32_t mf)
{
    return nch >= ws.counters[kCntLongChunks] && mf + nch <= ws.counters[kCntItems];
}

// After k_schedule: the final values of an empty tile's pixels (background,
// T = 1, no contributor), so that the blend never visits it, and the chunk item
// -> tile map of a heavy tile's chunks. Bound by its writes: with one tile per
// workgroup (64-byte rows) 62k empty tiles took 107 us; four side by side, 16
// bytes per store, 63 us, what their 317 MB take at the rate of a copy. With the
// 8160 tiles of one view that leaves too few workgroups (8.3 us, 9.3 by fours),
// so per_wg is 4 only for the tiles of many views.
__global__ __launch_bounds__(kThreads) void k_tile_prep(int64_t n_tiles, int per_wg, RenderViews V, float bg0, float bg1,
                                                        float bg2, RenderWs ws, int64_t max_items,
                                                        float* __restrict__ image, float* __restrict__ final_T,
                                                        uint32_t* __restrict__ n_contrib)
{
    // four consecutive tiles at a time: where they are empty, side by side and
    // wholly inside, a thread writes four pixels of a row
    for (int64_t t0 = per_wg * (int64_t)blockIdx.x; t0 < n_tiles; t0 += per_wg * (int64_t)gridDim.x) {
        const int n = n_tiles - t0 < per_wg ? (int)(n_tiles - t0) : per_wg;
        uint32_t c[4];
#pragma unroll
        for (int k = 0; k < 4; k++) c[k] = k < n ? ws.nch[t0 + k] : 1u;
        if ((c[0] | c[1] | c[2] | c[3]) == 0u) {
            const TileGeom g = tile_geom(V, (uint32_t)t0), e = tile_geom(V, (uint32_t)t0 + 3);
            const int64_t plane = (int64_t)g.W * g.H;
            float* img = image + 3 * g.pix0;
            const uintptr_t at = (uintptr_t)img | (uintptr_t)(final_T + g.pix0) | (uintptr_t)(n_contrib + g.pix0);
            if (e.pix0 == g.pix0 && e.ty == g.ty && (g.tx + 4) * fgd::kTile <= g.W && (g.ty + 1) * fgd::kTile <= g.H &&
                g.W % 4 == 0 && at % 16 == 0) {
                const int64_t o = (int64_t)(g.ty * fgd::kTile + (int)threadIdx.x / 16) * g.W + g.tx * fgd::kTile +
                                  4 * ((int)threadIdx.x % 16);
                *reinterpret_cast<float4*>(img + o) = make_float4(bg0, bg0, bg0, bg0);
                *reinterpret_cast<float4*>(img + plane + o) = make_float4(bg1, bg1, bg1, bg1);
                *reinterpret_cast<float4*>(img + 2 * plane + o) = make_float4(bg2, bg2, bg2, bg2);
                *reinterpret_cast<float4*>(final_T + g.pix0 + o) = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
                *reinterpret_cast<uint4*>(n_contrib + g.pix0 + o) = make_uint4(0u, 0u, 0u, 0u);
                continue;
            }
        }
        for (int k = 0; k < n; k++) {
            const int64_t t = t0 + k;
            if (c[k] == 0) {
                const TileGeom g = tile_geom(V, (uint32_t)t);
                const int px = g.tx * fgd::kTile + (int)threadIdx.x % fgd::kTile;
                const int py = g.ty * fgd::kTile + (int)threadIdx.x / fgd::kTile;
                if (px < g.W && py < g.H) {
                    const size_t o = (size_t)py * g.W + px;
                    const size_t plane = (size_t)g.W * g.H;
                    float* img = image + 3 * g.pix0;
                    img[o] = bg0;
                    img[plane + o] = bg1;
                    img[2 * plane + o] = bg2;
                    final_T[g.pix0 + o] = 1.0f;
                    n_contrib[g.pix0 + o] = 0u;
                }
            } else if (c[k] > 1) {
                const uint32_t mf = ws.mfirst[t];
                for (uint32_t i = threadIdx.x; i < c[k]; i += kThreads)
                    if ((int64_t)(mf + i) < max_items) ws.mitem[mf + i] = (uint32_t)t;
            }
        }
    }
}

// One workgroup, one pass: each tile's chunk count (0 for a tile with no
// splats); lists the tiles that hold splats, heavy ones from the front of
// order[] in tile order and light ones from its back in reverse tile order;
// numbers the chunk items of heavy tiles (first item per tile). With h heavy
// tiles, tile i of the blend is order[i] for i < h, else the light tile
// order[n_tiles - 1 - (i - h)]. 8 consecutive tiles per thread per
// round (the ranges are read and the chunk counts written with consecutive
// lanes on consecutive tiles, and handed over through LDS); the running
// counts of heavy and light tiles (one 64-bit word) and of chunk items are
// scanned together.
template <int CHUNK>
__global__ __launch_bounds__(kScanThreads) void k_schedule(const uint32_t* __restrict__ ranges, int64_t n_tiles,
                                                           int64_t max_mask_items, uint32_t* __restrict__ nch,
                                                           uint32_t* __restrict__ mfirst, uint32_t* __restrict__ order,
                                                           uint32_t* __restrict__ counters)
{
    __shared__ unsigned long long s_wave[kScanThreads / fgd::kWave];
    __shared__ uint32_t s_wave_m[kScanThreads / fgd::kWave];
    __shared__ unsigned long long s_carry;
    __shared__ uint32_t s_carry_m;
    __shared__ uint32_t s_c[8 * kScanThreads];
    const int tid = threadIdx.x, lane = fgd::lane_id(), wave = tid / fgd::kWave;
    float squares = 0.0f;  // of the heavy tiles' chunk counts
    if (tid == 0) {
        s_carry = 0ull;
        s_carry_m = 0u;
    }
    __syncthreads();
    for (int64_t base = 0; base < n_tiles; base += 8 * kScanThreads) {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int64_t t = base + (int64_t)k * kScanThreads + tid;
            uint32_t ck = 0u;
            if (t < n_tiles) {
                const uint2 r = reinterpret_cast<const uint2*>(ranges)[t];
                ck = (r.y - r.x + CHUNK - 1) / CHUNK;
                nch[t] = ck;
            }
            s_c[k * kScanThreads + tid] = ck;
        }
        __syncthreads();
        uint32_t c[8];
        unsigned long long sum = 0;  // low 32: heavy tiles, high 32: light tiles
        uint32_t msum = 0;           // mask items
#pragma unroll
        for (int k = 0; k < 8; k++) {
            c[k] = s_c[tid * 8 + k];
            if (c[k] > 1) {
                sum += 1ull;
                msum += c[k];
                squares += (float)c[k] * (float)c[k];
            } else if (c[k] == 1) {
                sum += 1ull << 32;
            }
        }
        unsigned long long x = sum;
        uint32_t xm = msum;
#pragma unroll
        for (int d = 1; d < fgd::kWave; d <<= 1) {
            const unsigned long long y = __shfl_up(x, d, fgd::kWave);
            const uint32_t ym = __shfl_up(xm, d, fgd::kWave);
            if (lane >= d) {
                x += y;
                xm += ym;
            }
        }
        if (lane == fgd::kWave - 1) {
            s_wave[wave] = x;
            s_wave_m[wave] = xm;
        }
        __syncthreads();
        unsigned long long before = s_carry, total = 0;
        uint32_t before_m = s_carry_m, total_m = 0;
        for (int w = 0; w < kScanThreads / fgd::kWave; w++) {
            if (w < wave) {
                before += s_wave[w];
                before_m += s_wave_m[w];
            }
            total += s_wave[w];
            total_m += s_wave_m[w];
        }
        unsigned long long run = before + x - sum;
        uint32_t mf = before_m + xm - msum;  // mask items before t
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int64_t t = base + (int64_t)tid * 8 + k;
            if (t < n_tiles && c[k] > 0) {
                if (c[k] > 1) {
                    order[(uint32_t)run] = (uint32_t)t;  // heavy tiles before t
                    mfirst[t] = mf;
                    run += 1ull;
                    mf += c[k];
                } else {
                    order[n_tiles - 1 - (int64_t)(run >> 32)] = (uint32_t)t;  // light tiles before t
                    run += 1ull << 32;
                }
            }
        }
        __syncthreads();
        if (tid == 0) {
            s_carry += total;
            s_carry_m += total_m;
        }
        __syncthreads();
    }
    const uint32_t heavy = (uint32_t)s_carry;
    if ((float)heavy >= kAlikeTiles) {  // else the squares decide nothing
#pragma unroll
        for (int d = fgd::kWave / 2; d > 0; d >>= 1) squares += __shfl_xor(squares, d, fgd::kWave);
        if (lane == 0) s_wave_m[wave] = __float_as_uint(squares);
        __syncthreads();
        squares = 0.0f;
        for (int w = 0; w < kScanThreads / fgd::kWave; w++) squares += __uint_as_float(s_wave_m[w]);
    }
    if (tid == 0)
        init_counters(counters, heavy, s_carry_m, heavy + (uint32_t)(s_carry >> 32), squares, CHUNK, max_mask_items);
}

// The same schedule for many tiles (a batch of views), in three launches:
// per block of 8192 tiles the chunk counts and the block's totals (heavy
// tiles, light tiles, mask items, squares of chunk counts); one workgroup scans
// the block totals; each block then writes its part of order[] and mfirst[] from
// its base. Results equal k_schedule's.
constexpr int kSchedTiles = 8 * kScanThreads;
constexpr int kSchedWords = 4;

template <int CHUNK>
__global__ __launch_bounds__(kScanThreads) void k_sched_count(const uint32_t* __restrict__ ranges, int64_t n_tiles,
                                                              uint32_t* __restrict__ nch,
                                                              uint32_t* __restrict__ bsum)
{
    __shared__ uint32_t s_h[kScanThreads / fgd::kWave], s_l[kScanThreads / fgd::kWave],
        s_m[kScanThreads / fgd::kWave];
    __shared__ float s_q[kScanThreads / fgd::kWave];
    const int tid = threadIdx.x, lane = fgd::lane_id(), wave = tid / fgd::kWave;
    const int64_t base = (int64_t)blockIdx.x * kSchedTiles;
    uint32_t h = 0, l = 0, m = 0;
    float q = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int64_t t = base + (int64_t)tid * 8 + k;
        const uint32_t c = t < n_tiles ? (ranges[2 * t + 1] - ranges[2 * t] + CHUNK - 1) / CHUNK : 0u;
        if (t < n_tiles) nch[t] = c;
        if (c > 1) {
            h += 1u;
            m += c;
            q += (float)c * (float)c;
        } else if (c == 1) {
            l += 1u;
        }
    }
#pragma unroll
    for (int d = fgd::kWave / 2; d > 0; d >>= 1) {
        h += __shfl_xor(h, d, fgd::kWave);
        l += __shfl_xor(l, d, fgd::kWave);
        m += __shfl_xor(m, d, fgd::kWave);
        q += __shfl_xor(q, d, fgd::kWave);
    }
    if (lane == 0) {
        s_h[wave] = h;
        s_l[wave] = l;
        s_m[wave] = m;
        s_q[wave] = q;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t th = 0, tl = 0, tm = 0;
        float tq = 0.0f;
        for (int w = 0; w < kScanThreads / fgd::kWave; w++) {
            th += s_h[w];
            tl += s_l[w];
            tm += s_m[w];
            tq += s_q[w];
        }
        uint32_t* b = bsum + kSchedWords * blockIdx.x;
        b[0] = th;
        b[1] = tl;
        b[2] = tm;
        b[3] = __float_as_uint(tq);
    }
}

// One thread: exclusive scan of the blocks' totals in place, and the counters.
__global__ void k_sched_scan(uint32_t* __restrict__ bsum, int64_t nb, int chunk, int64_t max_mask_items,
                             uint32_t* __restrict__ counters)
{
    if (threadIdx.x != 0) return;
    uint32_t h = 0, l = 0, m = 0;
    float q = 0.0f;
    for (int64_t i = 0; i < nb; i++) {
        uint32_t* b = bsum + kSchedWords * i;
        const uint32_t a0 = b[0], a1 = b[1], a2 = b[2];
        q += __uint_as_float(b[3]);
        b[0] = h;
        b[1] = l;
        b[2] = m;
        h += a0;
        l += a1;
        m += a2;
    }
    init_counters(counters, h, m, h + l, q, chunk, max_mask_items);
}

template <int CHUNK>
__global__ __launch_bounds__(kScanThreads) void k_sched_write(int64_t n_tiles, const uint32_t* __restrict__ nch,
                                                              const uint32_t* __restrict__ bsum,
                                                              uint32_t* __restrict__ mfirst,
                                                              uint32_t* __restrict__ order)
{
    __shared__ unsigned long long s_wave[kScanThreads / fgd::kWave];
    __shared__ uint32_t s_wave_m[kScanThreads / fgd::kWave];
    const int tid = threadIdx.x, lane = fgd::lane_id(), wave = tid / fgd::kWave;
    const int64_t base = (int64_t)blockIdx.x * kSchedTiles;
    uint32_t c[8];
    unsigned long long sum = 0;  // low 32: heavy tiles, high 32: light tiles
    uint32_t msum = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int64_t t = base + (int64_t)tid * 8 + k;
        c[k] = t < n_tiles ? nch[t] : 0u;
        if (c[k] > 1) {
            sum += 1ull;
            msum += c[k];
        } else if (c[k] == 1) {
            sum += 1ull << 32;
        }
    }
    unsigned long long x = sum;
    uint32_t xm = msum;
#pragma unroll
    for (int d = 1; d < fgd::kWave; d <<= 1) {
        const unsigned long long y = __shfl_up(x, d, fgd::kWave);
        const uint32_t ym = __shfl_up(xm, d, fgd::kWave);
        if (lane >= d) {
            x += y;
            xm += ym;
        }
    }
    if (lane == fgd::kWave - 1) {
        s_wave[wave] = x;
        s_wave_m[wave] = xm;
    }
    __syncthreads();
    const uint32_t* b = bsum + kSchedWords * blockIdx.x;
    unsigned long long run = (unsigned long long)b[0] | ((unsigned long long)b[1] << 32);
    uint32_t mf = b[2];
    for (int w = 0; w < wave; w++) {
        run += s_wave[w];
        mf += s_wave_m[w];
    }
    run += x - sum;
    mf += xm - msum;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int64_t t = base + (int64_t)tid * 8 + k;
        if (t < n_tiles && c[k] > 0) {
            if (c[k] > 1) {
                order[(uint32_t)run] = (uint32_t)t;
                mfirst[t] = mf;
                run += 1ull;
                mf += c[k];
            } else {
                order[n_tiles - 1 - (int64_t)(run >> 32)] = (uint32_t)t;
                run += 1ull << 32;
            }
        }
    }
}

template <bool STATS, int N>
__device__ __forceinline__ void flush_stats(const Frag& f, unsigned long long* frag_stats)
{
    if (!STATS) return;
    const unsigned long long c[4] = {f.n_eval, f.n_exp, f.n_pass, f.n_blend};
#pragma unroll
    for (int k = 0; k < N; k++) {
        unsigned long long v = c[k];
#pragma unroll
        for (int d = fgd::kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, fgd::kWave);
        if (fgd::lane_id() == 0) atomicAdd(&frag_stats[k], v);
    }
}


struct PixelState {
    float T, C0, C1, C2;
    uint32_t last;
    bool done;
};

// One blend step of Eq. (2) in list order, for a lane whose step is valid
// and whose pixel has not stopped: stop before a splat that would take T
// below 1e-4, otherwise accumulate its colour and attenuate T. Written with
// selects rather than branches (the kept values are the same expressions),
// so the four steps of a group run without divergent control flow.
template <bool STATS>
__device__ __forceinline__ void blend_step(PixelState& p, bool valid, float alpha, float4 c, uint32_t pos, Frag& f)
{
    const float Tn = p.T * (1.0f - alpha);
    const bool live = valid && !p.done;
    const bool stop = Tn < 1e-4f;
    const bool take = live && !stop;
    const float n0 = p.C0 + (c.x * alpha) * p.T;
    const float n1 = p.C1 + (c.y * alpha) * p.T;
    const float n2 = p.C2 + (c.z * alpha) * p.T;
    p.C0 = take ? n0 : p.C0;
    p.C1 = take ? n1 : p.C1;
    p.C2 = take ? n2 : p.C2;
    p.T = take ? Tn : p.T;
    p.last = take ? pos + 1u : p.last;
    p.done = p.done || (live && stop);
    if (STATS) f.n_blend += take ? 1u : 0u;
}

// Walks this lane's block list over one staged batch, four splats at a time:
// their alphas do not depend on T and are computed together, then the blend
// steps run in list order. pos0: list position of the batch's first splat.
template <bool STATS>
__device__ __forceinline__ void walk(const float4* s_a, const float4* s_b, const float* s_c, const uint8_t* list, int n,
                                     float fpx, float fpy, uint32_t pos0, PixelState& p, Frag& f)
{
    for (int k = 0; k < n && !p.done; k += 4) {
        const uint32_t e = *reinterpret_cast<const uint32_t*>(list + k);
        float alpha[4];
        float4 b[4];
        float cb[4];
        bool pass[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int j = (int)((e >> (8 * u)) & 255u);
            b[u] = s_b[j];
            cb[u] = s_c[j];
            bool in_range;
            pass[u] = fgb::eval_alpha(s_a[j], b[u], fpx, fpy, alpha[u], in_range) && k + u < n;
            if (STATS) {
                f.n_eval += k + u < n ? 1u : 0u;
                f.n_exp += k + u < n && in_range ? 1u : 0u;
                f.n_pass += pass[u] ? 1u : 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; u++)
            blend_step<STATS>(p, pass[u], alpha[u], make_float4(b[u].z, b[u].w, cb[u], 0.0f), pos0 + ((e >> (8 * u)) & 255u),
                              f);
    }
}

// ---- long tiles: pass masks, then the walk -----------------------------------

// Rows and columns of a splat's skip ellipse on one tile: on a row at offset dy
// from its centre the passing pixel centres lie within u + (B dy -+ sqrt(11.2 A
// - det dy^2)) / A (see fgb::block_mask for the bound, the slack and the
// conics that take the conservative box instead).
struct Spans {
    float ox, oy, A, B, det, inv;
    int y0, y1, x0, x1;
    bool box;  // whole rows of the box

    __device__ __forceinline__ Spans(float2 mm, float4 co, int tx, int ty, int W, int H)
    {
        A = co.x;
        B = co.y;
        const float C = co.z;
        box = !(A > 0.0f && B * B <= 0.98f * (A * C));
        if (box) {
            const uint32_t b = fgd::splat_box(mm, co, tx, ty, W, H);
            x0 = (int)(b & 255u);
            x1 = (int)((b >> 8) & 255u);
            y0 = (int)((b >> 16) & 255u);
            y1 = x0 <= x1 ? (int)(b >> 24) : -1;
            return;
        }
        ox = (mm.x - (float)(tx * fgd::kTile)) - 0.5f;
        oy = (mm.y - (float)(ty * fgd::kTile)) - 0.5f;
        x0 = 0;
        x1 = W - 1 - tx * fgd::kTile < 15 ? W - 1 - tx * fgd::kTile : 15;
        det = A * C - B * B;
        inv = __builtin_amdgcn_rcpf(A);
        const float ey = __builtin_amdgcn_sqrtf((fgb::kBound * A) * __builtin_amdgcn_rcpf(det));
        const float ys = 0.05f + 1e-4f * (fabsf(oy) + ey);
        const float fa = fmaxf(ceilf(oy - ey - ys), 0.0f);
        const float fb = fminf(floorf(oy + ey + ys), fminf(15.0f, (float)(H - 1 - ty * fgd::kTile)));
        y0 = fa <= fb ? (int)fa : 0;
        y1 = fa <= fb ? (int)fb : -1;
    }

    __device__ __forceinline__ void row(int ly, int& a, int& e) const
    {
        a = x0;
        e = x1;
        if (box) return;
        const float dy = oy - (float)ly;
        const float disc = fgb::kBound * A - det * (dy * dy);
        if (disc < 0.0f) {
            e = a - 1;
            return;
        }
        const float half = __builtin_amdgcn_sqrtf(disc) * inv;
        const float cen = ox + (B * dy) * inv;
        const float slack = 0.05f + 1e-4f * (fabsf(cen) + half);
        // clipped in float (a NaN bound keeps the column) before converting
        const float fa = fminf(fmaxf(ceilf(cen - half - slack), 0.0f), 16.0f);
        const float fe = fmaxf(fminf(floorf(cen + half + slack), (float)x1), -1.0f);
        a = (int)fa;
        e = (int)fe;
    }
};

// Pass masks of the chunks of long tiles, one chunk per work item, to global
// memory [word][pixel]. Each thread takes a whole splat of the chunk (they are
// mostly small), straight from the splat records, since no other thread reads
// them, and tests the pixels of its row spans.
template <int CHUNK, bool STATS>
__device__ __forceinline__ void make_masks(uint32_t* s_mask, uint32_t block, uint32_t blocks,
                                           const float2* __restrict__ xy, const float4* __restrict__ conic_o,
                                           const uint32_t* __restrict__ vals, const uint32_t* __restrict__ ranges,
                                           const RenderViews& V, const RenderWs& ws,
                                           unsigned long long* __restrict__ frag_stats)
{
    constexpr int kWords = CHUNK / 32;
    Frag f = {0, 0, 0, 0};
    const int tid = threadIdx.x;
    const uint32_t n_items = ws.counters[kCntItems];
#pragma unroll
    for (int w = 0; w < kWords; w++) s_mask[w * kThreads + tid] = 0u;
    __syncthreads();
    for (uint32_t item = block; item < n_items; item += blocks) {
        const uint32_t tile = ws.mitem[item];
        const uint32_t mf = ws.mfirst[tile];
        if (!is_long(ws, ws.nch[tile], mf)) continue;
        const uint32_t start = ranges[2 * tile] + (item - mf) * CHUNK, r1 = ranges[2 * tile + 1];
        const int cnt = (int)(r1 - start < (uint32_t)CHUNK ? r1 - start : (uint32_t)CHUNK);
        const TileGeom tg = tile_geom(V, tile);
        for (int j = tid; j < cnt; j += kThreads) {
            const uint32_t g = vals[start + j];
            const float2 mm = xy[g];
            const float4 co = conic_o[g];
            const Spans sp(mm, co, tg.tx, tg.ty, tg.W, tg.H);
            const float4 a = fgb::stage_a(mm, co), b = fgb::stage_b(co, make_float4(0.f, 0.f, 0.f, 0.f));
            const uint32_t bit = 1u << (j & 31);
            uint32_t* mrow = s_mask + (j >> 5) * kThreads;
            for (int ly = sp.y0; ly <= sp.y1; ly++) {
                const float fy = (float)(tg.ty * fgd::kTile + ly) + 0.5f;
                int x, e;
                sp.row(ly, x, e);
                for (; x <= e; x++) {
                    float alpha;
                    bool in_range;
                    const bool pass =
                        fgb::eval_alpha(a, b, (float)(tg.tx * fgd::kTile + x) + 0.5f, fy, alpha, in_range);
                    if (STATS) {
                        ++f.n_eval;
                        f.n_exp += in_range ? 1u : 0u;
                        f.n_pass += pass ? 1u : 0u;
                    }
                    if (pass) atomicOr(&mrow[ly * fgd::kTile + x], bit);
                }
            }
        }
        __syncthreads();
        uint32_t* out = ws.masks + (size_t)item * (kWords * kThreads);
#pragma unroll
        for (int w = 0; w < kWords; w++) {
            out[w * kThreads + tid] = s_mask[w * kThreads + tid];
            s_mask[w * kThreads + tid] = 0u;  // this thread's column, for the next item
        }
        __syncthreads();
    }
    flush_stats<STATS, 3>(f, STATS ? frag_stats + 4 : frag_stats);
}

__device__ __forceinline__ void write_pixel(const PixelState& p, int px, int py, const TileGeom& tg, float bg0, float bg1,
                                            float bg2, float* __restrict__ image, float* __restrict__ final_T,
                                            uint32_t* __restrict__ n_contrib)
{
    const size_t o = (size_t)py * tg.W + px;
    const size_t plane = (size_t)tg.W * tg.H;
    float* img = image + 3 * tg.pix0;
    img[o] = p.C0 + p.T * bg0;
    img[plane + o] = p.C1 + p.T * bg1;
    img[2 * plane + o] = p.C2 + p.T * bg2;
    final_T[tg.pix0 + o] = p.T;
    n_contrib[tg.pix0 + o] = p.last;
}

// One batch of splats as the workgroup's waves visit it.
struct Staged {
    float4 a[fgb::kBatch];
    float4 b[fgb::kBatch];
    float c[fgb::kBatch];
    uint32_t bm[fgb::kBatch];
    __align__(16) uint8_t list[fgb::kBlocks][fgb::kBatch];
};

// Blends the n splats of a tile, batch by batch: each thread stages one
// splat, each wave lists its blocks' splats and walks them. While a batch is
// walked, the next one's records are loaded into registers. keep: the tile's
// chunks have items (first: mf), whose state is saved when asked for.
template <int CHUNK, bool STATS>
__device__ __forceinline__ void blend_batches(Staged& st, const RenderWs& ws, const float2* __restrict__ xy,
                                              const float4* __restrict__ conic_o, const float4* __restrict__ rgb_depth,
                                              const uint32_t* __restrict__ vals, uint32_t n, bool keep, uint32_t nch,
                                              uint32_t mf, const TileGeom& tg, PixelState& p, Frag& f)
{
    constexpr int kBatch = CHUNK < fgb::kBatch ? CHUNK : fgb::kBatch;
    const int tid = threadIdx.x, wave = tid / fgd::kWave;
    const int lx = fgb::pixel_x(tid), ly = fgb::pixel_y(tid);
    const float fpx = (float)(tg.tx * fgd::kTile + lx) + 0.5f, fpy = (float)(tg.ty * fgd::kTile + ly) + 0.5f;
    const uint32_t n_items = ws.counters[kCntItems];
    float2 mm;
    float4 co, c;
    auto fetch = [&](uint32_t from) {
        if (tid < kBatch && from + tid < n) {
            const uint32_t g = vals[from + tid];
            mm = xy[g];
            co = conic_o[g];
            c = rgb_depth[g];
        }
    };
    fetch(0u);
    for (uint32_t pos = 0; pos < n; pos += kBatch) {
        const int cnt = (int)(n - pos < (uint32_t)kBatch ? n - pos : (uint32_t)kBatch);
        if (tid < cnt) {
            st.a[tid] = fgb::stage_a(mm, co);
            st.b[tid] = fgb::stage_b(co, c);
            st.c[tid] = c.z;
            st.bm[tid] = fgb::block_mask(mm, co, tg.tx, tg.ty, tg.W, tg.H);
        }
        __syncthreads();
        if (pos + kBatch < n) fetch(pos + kBatch);
        if (__ballot(!p.done) != 0ull) {
            const int m = fgb::build_lists(st.bm, cnt, st.list + 8 * wave);
            fgb::wave_sync();
            walk<STATS>(st.a, st.b, st.c, st.list[tid >> 3], m, fpx, fpy, pos, p, f);
        }
        const int alive = __syncthreads_count(!p.done);
        const bool end = pos + kBatch >= n;
        if (ws.state && keep && (end || (pos + kBatch) % CHUNK == 0 || alive == 0)) {
            // once all pixels have stopped, the state after every later chunk equals this one
            uint32_t ch = pos / CHUNK;
            const uint32_t ce = alive == 0 ? nch - 1 : ch;
            for (; ch <= ce && mf + ch < n_items; ch++) {
                float* to = ws.state + (size_t)(mf + ch) * (4 * kThreads) + ly * fgd::kTile + lx;
                to[0] = p.T;
                to[kThreads] = p.C0;
                to[2 * kThreads] = p.C1;
                to[3 * kThreads] = p.C2;
            }
        }
        if (alive == 0) break;
    }
}

// ---- the walk of a long tile ---------------------------------------------------

// alpha of a fragment that passed the skip tests (so -5.6 <= power <= 0). Its
// power is fgb::eval_alpha's, which scales the conic's diagonal by -0.5 before
// the products where this scales their sum: a power of two, exact unless a product
// is denormal, and then the exponential is 1 either way.
__device__ __forceinline__ float passed_alpha(float2 mm, float4 co, float fpx, float fpy)
{
    const float dx = mm.x - fpx;
    const float dy = mm.y - fpy;
    const float power = -0.5f * ((co.x * dx) * dx + (co.z * dy) * dy) - (co.y * dx) * dy;
    const float alpha = co.w * fgd::exp_neg_in_range(power);
    return alpha < 0.99f ? alpha : 0.99f;
}

// Walks the marked splats of one staged chunk for this lane's pixel. mcol
// points at the pixel's first mask word (words STRIDE apart). A summary
// bit per 64-splat pair of words, read first, sends the lane straight to the
// non-empty words. Up to four marked splats of one such word are taken at a
// time and their alphas (independent of T) computed together, so their LDS
// reads and arithmetic overlap; the blend steps then run strictly in list
// order.
//
// The two lanes of a pixel (32 apart) hold the same mask words and state and
// run the same steps in lockstep; lane `sub` of the pixel computes the alphas
// of group positions sub and sub + 2, and the group's alphas are exchanged
// before the blend steps, so each lane evaluates two exponentials per group
// instead of four. Both then apply the same steps to the same values, and the
// results equal a one-lane walk's.
constexpr int kPixels = fgd::kWave / 2;  // pixels per wave

__device__ __forceinline__ void group_alphas(const float2* s_xy, const float4* s_co, float fpx, float fpy, int sub,
                                             int j0, int j1, int j2, int j3, float& a0, float& a1, float& a2,
                                             float& a3)
{
    const int ja = sub ? j1 : j0, jb = sub ? j3 : j2;
    const float ma = passed_alpha(s_xy[ja], s_co[ja], fpx, fpy);
    const float mb = passed_alpha(s_xy[jb], s_co[jb], fpx, fpy);
    const float oa = __shfl_xor(ma, kPixels, fgd::kWave);
    const float ob = __shfl_xor(mb, kPixels, fgd::kWave);
    a0 = sub ? oa : ma;
    a1 = sub ? ma : oa;
    a2 = sub ? ob : mb;
    a3 = sub ? mb : ob;
}

template <int CHUNK, bool STATS>
__device__ __forceinline__ void walk_masks(const uint32_t* mcol, const float2* s_xy, const float4* s_co,
                                     const float4* s_rgb, float fpx, float fpy, uint32_t base, PixelState& p,
                                     Frag& f, int sub)
{
    constexpr int STRIDE = fgd::kWave;
    constexpr int kPairs = CHUNK / 64;
    uint32_t summary = 0;
#pragma unroll
    for (int k = 0; k < kPairs; k++)
        summary |= ((mcol[(2 * k) * STRIDE] | mcol[(2 * k + 1) * STRIDE]) != 0u ? 1u : 0u) << k;
    while (summary != 0u && !p.done) {
        const int k = __builtin_ctz(summary);
        summary &= summary - 1u;
        unsigned long long m = (unsigned long long)mcol[(2 * k) * STRIDE] |
                               ((unsigned long long)mcol[(2 * k + 1) * STRIDE] << 32);
        const int b = k << 6;
        while (m != 0ull && !p.done) {
            const int j0 = b + __builtin_ctzll(m);
            m &= m - 1ull;
            const bool v1 = m != 0ull;
            const int j1 = v1 ? b + __builtin_ctzll(m) : j0;
            m &= m - 1ull;
            const bool v2 = m != 0ull;
            const int j2 = v2 ? b + __builtin_ctzll(m) : j0;
            m &= m - 1ull;
            const bool v3 = m != 0ull;
            const int j3 = v3 ? b + __builtin_ctzll(m) : j0;
            m &= m - 1ull;
            float a0, a1, a2, a3;
            group_alphas(s_xy, s_co, fpx, fpy, sub, j0, j1, j2, j3, a0, a1, a2, a3);
            const float4 c0 = s_rgb[j0], c1 = s_rgb[j1], c2 = s_rgb[j2], c3 = s_rgb[j3];
            blend_step<STATS>(p, true, a0, c0, base + (uint32_t)j0, f);
            blend_step<STATS>(p, v1, a1, c1, base + (uint32_t)j1, f);
            blend_step<STATS>(p, v2, a2, c2, base + (uint32_t)j2, f);
            blend_step<STATS>(p, v3, a3, c3, base + (uint32_t)j3, f);
        }
    }
}

// Register copy of one chunk for one wave of a long tile: the splat records
// this lane stages (every 64th of the chunk) and the mask words of its pixel.
template <int CHUNK>
struct ChunkRegs {
    static constexpr int S = CHUNK / fgd::kWave;
    float2 xy[S];
    float4 co[S];
    float4 rgb[S];
    uint32_t m[CHUNK / 32];
};

template <int CHUNK>
__device__ __forceinline__ int chunk_count(uint32_t r0, uint32_t r1, uint32_t chunk)
{
    const uint32_t start = r0 + chunk * CHUNK;
    return r1 > start ? (int)(r1 - start < (uint32_t)CHUNK ? r1 - start : (uint32_t)CHUNK) : 0;
}

template <int CHUNK>
__device__ __forceinline__ void fetch_vals(const uint32_t* __restrict__ vals, uint32_t r0, uint32_t r1, uint32_t chunk,
                                           uint32_t (&g)[ChunkRegs<CHUNK>::S])
{
    const int cnt = chunk_count<CHUNK>(r0, r1, chunk);
    const uint32_t start = r0 + chunk * CHUNK;
#pragma unroll
    for (int k = 0; k < ChunkRegs<CHUNK>::S; k++) {
        const int j = k * fgd::kWave + fgd::lane_id();
        g[k] = j < cnt ? vals[start + j] : 0u;
    }
}

template <int CHUNK>
__device__ __forceinline__ void fetch_chunk(const float2* __restrict__ xy, const float4* __restrict__ conic_o,
                                            const float4* __restrict__ rgb_depth, const uint32_t* __restrict__ masks,
                                            uint32_t r0, uint32_t r1, uint32_t chunk,
                                            const uint32_t (&g)[ChunkRegs<CHUNK>::S], uint32_t mf,
                                            int pix, ChunkRegs<CHUNK>& R)
{
    const int cnt = chunk_count<CHUNK>(r0, r1, chunk);
#pragma unroll
    for (int k = 0; k < ChunkRegs<CHUNK>::S; k++) {
        const int j = k * fgd::kWave + fgd::lane_id();
        if (j < cnt) {
            R.xy[k] = xy[g[k]];
            R.co[k] = conic_o[g[k]];
            R.rgb[k] = rgb_depth[g[k]];
        } else {
            R.xy[k] = make_float2(0.0f, 0.0f);
            R.co[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            R.rgb[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    const uint32_t* src = masks + (size_t)(mf + chunk) * (CHUNK / 32 * kThreads);
#pragma unroll
    for (int w = 0; w < CHUNK / 32; w++) R.m[w] = src[w * kThreads + pix];
}

// The long tiles, two work items each (the upper and lower 8 pixel rows), 32
// pixels per wave with two lanes per pixel. Each wave walks the chunks for its
// own pixels at its own pace, with its own staging area, so no wave waits on
// the others between chunks. While one chunk is walked, the next chunk's
// splat records and masks are loaded into registers, and the indices of the
// chunk after it. What bounds it is the walk of the longest lists: two lanes
// per pixel in every long tile took 66 us on the 1M-leaf city and 196 us on the
// 20M-node one at 1440p, only from 10 chunks on 101 and 234 us.
template <int CHUNK, bool STATS>
__global__ __launch_bounds__(kThreads) void k_render_long(const float2* __restrict__ xy,
                                                          const float4* __restrict__ conic_o,
                                                          const float4* __restrict__ rgb_depth,
                                                          const uint32_t* __restrict__ vals,
                                                          const uint32_t* __restrict__ ranges, RenderViews V, float bg0,
                                                          float bg1, float bg2, RenderWs ws, float* __restrict__ image,
                                                          float* __restrict__ final_T, uint32_t* __restrict__ n_contrib,
                                                          unsigned long long* __restrict__ frag_stats)
{
    constexpr int kWords = CHUNK / 32;
    constexpr int kWaves = kThreads / fgd::kWave;
    __shared__ float2 s_xy[kWaves * CHUNK];
    __shared__ float4 s_co[kWaves * CHUNK];
    __shared__ float4 s_rgb[kWaves * CHUNK];
    __shared__ uint32_t s_mask[kWords * kThreads];
    const int tid = threadIdx.x;
    const int wave = tid / fgd::kWave, lane = fgd::lane_id();
    const int sub = lane / kPixels;  // this lane's place among its pixel's lanes
    const uint32_t n_work = 2u * ws.counters[kCntHeavy];
    Frag f = {0, 0, 0, 0};
    for (uint32_t item = blockIdx.x; item < n_work; item += gridDim.x) {
        const uint32_t tile = ws.order[item / 2];
        const uint32_t nch = ws.nch[tile], mf = ws.mfirst[tile];
        if (!is_long(ws, nch, mf)) continue;
        const int pix = (int)(item % 2) * (kThreads / 2) + wave * kPixels + lane % kPixels;
        const uint32_t r0 = ranges[2 * tile], r1 = ranges[2 * tile + 1];
        const TileGeom tg = tile_geom(V, tile);
        const int px = tg.tx * fgd::kTile + pix % fgd::kTile, py = tg.ty * fgd::kTile + pix / fgd::kTile;
        const bool inside = px < tg.W && py < tg.H;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        PixelState p = {1.0f, 0.0f, 0.0f, 0.0f, 0u, !inside};
        float2* w_xy = s_xy + wave * CHUNK;
        float4* w_co = s_co + wave * CHUNK;
        float4* w_rgb = s_rgb + wave * CHUNK;
        uint32_t* w_mask = s_mask + wave * (kWords * fgd::kWave);
        ChunkRegs<CHUNK> R;
        uint32_t gnext[ChunkRegs<CHUNK>::S];
        {
            uint32_t g0[ChunkRegs<CHUNK>::S];
            fetch_vals<CHUNK>(vals, r0, r1, 0u, g0);
            fetch_chunk<CHUNK>(xy, conic_o, rgb_depth, ws.masks, r0, r1, 0u, g0, mf, pix, R);
            fetch_vals<CHUNK>(vals, r0, r1, 1u, gnext);
        }
        auto save_state = [&](uint32_t ch) {  // per-pixel state after this chunk, for the backward
            float* st = ws.state + (size_t)(mf + ch) * (4 * kThreads) + pix;
            st[0] = p.T;
            st[kThreads] = p.C0;
            st[2 * kThreads] = p.C1;
            st[3 * kThreads] = p.C2;
        };
        const unsigned n_blend0 = f.n_blend;
        uint32_t chunk = 0;
        for (; chunk < nch; chunk++) {
            // the wave stops once all of its pixels have terminated
            if (__ballot(!p.done) == 0ull) break;
            const int cnt = chunk_count<CHUNK>(r0, r1, chunk);
            fgb::wave_sync();  // the previous chunk's reads are done
#pragma unroll
            for (int k = 0; k < ChunkRegs<CHUNK>::S; k++) {
                const int j = k * fgd::kWave + lane;
                if (j < cnt) {
                    w_xy[j] = R.xy[k];
                    w_co[j] = R.co[k];
                    w_rgb[j] = R.rgb[k];
                }
            }
#pragma unroll
            for (int w = 0; w < kWords; w++) w_mask[w * fgd::kWave + lane] = R.m[w];
            fgb::wave_sync();
            if (chunk + 1 < nch) {
                fetch_chunk<CHUNK>(xy, conic_o, rgb_depth, ws.masks, r0, r1, chunk + 1, gnext, mf, pix, R);
                if (chunk + 2 < nch) fetch_vals<CHUNK>(vals, r0, r1, chunk + 2, gnext);
            }
            walk_masks<CHUNK, STATS>(w_mask + lane, w_xy, w_co, w_rgb, fpx, fpy, chunk * CHUNK, p, f, sub);
            if (ws.state && sub == 0) save_state(chunk);
        }
        if (ws.state && sub == 0)  // the state after every later chunk equals the final one
            for (; chunk < nch; chunk++) save_state(chunk);
        if (STATS && sub != 0) f.n_blend = n_blend0;  // a pixel's blends count on its first lane only
        if (inside && sub == 0) write_pixel(p, px, py, tg, bg0, bg1, bg2, image, final_T, n_contrib);
    }
    flush_stats<STATS, 4>(f, frag_stats);
}

// The first mask_blocks workgroups make the long tiles' pass masks; the others
// blend the tiles that hold splats and are not long, from the first-th on, one
// each, heavy ones first (those past the last find nothing). One launch, since the two need
// nothing of each other and neither fills the chip by itself in most frames.
// The dispatcher balances the tiles: a work ticket (one atomic per tile, all
// on one address) took longer than the tiles themselves in frames of few
// splats.
template <int CHUNK, bool STATS>
__global__ __launch_bounds__(kThreads) void k_render(const float2* __restrict__ xy, const float4* __restrict__ conic_o,
                                                     const float4* __restrict__ rgb_depth,
                                                     const uint32_t* __restrict__ vals,
                                                     const uint32_t* __restrict__ ranges, int64_t n_tiles,
                                                     RenderViews V, float bg0, float bg1, float bg2, RenderWs ws,
                                                     uint32_t mask_blocks, uint32_t first, float* __restrict__ image,
                                                     float* __restrict__ final_T, uint32_t* __restrict__ n_contrib,
                                                     unsigned long long* __restrict__ frag_stats)
{
    __shared__ union {
        Staged st;
        uint32_t mask[CHUNK / 32 * kThreads];
    } s;
    if (blockIdx.x < mask_blocks) {
        make_masks<CHUNK, STATS>(s.mask, blockIdx.x, mask_blocks, xy, conic_o, vals, ranges, V, ws, frag_stats);
        return;
    }
    const uint32_t item = first + (blockIdx.x - mask_blocks), n_heavy = ws.counters[kCntHeavy];
    if (item >= ws.counters[kCntTiles]) return;
    const bool heavy = item < n_heavy;
    const uint32_t tile = ws.order[heavy ? (int64_t)item : n_tiles - 1 - (int64_t)(item - n_heavy)];
    const uint32_t nch = ws.nch[tile];
    const uint32_t mf = heavy ? ws.mfirst[tile] : 0u;
    if (heavy && is_long(ws, nch, mf)) return;
    const uint32_t r0 = ranges[2 * tile], n = ranges[2 * tile + 1] - r0;
    const TileGeom tg = tile_geom(V, tile);
    const int px = tg.tx * fgd::kTile + fgb::pixel_x(threadIdx.x), py = tg.ty * fgd::kTile + fgb::pixel_y(threadIdx.x);
    const bool inside = px < tg.W && py < tg.H;
    PixelState p = {1.0f, 0.0f, 0.0f, 0.0f, 0u, !inside};
    Frag f = {0, 0, 0, 0};
    blend_batches<CHUNK, STATS>(s.st, ws, xy, conic_o, rgb_depth, vals + r0, n, heavy, nch, mf, tg, p, f);
    if (inside) write_pixel(p, px, py, tg, bg0, bg1, bg2, image, final_T, n_contrib);
    flush_stats<STATS, 4>(f, frag_stats);
}

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int chunk_of(const fg_tune* tune)
{
    if (!tune || !tune->render_batch) return 256;
    return tune->render_batch;
}

// The mask store is capped; long tiles past it are walked whole by one
// workgroup (same results, less parallelism).
constexpr int64_t kMaskStoreBytes = (int64_t)512 << 20;

size_t carve(void* base, int64_t n_tiles, int64_t cap_pairs, int chunk, bool save_state, int mask_items,
             RenderWs* w, int64_t* max_items)
{
    const int64_t mask_bytes = (int64_t)(chunk / 32) * kThreads * 4;
    const int64_t need = 2 * ((cap_pairs + chunk - 1) / chunk) + 1;
    int64_t cap = kMaskStoreBytes / mask_bytes;
    if (mask_items > 0 && mask_items < cap) cap = mask_items;
    *max_items = need < cap ? need : cap;
    const size_t state_bytes = save_state ? (size_t)*max_items * 4 * kThreads * 4 : 0;
    const size_t sched_bytes = (size_t)kSchedWords * 4 * (size_t)((n_tiles + kSchedTiles - 1) / kSchedTiles + 1);
    const size_t sizes[8] = {(size_t)n_tiles * 4, (size_t)n_tiles * 4, (size_t)n_tiles * 4, (size_t)*max_items * 4, 64,
                             (size_t)*max_items * (size_t)mask_bytes, state_bytes, sched_bytes};
    void** dst[8] = {(void**)&w->nch, (void**)&w->mfirst, (void**)&w->order, (void**)&w->mitem, (void**)&w->counters,
                     (void**)&w->masks, (void**)&w->state, (void**)&w->sched};
    size_t off = 0;
    for (int i = 0; i < 8; i++) {
        if (base) *dst[i] = (char*)base + off;
        off += align_up(sizes[i] + 4);
    }
    if (base && !save_state) w->state = nullptr;
    return off;
}

bool save_of(const fg_tune* tune) { return tune && tune->save_state; }

int mask_items_of(const fg_tune* tune) { return tune ? tune->mask_items : 0; }

template <int CHUNK>
void launch(const fg_splats* splats, const uint32_t* vals, const uint32_t* ranges, const RenderViews& V,
            const float bg[3], float* image, float* final_T, uint32_t* n_contrib, unsigned long long* frag_stats,
            const RenderWs& w, int64_t n_tiles, int64_t max_mask_items, const fg_tune* tune, hipStream_t s)
{
    if (n_tiles <= 4 * kSchedTiles) {
        hipLaunchKernelGGL(k_schedule<CHUNK>, dim3(1), dim3(kScanThreads), 0, s, ranges, n_tiles, max_mask_items,
                           w.nch, w.mfirst, w.order, w.counters);
    } else {
        const int64_t nb = (n_tiles + kSchedTiles - 1) / kSchedTiles;
        hipLaunchKernelGGL(k_sched_count<CHUNK>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, ranges, n_tiles, w.nch,
                           w.sched);
        hipLaunchKernelGGL(k_sched_scan, dim3(1), dim3(64), 0, s, w.sched, nb, CHUNK, max_mask_items, w.counters);
        hipLaunchKernelGGL(k_sched_write<CHUNK>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, n_tiles, w.nch,
                           w.sched, w.mfirst, w.order);
    }
    const int per_wg = n_tiles <= 4 * kSchedTiles ? 1 : 4;
    const int64_t preps = (n_tiles + per_wg - 1) / per_wg;
    const unsigned gp = (unsigned)(preps < 65536 ? preps : 65536);
    hipLaunchKernelGGL(k_tile_prep, dim3(gp), dim3(kThreads), 0, s, n_tiles, per_wg, V, bg[0], bg[1], bg[2], w,
                       max_mask_items, image, final_T, n_contrib);
    const float2* xy = (const float2*)splats->xy;
    const float4* co = (const float4*)splats->conic_o;
    const float4* rgb = (const float4*)splats->rgb_depth;
    const unsigned gm = (unsigned)(max_mask_items < 2048 ? (max_mask_items < 1 ? 1 : max_mask_items) : 2048);
    const unsigned gl = (unsigned)(2 * n_tiles < 4096 ? 2 * n_tiles : 4096);
    // a grid holds fewer than 2^32 threads: one launch up to 16.7 million tiles
    auto blend = [&](auto kernel) {
        const int64_t most = (((int64_t)1 << 32) - 1) / kThreads;
        unsigned masks = gm;
        for (int64_t t = 0; t < n_tiles;) {
            const int64_t n = n_tiles - t < most - masks ? n_tiles - t : most - masks;
            hipLaunchKernelGGL(kernel, dim3(masks + (unsigned)n), dim3(kThreads), 0, s, xy, co, rgb, vals, ranges, n_tiles,
                               V, bg[0], bg[1], bg[2], w, masks, (uint32_t)t, image, final_T, n_contrib, frag_stats);
            t += n;
            masks = 0;
        }
    };
    auto blend_long = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(gl), dim3(kThreads), 0, s, xy, co, rgb, vals, ranges, V, bg[0], bg[1], bg[2], w,
                           image, final_T, n_contrib, frag_stats);
    };
    if (frag_stats) {
        blend(k_render<CHUNK, true>);
        blend_long(k_render_long<CHUNK, true>);
    } else {
        const bool timed = tune && tune->blend_events[0] && tune->blend_events[1];
        if (timed) (void)hipEventRecord((hipEvent_t)tune->blend_events[0], s);
        blend(k_render<CHUNK, false>);
        blend_long(k_render_long<CHUNK, false>);
        if (timed) (void)hipEventRecord((hipEvent_t)tune->blend_events[1], s);
    }
}

}  // namespace

namespace {

// The views' geometry and total tile count (-1: invalid views: sizes, more
// than kMaxViews, or global tile ids that are not consecutive from view to
// view).
int64_t make_views(const fg_camera* cams, int32_t n_views, RenderViews* V)
{
    if (!cams || n_views < 1 || n_views > kMaxViews) return -1;
    int64_t total = 0, pix = 0;
    V->n = n_views;
    for (int v = 0; v < n_views; v++) {
        const fg_camera& c = cams[v];
        if (c.width <= 0 || c.height <= 0) return -1;
        if ((int64_t)c.tile_base != (int64_t)cams[0].tile_base + total) return -1;
        V->tile0[v] = (uint32_t)total;
        V->W[v] = c.width;
        V->H[v] = c.height;
        V->Wt[v] = (c.width + 15) / 16;
        V->pix0[v] = pix;
        total += (int64_t)V->Wt[v] * ((c.height + 15) / 16);
        pix += (int64_t)c.width * c.height;
        if (total >= ((int64_t)1 << 31)) return -1;
    }
    V->tile0[n_views] = (uint32_t)total;
    for (int v = n_views; v < kMaxViews; v++) {
        V->tile0[v + 1] = (uint32_t)total;
        V->W[v] = V->H[v] = V->Wt[v] = 1;
        V->pix0[v] = pix;
    }
    return total;
}

}  // namespace

extern "C" size_t fg_render_workspace_size(const fg_camera* cams, int32_t n_views, int64_t cap_pairs,
                                           const fg_tune* tune)
{
    RenderViews V;
    const int64_t n_tiles = make_views(cams, n_views, &V);
    if (n_tiles < 0 || cap_pairs < 0) return 0;
    RenderWs w;
    int64_t mi;
    return carve(nullptr, n_tiles, cap_pairs, chunk_of(tune), save_of(tune), mask_items_of(tune), &w, &mi);
}

extern "C" int fg_render(const fg_splats* splats, const uint32_t* vals, const uint32_t* ranges,
                         const fg_camera* cams, int32_t n_views, const float bg[3], float* image, float* final_T,
                         uint32_t* n_contrib, int64_t cap_pairs, unsigned long long* frag_stats, uint32_t* status,
                         void* ws, size_t ws_bytes, const fg_tune* tune, void* stream)
{
    (void)status;
    if (!splats || !ranges || !cams || !bg || !image || !final_T || !n_contrib || cap_pairs < 0)
        return FG_ERR_INVALID_ARG;
    RenderViews V;
    const int64_t n_tiles = make_views(cams, n_views, &V);
    if (n_tiles < 0) return FG_ERR_INVALID_ARG;
    const int chunk = chunk_of(tune);
    if (chunk != 128 && chunk != 256 && chunk != 512) return FG_ERR_INVALID_ARG;
    RenderWs w;
    int64_t max_mask_items;
    const bool save = save_of(tune);
    if (!ws || ws_bytes < carve(nullptr, n_tiles, cap_pairs, chunk, save, mask_items_of(tune), &w, &max_mask_items))
        return FG_ERR_WORKSPACE;
    carve(ws, n_tiles, cap_pairs, chunk, save, mask_items_of(tune), &w, &max_mask_items);
    hipStream_t s = (hipStream_t)stream;
    switch (chunk) {
        case 128: launch<128>(splats, vals, ranges, V, bg, image, final_T, n_contrib, frag_stats, w, n_tiles,
                              max_mask_items, tune, s); break;
        case 512: launch<512>(splats, vals, ranges, V, bg, image, final_T, n_contrib, frag_stats, w, n_tiles,
                              max_mask_items, tune, s); break;
        default: launch<256>(splats, vals, ranges, V, bg, image, final_T, n_contrib, frag_stats, w, n_tiles,
                             max_mask_items, tune, s); break;
    }
    return hipGetLastError() == hipSuccess ? FG_OK : FG_ERR_HIP;
}

namespace fgr {

bool render_ws_view(const void* ws, size_t ws_bytes, const fg_camera* cam, int64_t cap_pairs, const fg_tune* tune,
                    RenderWsView* v)
{
    if (!ws || !cam || !v || !save_of(tune) || cam->width <= 0 || cam->height <= 0 || cap_pairs < 0) return false;
    const int chunk = chunk_of(tune);
    if (chunk != 128 && chunk != 256 && chunk != 512) return false;
    const int64_t n_tiles = (int64_t)((cam->width + 15) / 16) * ((cam->height + 15) / 16);
    RenderWs w;
    int64_t mi;
    if (ws_bytes < carve(nullptr, n_tiles, cap_pairs, chunk, true, mask_items_of(tune), &w, &mi)) return false;
    carve(const_cast<void*>(ws), n_tiles, cap_pairs, chunk, true, mask_items_of(tune), &w, &mi);
    v->nch = w.nch;
    v->mfirst = w.mfirst;
    v->mitem = w.mitem;
    v->counters = w.counters + kCntItems;
    v->state = w.state;
    v->chunk = chunk;
    v->max_items = mi;
    return true;
}

}  // namespace fgr

extern "C" const char* fg_status_string(int code)
{
    switch (code) {
        case FG_OK: return "ok";
        case FG_ERR_INVALID_ARG: return "invalid argument";
        case FG_ERR_INVALID_TREE: return "invalid tree";
        case FG_ERR_UNSUPPORTED: return "unsupported configuration";
        case FG_ERR_WORKSPACE: return "workspace too small";
        case FG_ERR_HIP: return "HIP launch or runtime error";
        case FG_ERR_SCRATCH: return "problem larger than the fixed scratch array of fg_filter_noalloc";
        default: return "unknown status";
    }
}
