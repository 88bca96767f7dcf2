// GTC pre-pass (Sec. 3.3, Fig. 2(b)): the key-value pair contribution of every
// Gaussian-tile pair of a rendered view (Eq. (5)), the Gaussian-to-tile
// contribution of every tile (Eq. (6)), the view's mean over its tiles
// (Eq. (7)), and the scene threshold tau = lambda_G / G_bar over several views
// (Eq. (8)).
//
//   k_kpc       one workgroup per tile. The tile's sorted splats are staged
//               128 at a time in LDS and listed per 4 x 2 pixel block
//               (fg_blocks.h); every 8 lanes walk their own block's list front
//               to back with the blend's own tests (power, alpha skip,
//               termination), and the alpha * T of the blended fragments is
//               summed in one fixed tree (see Staged).
//               A wave stops once its pixels have all terminated; when the
//               whole tile has terminated the remaining pairs get 0 without
//               being visited. The pair sums go to kpc[], their mean over the
//               tile's pairs to tile_gtc[t] (Eq. (6): pairs with zero
//               contribution count), and the tiles with pairs add their G_t
//               and their number to the view's two float64 accumulators.
//   k_kpc_items the same KPC when the view was blended with saved
//               per-chunk state: the chunks of long lists walk in parallel
//               from the saved transmittance, the other tiles whole;
//               k_tile_gtc then forms each tile's GTC from the pairs' KPC.
//   k_gtc_view  turns the accumulators into the view GTC of Eq. (7).
//   k_gtc_tau   mean of the view GTCs over the views that hold pairs, and
//               tau = lambda_G / G_bar.
//
// The transmittance chain is the blend's, in the same binary32 operations, so
// the set of blended fragments and each alpha * T are those of the sequential
// definition; only the summation order of a pair's terms differs. That order is
// fixed, so a pair's KPC is the same in every run and in both walks.
#include "fg_blocks.h"
#include "fg_device.h"
#include "fg_render_ws.h"

namespace {

constexpr int kThreads = 256;
constexpr int kMaxEdges = 16;

struct Edges {
    float e[kMaxEdges];
    int n;
};

// LDS of a KPC walk: the staged splats, their block bits, the block lists and
// the partial sums of alpha * T. A splat's 256 terms meet in one fixed tree:
// four pixels of a row ((0 + 1) + (2 + 3), by DPP), the four such quads of a row
// ((0 + 1) + (2 + 3)), a wave's four rows ((0 + 1) + (2 + 3)), then the waves
// one after another: 9 roundings. Every block writes its two quads to their own
// places, since its neighbours reach the same splat at other steps. Adding
// the blocks' sums to one LDS float instead took up to 34 roundings, in an order
// that changed from run to run. The quads' places are what limits the batch:
// 128 splats let four workgroups share a CU's LDS.
constexpr int kBatch = 128;
constexpr int kWaves = kThreads / fgd::kWave;

struct Staged {
    float4 a[kBatch];
    float2 b[kBatch];  // -C / 2, opacity
    uint32_t bm[kBatch];
    // [wave][row][splat]: its four quads; zero where no pixel of the quad blends it
    float4 quad[kWaves][4][kBatch];
    __align__(16) uint8_t list[fgb::kBlocks][kBatch];
};

__device__ __forceinline__ void clear_quads(Staged& st)
{
    float4* q = &st.quad[0][0][0];
    for (int i = threadIdx.x; i < kWaves * 4 * kBatch; i += kThreads) q[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__device__ __forceinline__ void stage(Staged& st, int i, uint32_t g, const float2* __restrict__ xy,
                                      const float4* __restrict__ conic_o, int tx, int ty, int W, int H)
{
    const float2 mm = xy[g];
    const float4 co = conic_o[g];
    st.a[i] = fgb::stage_a(mm, co);
    st.b[i] = make_float2(-0.5f * co.z, co.w);
    st.bm[i] = fgb::block_mask(mm, co, tx, ty, W, H);
}

// Walks this lane's block list of m entries from transmittance T; TERM: until
// the pixel terminates (Eq. (2)), else up to the list position last. Writes
// each splat's alpha * T over the block's two quads. Four alphas (independent of
// T) are computed together, the T chain then runs in list order.
template <bool TERM>
__device__ __forceinline__ void walk(Staged& st, const uint8_t* list, int m, float fpx, float fpy, uint32_t pos,
                                     uint32_t last, float& T, bool& done)
{
    const int lane = fgd::lane_id();
    // this lane's quad: row ((lane >> 5) << 1) + ((lane >> 2) & 1) of its wave, place (lane >> 3) & 3
    float* quad = &st.quad[threadIdx.x / fgd::kWave][((lane >> 4) & 2) | ((lane >> 2) & 1)][0].x + ((lane >> 3) & 3);
    for (int k = 0; k < m; k += 4) {
        const uint32_t e4 = *reinterpret_cast<const uint32_t*>(list + k);
        float alpha[4];
        bool hit[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int j = (int)((e4 >> (8 * u)) & (uint32_t)(kBatch - 1));  // past m the byte is any
            const float4 a = st.a[j];
            const float2 b = st.b[j];
            bool in_range;
            hit[u] = fgb::eval_alpha(a, make_float4(b.x, b.y, 0.f, 0.f), fpx, fpy, alpha[u], in_range) && k + u < m;
            if (!TERM) hit[u] = hit[u] && pos + (uint32_t)j < last;
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            float c = 0.0f;
            if (hit[u] && !(TERM && done)) {
                const float Tn = T * (1.0f - alpha[u]);
                if (TERM && Tn < 1e-4f) {
                    done = true;  // stops before this splat
                } else {
                    c = alpha[u] * T;
                    T = Tn;
                }
            }
            if (__ballot(c != 0.0f) == 0ull) continue;
            c += fgd::dpp_mov<0xB1>(c);  // lane bit 0
            c += fgd::dpp_mov<0x4E>(c);  // lane bit 1
            if ((lane & 3) == 0 && c != 0.0f) quad[4 * ((e4 >> (8 * u)) & (uint32_t)(kBatch - 1))] = c;
        }
        if (TERM && __ballot(!done) == 0ull) break;
    }
}

// After a wave's walk of cnt staged splats: its sum of each, left in the first
// place of the splat's first row; the other places are zero again.
__device__ __forceinline__ void wave_sums(Staged& st, int cnt)
{
    const int wave = threadIdx.x / fgd::kWave;
    for (int j = fgd::lane_id(); j < cnt; j += fgd::kWave) {
        if (((st.bm[j] >> (8 * wave)) & 255u) == 0u) continue;  // in none of the wave's lists
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float4 q = st.quad[wave][i][j];
            r[i] = (q.x + q.y) + (q.z + q.w);
            if (i) st.quad[wave][i][j] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        st.quad[wave][0][j] = make_float4((r[0] + r[1]) + (r[2] + r[3]), 0.f, 0.f, 0.f);
    }
}

// The sum of splat j over the waves; its places are zero again.
__device__ __forceinline__ float pair_sum(Staged& st, int j)
{
    float k = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
        k += st.quad[w][0][j].x;
        st.quad[w][0][j].x = 0.0f;
    }
    return k;
}

template <bool HIST>
__global__ __launch_bounds__(kThreads) void k_kpc(const float2* __restrict__ xy, const float4* __restrict__ conic_o,
                                                  const uint32_t* __restrict__ vals,
                                                  const uint32_t* __restrict__ ranges,
                                                  const uint32_t* __restrict__ n_pairs, int64_t n_tiles,
                                                  int64_t cap_pairs, int W, int H, int Wt,
                                                  float* __restrict__ kpc, float* __restrict__ tile_gtc,
                                                  double* __restrict__ acc, Edges edges,
                                                  uint32_t* __restrict__ hist)
{
    __shared__ Staged st;
    __shared__ double s_red[kThreads / fgd::kWave];
    __shared__ uint32_t s_hist[kMaxEdges + 1];

    const int tid = threadIdx.x;
    const int lane = fgd::lane_id();
    const int wave = tid / fgd::kWave;
    const int lx = fgb::pixel_x(tid), ly = fgb::pixel_y(tid);
    // the pairs of a sort that overflowed its capacity are incomplete: every
    // tile is then left undefined and the view is marked (acc[1] < 0)
    const bool overflow = (int64_t)*n_pairs > cap_pairs;
    double g_sum = 0.0, g_num = 0.0;  // thread 0: this workgroup's tiles
    clear_quads(st);
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const int tx = (int)(t % Wt), ty = (int)(t / Wt);
        uint32_t lo = ranges[2 * t], hi = ranges[2 * t + 1];
        if (overflow || (int64_t)hi > cap_pairs || lo > hi) lo = hi = 0;
        const uint32_t n = hi - lo;
        if (n == 0) {
            if (tid == 0) tile_gtc[t] = __int_as_float(0x7fc00000);  // Eq. (6) is 0/0: undefined
            continue;
        }
        if (HIST && tid <= edges.n) s_hist[tid] = 0u;
        const int px = tx * fgd::kTile + lx;
        const int py = ty * fgd::kTile + ly;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        bool done = !(px < W && py < H);
        float T = 1.0f;
        double my_sum = 0.0;  // this thread's share of the tile's KPC sum
        for (uint32_t b = 0; b < n; b += kBatch) {
            const int cnt = (int)(n - b < (uint32_t)kBatch ? n - b : (uint32_t)kBatch);
            if (tid < cnt) stage(st, tid, vals[lo + b + tid], xy, conic_o, tx, ty, W, H);
            __syncthreads();
            if (__ballot(!done) != 0ull) {
                const int m = fgb::build_lists(st.bm, cnt, st.list + 8 * wave);
                fgb::wave_sync();
                walk<true>(st, st.list[tid >> 3], m, fpx, fpy, b, 0u, T, done);
                fgb::wave_sync();
                wave_sums(st, cnt);
            }
            __syncthreads();
            // thread t sums the tile's pairs t, t + 256, ...
            const int j = tid - (int)(b % kThreads);
            if (j >= 0 && j < cnt) {
                const float k = pair_sum(st, j);
                kpc[lo + b + j] = k;
                my_sum += (double)k;
                if (HIST) {
                    int bin = 0;
                    while (bin < edges.n && k >= edges.e[bin]) bin++;
                    atomicAdd(&s_hist[bin], 1u);
                }
            }
            const int alive = __syncthreads_count(!done);
            if (alive == 0 && b + kBatch < n) {
                // the whole tile has terminated: the remaining pairs contribute nothing
                for (uint32_t k = b + kBatch + tid; k < n; k += kThreads) kpc[lo + k] = 0.0f;
                if (HIST && tid == 0) {
                    int bin = 0;
                    while (bin < edges.n && 0.0f >= edges.e[bin]) bin++;
                    atomicAdd(&s_hist[bin], n - (b + kBatch));
                }
                break;
            }
        }
        // tile sum in float64: wave sums through LDS, then one thread
        double v = my_sum;
        for (int off = fgd::kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, fgd::kWave);
        if (lane == 0) s_red[wave] = v;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < kThreads / fgd::kWave; w++) s += s_red[w];
            const double G = s / (double)n;
            tile_gtc[t] = (float)G;
            g_sum += G;
            g_num += 1.0;
        }
        if (HIST && tid <= edges.n && s_hist[tid]) atomicAdd(&hist[tid], s_hist[tid]);
        __syncthreads();
    }
    if (tid == 0 && g_num != 0.0) {
        atomicAdd(&acc[0], g_sum);
        atomicAdd(&acc[1], g_num);
    }
}

// The same per-pair KPC from the blend's saved state, with the long ranges
// split into their chunks: work items are the chunk items of the tiles whose
// every chunk has saved state (each walked from the transmittance the blend
// had after the previous chunk) and whole tiles otherwise (walked from
// T = 1). A fragment at list position pos is blended by a pixel exactly when
// pos is below the pixel's contributor count and it passes the skip tests,
// so the walk needs no termination test, and a chunk does not wait for the
// ones before it. The fragments, their alpha * T and each splat's sum are those
// of k_kpc, bit for bit (the transmittance chain is the blend's, in the same
// operations). Only the per-pair KPC is written here;
// k_tile_gtc then sums each tile's pairs in k_kpc's order. The arithmetic of
// the walk and the short lists of small batches bound it: per view of the
// 20M-node scene at 1080p it took 792 us with 64 lanes per splat and takes 359
// with 8 (236 with batches of 256 and each block's sum added to one LDS float,
// whose rounding was neither bounded by 9 steps nor the same in every run;
// batches of 64 take as long as 128, of 256 583 us).
__global__ __launch_bounds__(kThreads) void k_kpc_items(const float2* __restrict__ xy,
                                                        const float4* __restrict__ conic_o,
                                                        const uint32_t* __restrict__ vals,
                                                        const uint32_t* __restrict__ ranges,
                                                        const uint32_t* __restrict__ n_pairs, int64_t n_tiles,
                                                        int64_t cap_pairs, int W, int H, int Wt,
                                                        const uint32_t* __restrict__ n_contrib,
                                                        fgr::RenderWsView view, float* __restrict__ kpc)
{
    __shared__ Staged st;
    __shared__ uint32_t s_max;

    const int tid = threadIdx.x;
    const int lane = fgd::lane_id();
    const int wave = tid / fgd::kWave;
    const int lx = fgb::pixel_x(tid), ly = fgb::pixel_y(tid);
    if ((int64_t)*n_pairs > cap_pairs) return;  // incomplete pairs: k_tile_gtc marks the view
    clear_quads(st);
    int64_t n_chunk_items = (int64_t)*view.counters;
    if (n_chunk_items > view.max_items) n_chunk_items = view.max_items;
    for (int64_t item = blockIdx.x; item < n_chunk_items + n_tiles; item += gridDim.x) {
        uint32_t tile;
        int64_t lo, hi;  // positions in the tile's list
        int64_t citem = -1;
        const uint32_t* rg;
        if (item < n_chunk_items) {
            tile = view.mitem[item];
            if ((int64_t)tile >= n_tiles) continue;  // a map this frame's blend did not write
            if ((int64_t)view.mfirst[tile] + view.nch[tile] > n_chunk_items) continue;  // walked whole
            rg = ranges + 2 * (int64_t)tile;
            lo = (int64_t)(item - view.mfirst[tile]) * view.chunk;
            hi = lo + view.chunk;
            citem = item;
        } else {
            tile = (uint32_t)(item - n_chunk_items);
            if (view.nch[tile] > 1 && (int64_t)view.mfirst[tile] + view.nch[tile] <= n_chunk_items) continue;
            rg = ranges + 2 * (int64_t)tile;
            lo = 0;
            hi = INT64_MAX;
        }
        const uint32_t r0 = rg[0], r1 = rg[1];
        if ((int64_t)r1 > cap_pairs || r0 > r1) continue;
        const int64_t n = (int64_t)(r1 - r0);
        if (hi > n) hi = n;
        if (lo >= hi) continue;
        const int tx = (int)(tile % (uint32_t)Wt), ty = (int)(tile / (uint32_t)Wt);
        const int px = tx * fgd::kTile + lx;
        const int py = ty * fgd::kTile + ly;
        const bool inside = px < W && py < H;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        const uint32_t last = inside ? n_contrib[(size_t)py * W + px] : 0u;
        // the transmittance after the previous chunk, as the blend saved it
        float T = citem > (int64_t)view.mfirst[tile] ? view.state[(size_t)(citem - 1) * (4 * kThreads) + ly * fgd::kTile + lx] : 1.0f;
        __syncthreads();  // LDS of the previous item
        if (tid == 0) s_max = 0u;
        __syncthreads();
        uint32_t wlast = last;
#pragma unroll
        for (int d = fgd::kWave / 2; d > 0; d >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)wlast, d, fgd::kWave);
            wlast = o > wlast ? o : wlast;
        }
        if (lane == 0) atomicMax(&s_max, wlast);
        __syncthreads();
        // every blended fragment of the tile lies below s_max
        const int64_t end = hi < (int64_t)s_max ? hi : (int64_t)s_max;
        for (int64_t b = lo; b < end; b += kBatch) {
            const int cnt = (int)(end - b < kBatch ? end - b : kBatch);
            if (tid < cnt) stage(st, tid, vals[r0 + b + tid], xy, conic_o, tx, ty, W, H);
            __syncthreads();
            if (b < (int64_t)wlast) {  // some pixel of this wave blends in this batch
                const int m = fgb::build_lists(st.bm, cnt, st.list + 8 * wave);
                fgb::wave_sync();
                bool done = false;
                walk<false>(st, st.list[tid >> 3], m, fpx, fpy, (uint32_t)b, last, T, done);
                fgb::wave_sync();
                wave_sums(st, cnt);
            }
            __syncthreads();
            if (tid < cnt) kpc[r0 + b + tid] = pair_sum(st, tid);
            __syncthreads();
        }
        // pairs behind every pixel's last blended fragment contribute nothing
        for (int64_t k = (end > lo ? end : lo) + tid; k < hi; k += kThreads) kpc[r0 + k] = 0.0f;
    }
}

// Eq. (6) from the per-pair KPC: one workgroup per tile sums its pairs in
// float64 in k_kpc's order (thread t the pairs t, t + 256, ..., then the
// wave sums through LDS); with edges, the pairs' KPC histogram. Additions to
// one address are served one after another, so a workgroup takes several tiles
// and adds their G_t and number to the view's accumulators once: with a pair of
// additions per tile (8160 at 1080p) this took 179 us per view, with 512
// workgroups 35 us (256: 49, 1024: 39, 2048: 59).
constexpr unsigned kTileBlocks = 512;

template <bool HIST>
__global__ __launch_bounds__(kThreads) void k_tile_gtc(const uint32_t* __restrict__ ranges,
                                                       const uint32_t* __restrict__ n_pairs, int64_t n_tiles,
                                                       int64_t cap_pairs, const float* __restrict__ kpc,
                                                       float* __restrict__ tile_gtc, double* __restrict__ acc,
                                                       Edges edges, uint32_t* __restrict__ hist)
{
    __shared__ double s_red[kThreads / fgd::kWave];
    __shared__ uint32_t s_hist[kMaxEdges + 1];
    const int tid = threadIdx.x;
    const int lane = fgd::lane_id();
    const int wave = tid / fgd::kWave;
    const bool overflow = (int64_t)*n_pairs > cap_pairs;
    double g_sum = 0.0, g_num = 0.0;  // thread 0: this workgroup's tiles
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        uint32_t lo = ranges[2 * t], hi = ranges[2 * t + 1];
        if (overflow || (int64_t)hi > cap_pairs || lo > hi) lo = hi = 0;
        const uint32_t n = hi - lo;
        if (n == 0) {
            if (tid == 0) tile_gtc[t] = __int_as_float(0x7fc00000);  // Eq. (6) is 0/0: undefined
            continue;
        }
        if (HIST && tid <= edges.n) s_hist[tid] = 0u;
        __syncthreads();
        double my_sum = 0.0;
        for (uint32_t k = tid; k < n; k += kThreads) {
            const float v = kpc[lo + k];
            my_sum += (double)v;
            if (HIST) {
                int bin = 0;
                while (bin < edges.n && v >= edges.e[bin]) bin++;
                atomicAdd(&s_hist[bin], 1u);
            }
        }
        double v = my_sum;
        for (int off = fgd::kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, fgd::kWave);
        if (lane == 0) s_red[wave] = v;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < kThreads / fgd::kWave; w++) s += s_red[w];
            const double G = s / (double)n;
            tile_gtc[t] = (float)G;
            g_sum += G;
            g_num += 1.0;
        }
        if (HIST && tid <= edges.n && s_hist[tid]) atomicAdd(&hist[tid], s_hist[tid]);
        __syncthreads();
    }
    if (tid == 0 && g_num != 0.0) {
        atomicAdd(&acc[0], g_sum);
        atomicAdd(&acc[1], g_num);
    }
}

__global__ void k_gtc_zero(double* __restrict__ acc)
{
    if (threadIdx.x < 2) acc[threadIdx.x] = 0.0;
}

// Eq. (7): mean of the tile GTCs over the tiles holding pairs; acc[1] keeps
// their number (0: undefined view, acc[0] = 0; -1: the sort overflowed).
__global__ void k_gtc_view(double* __restrict__ acc, const uint32_t* __restrict__ n_pairs, int64_t cap_pairs)
{
    if (threadIdx.x != 0) return;
    if ((int64_t)*n_pairs > cap_pairs) {
        acc[0] = __longlong_as_double(0x7ff8000000000000ll);
        acc[1] = -1.0;
        return;
    }
    acc[0] = acc[1] > 0.0 ? acc[0] / acc[1] : 0.0;
}

// Eq. (8): G_bar over the views with pairs, tau = lambda_G / G_bar.
__global__ void k_gtc_tau(const double* __restrict__ view_gtc, int n_views, float lambda_G,
                          double* __restrict__ g_bar, float* __restrict__ tau, uint32_t* __restrict__ status)
{
    if (threadIdx.x != 0) return;
    double s = 0.0;
    int m = 0;
    bool overflow = false;
    for (int v = 0; v < n_views; v++) {
        if (view_gtc[2 * v + 1] < 0.0) overflow = true;
        if (view_gtc[2 * v + 1] > 0.0) {
            s += view_gtc[2 * v];
            m++;
        }
    }
    if (overflow) {
        *g_bar = __longlong_as_double(0x7ff8000000000000ll);
        *tau = __int_as_float(0x7fc00000);
        if (status) atomicOr(status, FG_STATUS_PAIR_OVERFLOW);
        return;
    }
    if (m == 0) {
        *g_bar = 0.0;
        *tau = __int_as_float(0x7fc00000);
        if (status) atomicOr(status, FG_STATUS_GTC_UNDEFINED);
        return;
    }
    const double G = s / (double)m;
    *g_bar = G;
    *tau = (float)((double)lambda_G / G);
}

}  // namespace

extern "C" int fg_gtc(const fg_splats* splats, const uint32_t* vals, const uint32_t* ranges, const fg_camera* cam,
                      const uint32_t* n_pairs, int64_t cap_pairs, float* kpc, float* tile_gtc, double* view_gtc, const float* hist_edges,
                      int32_t n_edges, uint32_t* kpc_hist, const uint32_t* n_contrib, const void* render_ws,
                      size_t render_ws_bytes, const fg_tune* tune, void* stream)
{
    if (!splats || !vals || !ranges || !cam || !n_pairs || !kpc || !tile_gtc || !view_gtc || cap_pairs < 0)
        return FG_ERR_INVALID_ARG;
    if (cam->width <= 0 || cam->height <= 0) return FG_ERR_INVALID_ARG;
    if (n_edges < 0 || n_edges > kMaxEdges || (n_edges > 0 && (!hist_edges || !kpc_hist)) ||
        (kpc_hist && n_edges == 0))
        return FG_ERR_INVALID_ARG;
    Edges e{};
    e.n = n_edges;
    for (int i = 0; i < n_edges; i++) {
        e.e[i] = hist_edges[i];
        if (i > 0 && !(e.e[i] > e.e[i - 1])) return FG_ERR_INVALID_ARG;
    }
    const int Wt = (cam->width + 15) / 16;
    const int64_t n_tiles = (int64_t)Wt * ((cam->height + 15) / 16);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_gtc_zero, dim3(1), dim3(64), 0, s, view_gtc);
    const unsigned grid = (unsigned)(n_tiles < 65536 ? (n_tiles < 1 ? 1 : n_tiles) : 65536);
    const float2* xy = (const float2*)splats->xy;
    const float4* co = (const float4*)splats->conic_o;
    fgr::RenderWsView rv;
    if (render_ws || n_contrib) {
        // from the blend's saved state: chunk items in parallel, then the tiles
        if (!render_ws || !n_contrib || !fgr::render_ws_view(render_ws, render_ws_bytes, cam, cap_pairs, tune, &rv))
            return FG_ERR_INVALID_ARG;
        const int64_t items = rv.max_items + n_tiles;
        const unsigned gi = (unsigned)(items < 8192 ? items : 8192);
        const unsigned gt = grid < kTileBlocks ? grid : kTileBlocks;
        hipLaunchKernelGGL(k_kpc_items, dim3(gi), dim3(kThreads), 0, s, xy, co, vals, ranges, n_pairs, n_tiles,
                           cap_pairs, cam->width, cam->height, Wt, n_contrib, rv, kpc);
        if (kpc_hist)
            hipLaunchKernelGGL(k_tile_gtc<true>, dim3(gt), dim3(kThreads), 0, s, ranges, n_pairs, n_tiles,
                               cap_pairs, (const float*)kpc, tile_gtc, view_gtc, e, kpc_hist);
        else
            hipLaunchKernelGGL(k_tile_gtc<false>, dim3(gt), dim3(kThreads), 0, s, ranges, n_pairs, n_tiles,
                               cap_pairs, (const float*)kpc, tile_gtc, view_gtc, e, kpc_hist);
    } else if (kpc_hist) {
        hipLaunchKernelGGL(k_kpc<true>, dim3(grid), dim3(kThreads), 0, s, xy, co, vals, ranges, n_pairs, n_tiles,
                           cap_pairs, cam->width, cam->height, Wt, kpc, tile_gtc, view_gtc, e, kpc_hist);
    } else {
        hipLaunchKernelGGL(k_kpc<false>, dim3(grid), dim3(kThreads), 0, s, xy, co, vals, ranges, n_pairs, n_tiles,
                           cap_pairs, cam->width, cam->height, Wt, kpc, tile_gtc, view_gtc, e, kpc_hist);
    }
    hipLaunchKernelGGL(k_gtc_view, dim3(1), dim3(64), 0, s, view_gtc, n_pairs, cap_pairs);
    return hipGetLastError() == hipSuccess ? FG_OK : FG_ERR_HIP;
}

extern "C" int fg_gtc_tau(const double* view_gtc, int32_t n_views, float lambda_G, double* g_bar, float* tau,
                          uint32_t* status, void* stream)
{
    if (!view_gtc || n_views < 1 || !g_bar || !tau) return FG_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_gtc_tau, dim3(1), dim3(64), 0, (hipStream_t)stream, view_gtc, n_views, lambda_G, g_bar, tau,
                       status);
    return hipGetLastError() == hipSuccess ? FG_OK : FG_ERR_HIP;
}
