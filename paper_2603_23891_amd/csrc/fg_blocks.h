// Device-side core of the kernels that visit a tile's fragments (blend, its
// backward, KPC): a tile's 16 x 16 pixels are 32 blocks of 4 x 2, eight per
// wave (wave w: pixel rows 4w .. 4w+3), and every group of 8 lanes visits its
// own block's list of splats.
//
// A splat's skip test passes on few pixels (about 9 to 20 per splat and tile
// on the city and training scenes), so 64 pixels walking one splat together
// would leave most lanes idle, and per-pixel lists need an ordered append per
// fragment. Eight lanes per splat keep about a third to a half of the lanes
// on passing pixels, need no atomics, and evaluate each alpha once, where
// the value is used.
#pragma once

#include "fg_device.h"

namespace fgb {

constexpr int kThreads = 256;
constexpr int kBatch = 256;   // splats staged at a time, one per thread
constexpr int kBlocks = 32;   // 4 x 2 pixel blocks per tile, b = (ly / 2) * 4 + lx / 4

// exp(power) <= exp(-5.6) < 1/255 for power < -5.6, so with opacity <= 1 the
// splat is skipped either way: testing this first avoids evaluating the
// exponential without changing any result.
constexpr float kSkipPower = -5.6f;

// Tile-relative pixel of a thread: lane l of wave w is pixel (l & 3, (l >> 2) & 1)
// of block 8 w + l / 8.
__device__ __forceinline__ int pixel_x(int tid) { return ((tid >> 1) & 12) | (tid & 3); }
__device__ __forceinline__ int pixel_y(int tid) { return ((tid >> 6) << 2) | ((tid >> 4) & 2) | ((tid >> 2) & 1); }

// The power form A dx^2 + 2 B dx dy + C dy^2 reaches 11.2 where power = -5.6;
// the tests for skipping whole pixels use a bound 1% above it.
constexpr float kBound = 11.2f * 1.01f;

// Blocks of the tile that can hold a pixel passing the skip tests, as bits.
// power >= -5.6 is the ellipse A dx^2 + 2 B dx dy + C dy^2 <= 11.2 (dx, dy:
// splat centre minus pixel centre), so on a row at offset dy the passing
// pixel centres lie within u + (B dy -+ sqrt(11.2 A - det dy^2)) / A, det =
// AC - B^2, and the rows within v -+ sqrt(11.2 A / det). Both are taken for the
// bound 11.2 * 1.01 and widened by a slack: for a conic with B^2 <= 0.98 AC
// the float test's rounding moves the form by less than 1e-3, far below the
// 0.11 added, which also covers the rounding of det, the discriminant and
// the approximate reciprocals and square roots here. Nearly degenerate or
// non-finite conics take the blocks of the conservative box. The bits only
// choose what is tested: every pixel of a block is still tested exactly.
__device__ __forceinline__ uint32_t block_mask(float2 mm, float4 co, int tx, int ty, int W, int H)
{
    const float A = co.x, B = co.y, C = co.z;
    if (A > 0.0f && B * B <= 0.98f * (A * C)) {
        const float ox = (mm.x - (float)(tx * fgd::kTile)) - 0.5f;
        const float oy = (mm.y - (float)(ty * fgd::kTile)) - 0.5f;
        const float x1 = fminf(15.0f, (float)(W - 1 - tx * fgd::kTile));
        const float y1 = fminf(15.0f, (float)(H - 1 - ty * fgd::kTile));
        const float det = A * C - B * B;
        const float ey = __builtin_amdgcn_sqrtf((kBound * A) * __builtin_amdgcn_rcpf(det));
        const float ys = 0.05f + 1e-4f * (fabsf(oy) + ey);
        // clipped in float (a NaN bound keeps the tile's rows) before converting
        const float fa = fmaxf(ceilf(oy - ey - ys), 0.0f), fb = fminf(floorf(oy + ey + ys), y1);
        if (!(fa <= fb)) return 0u;
        const float inv = __builtin_amdgcn_rcpf(A);
        uint32_t m = 0u;
        for (int ly = (int)fa; ly <= (int)fb; ly++) {
            const float dy = oy - (float)ly;
            const float disc = kBound * A - det * (dy * dy);
            if (disc < 0.0f) continue;
            const float half = __builtin_amdgcn_sqrtf(disc) * inv;
            const float cen = ox + (B * dy) * inv;
            const float slack = 0.05f + 1e-4f * (fabsf(cen) + half);
            const float a = fmaxf(ceilf(cen - half - slack), 0.0f), e = fminf(floorf(cen + half + slack), x1);
            if (a <= e) m |= ((2u << ((int)e >> 2)) - (1u << ((int)a >> 2))) << (4 * (ly >> 1));
        }
        return m;
    }
    const uint32_t b = fgd::splat_box(mm, co, tx, ty, W, H);
    const int x0 = (int)(b & 255u), x1 = (int)((b >> 8) & 255u);
    const int y0 = (int)((b >> 16) & 255u), y1 = (int)(b >> 24);
    if (x0 > x1) return 0u;
    uint32_t m = 0u;
    for (int r = y0 >> 1; r <= (y1 >> 1); r++) m |= ((2u << (x1 >> 2)) - (1u << (x0 >> 2))) << (4 * r);
    return m;
}

// Appends 64 splats (batch index j per lane, block bits bm of this wave's
// eight blocks) to the wave's block lists: list[b][k] is the k-th splat
// (ascending) whose bit b is set, n[b] the lengths.
template <int COLS>
__device__ __forceinline__ void append_lists(uint32_t bm, int j, uint8_t (*list)[COLS], int (&n)[8])
{
    if (__ballot(bm != 0u) == 0ull) return;
#pragma unroll
    for (int b = 0; b < 8; b++) {
        const bool in = (bm >> b) & 1u;
        const uint64_t m = __ballot(in);
        if (in)
            list[b][n[b] + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = (uint8_t)j;
        n[b] += (int)__popcll(m);
    }
}

// The length of this lane's list: lanes 8 b .. 8 b + 7 visit list b.
__device__ __forceinline__ int lane_list(const int (&n)[8])
{
    const int sub = fgd::lane_id() >> 3;
    int mine = n[0];
#pragma unroll
    for (int b = 1; b < 8; b++) mine = sub == b ? n[b] : mine;
    return mine;
}

// A wave's eight block lists from the staged splats' block bits (s_list: the
// wave's own eight rows). Every wave scans all splats for its own blocks, so
// no wave waits for another. Returns the length of this lane's list.
template <int COLS>
__device__ __forceinline__ int build_lists(const uint32_t* s_bm, int cnt, uint8_t (*list)[COLS])
{
    const int lane = fgd::lane_id(), wave = threadIdx.x / fgd::kWave;
    int n[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int j0 = 0; j0 < cnt; j0 += fgd::kWave) {
        const int j = j0 + lane;
        append_lists(j < cnt ? (s_bm[j] >> (8 * wave)) & 255u : 0u, j, list, n);
    }
    return lane_list(n);
}

// Orders this wave's LDS writes before its own later LDS reads (and reads
// before later writes); no other wave takes part.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A staged splat as the evaluation reads it: the conic's diagonal carries the
// factor -0.5 of the power (a power of two, so the power is the same value).
__device__ __forceinline__ float4 stage_a(float2 mm, float4 co) { return make_float4(mm.x, mm.y, -0.5f * co.x, co.y); }
__device__ __forceinline__ float4 stage_b(float4 co, float4 c) { return make_float4(-0.5f * co.z, co.w, c.x, c.y); }

// The skip tests of Eq. (2): false if power > 0 or power < -5.6 (then alpha <
// 1/255 since opacity <= 1) or alpha < 1/255; otherwise alpha = min(0.99,
// opacity exp(power)). power = -0.5 (A dx^2 + C dy^2) - B dx dy.
__device__ __forceinline__ bool eval_alpha(float4 a, float4 b, float fpx, float fpy, float& alpha, bool& in_range)
{
    const float dx = a.x - fpx;
    const float dy = a.y - fpy;
    const float power = ((a.z * dx) * dx + (b.x * dy) * dy) - (a.w * dx) * dy;
    in_range = !(power > 0.0f || power < kSkipPower);
    const float v = b.y * fgd::exp_neg_in_range(power);
    alpha = v < 0.99f ? v : 0.99f;
    return in_range && !(alpha < 1.0f / 255.0f);
}

}  // namespace fgb
