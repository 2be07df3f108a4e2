// lbm_tile_kernels.h -- several time steps of the two-buffer D2V9 scheme in one launch on tiles of
// the grid: grids below 8 M nodes, and beyond it those of few rows or columns.
//
// A step of a small grid takes 3 - 4 us whatever its size (a launch on an idle GPU, a round
// trip to memory and back); a step of a larger one is bound by its pass over memory. k_tile takes `steps` steps per launch on tiles of the grid: a
// block owns one node per thread of a tile and a halo of steps - 1 nodes around it (none
// along an axis that the tile spans as a whole: there it wraps inside the block). Step 1
// pulls from memory as the single step does; between the steps the post-collision
// populations go through LDS (two halves in turn, one barrier per step), with the region
// that is still exact shrinking by one node per step; the last step's tile is written.
//
// Node arithmetic, rounding of 16-bit storage between steps and bits are those of the single
// step. Between the steps bounced populations come from the node's own registers.
//
// What bounds it: a launch and the first reads (3 us), then the VALU and one barrier per step:
// 0.4 us per step with one wavefront per SIMD, 1 us with four; on grids of many tiles the VALU
// with its recomputed halo (a 24 x 24 tile with 5 steps: 1.55 times the nodes). So the first
// reads wait for nothing (both places a population may sit in are loaded beside the link
// mask), a thread's LDS places are laid out once and its last step is one compare, and the
// loop takes two steps, one per LDS half: 64 x 32 12.0 -> 9.4 us per launch of 9 steps, 4096 x 4
// 11.6 -> 9.2 (17 steps), 512 x 256 12.3 -> 11.0 (5 steps; 8.1 with slabs per XCD).
// Measured on MI355X, FP32 with solids, us per step against single steps: 64 x 32 0.76 (2.8),
// 4096 x 4 0.54 (3.1), 256 x 256 1.2 (3.8), 512 x 256 1.6 (4.0), 512 x 512 2.2 (6.0),
// 1024 x 512 3.8 (9.4), 2048^2 23.2.
#pragma once

#include "lbm_device.h"

namespace lbm {
namespace {

struct TileArgs {
    StepArgs a;
    TilePlan p;
    int steps;
    FastDiv div_rx, div_ntx, div_nx, div_ny;
    int xoff, yoff;  // first node of tile 0's region, plus multiples of nx, ny that make it >= 0
    uint32_t keys[kTileSteps];  // sr_key of the steps but the last
    uint32_t last_key;          // sr_key of the last step
};

template <int ST, bool MASK, bool SOFT, int FORCE, bool SLIP, bool SR>
__global__ __launch_bounds__(kTileThreads) void k_tile(TileArgs ta)
{
    constexpr int LAT = LBM_D2V9;
    using L = Lat<LAT>;
    using T = typename Codec<ST>::T;
    using LT = typename LinkMask<LAT>::T;
    __shared__ float sh[2][L::Q - 1][kTileThreads];  // q = 1..8
    const StepArgs &a = ta.a;
    Geometry g = a.g;
    if constexpr (!SLIP) g.slip = 0;
    const int nx = g.nx, ny = g.ny, steps = ta.steps;
    // halo along each axis (0 where the tile spans the axis) and the block's region rx x ry
    const int hx = ta.p.tx < nx ? 1 : 0, hy = ta.p.ty < ny ? 1 : 0;
    const int rx = ta.p.tx + 2 * hx * (steps - 1), ry = ta.p.ty + 2 * hy * (steps - 1);
    // blocks in contiguous slabs per XCD: what a tile reads beyond its edge, and the lines it
    // shares with its neighbours, are then in the L2 that wrote them (512 x 256 FP32 11.0 ->
    // 8.1 us per launch, 256 x 256 12.4 -> 10.6, 2048^2 130 -> 116; 64 x 32 6.8 -> 6.9)
    const int bid = xcd_remap((int)blockIdx.x, (int)gridDim.x), tyi = fast_div(bid, ta.div_ntx), txi = bid - tyi * ta.p.ntx;
    const int id = (int)threadIdx.x;
    const int j = fast_div(id, ta.div_rx), i = id - j * rx;
    const int xv = txi * ta.p.tx + ta.xoff + i, yv = tyi * ta.p.ty + ta.yoff + j;
    const int x = xv - nx * fast_div(xv, ta.div_nx), y = yv - ny * fast_div(yv, ta.div_ny);
    // steps after the first that the node takes: its inputs of step l + 1 are exact inside the
    // region shrunk by l
    const int more = j < ry ? min(hx ? min(i, rx - 1 - i) : steps, hy ? min(j, ry - 1 - j) : steps) : -1;
    Tile t{};
    t.x0 = x;
    t.y = y;
    t.own = x + nx * y;
    t.valid = true;
    // LDS index of the node each population comes from (clamped for threads that never use it)
    const int im = i > 0 ? i - 1 : (hx ? 0 : rx - 1), ip = i + 1 < rx ? i + 1 : (hx ? i : 0);
    const int jm = j > 0 ? j - 1 : (hy ? 0 : ry - 1), jp = j + 1 < ry ? j + 1 : (hy ? j : 0);
    int from[L::Q];
    for_q<L::Q>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        int jj = L::ey[q] > 0 ? jm : (L::ey[q] < 0 ? jp : j), p = q;
        if constexpr (SLIP && L::ey[q] != 0) {
            // beside a free-slip wall plane: the reflected population of the node's own row
            const int yw = L::ey[q] > 0 ? wrapm(y, ny) : wrapp(y, ny);
            if ((g.slip & LBM_SLIP_Y) && (yw == 0 || yw == ny - 1)) {
                jj = j;
                p = reflected<LAT>(q, true, false);
            }
        }
        from[q] = (p - 1) * kTileThreads + jj * rx + (L::ex[q] > 0 ? im : (L::ex[q] < 0 ? ip : i));
    });
    LT lk[1] = {0};
    float d[1][L::Q], o[1][L::Q], s = 0.f;
    if (more >= 0) {
        // Step 1. Own slot: the pulled value and the node's own slot qbar are both loaded, so
        // that neither waits for the link mask (the state is far below 4 GiB here)
        const PullRows r = pull_rows<1>(g, t);
        const T *src = static_cast<const T *>(a.src);
        constexpr bool kOwn = MASK && !kSolidSlotBB<ST>;
        T c[L::Q], own[L::Q];
        if (MASK) lk[0] = *at32(static_cast<const LT *>(a.links), (unsigned)t.own);
        for_q<L::Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            c[q] = *at32(src, (unsigned)pull_row<LAT, q>(g, t, r) + pull_x<LAT, q, 1>(r, 0));
            if constexpr (kOwn && q != 0)
                own[q] = *at32(src, (unsigned)L::opp[q] * (unsigned)g.stride + (unsigned)t.own);
        });
        if (SOFT) s = *at32(g.s, (unsigned)t.own);
        for_q<L::Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            d[0][q] = Codec<ST>::dec(c[q], 1.f);
            if constexpr (kOwn && q != 0) d[0][q] = link_select<q>(lk[0], Codec<ST>::dec(own[q], 1.f), d[0][q]);
        });
        collide<LAT, SOFT, FORCE>(a.ph, d[0], s, o[0]);
    }
    auto step = [&](int l, float(&buf)[L::Q - 1][kTileThreads]) {
        if (more >= l - 1) {
            if constexpr (ST != LBM_F32) {  // what step l stores
                const uint32_t h = SR ? sr_node((uint32_t)t.own, ta.keys[l - 1]) : 0u;
#pragma unroll
                for (int q = 0; q < L::Q; ++q) o[0][q] = Codec<ST>::dec(enc_store<ST, SR>(o[0][q], h, q), 1.f);
            }
#pragma unroll
            for (int q = 1; q < L::Q; ++q) buf[q - 1][id] = o[0][q];
        }
        __syncthreads();
        if (more >= l) {
            d[0][0] = o[0][0];
            const float *flat = &buf[0][0];
#pragma unroll
            for (int q = 1; q < L::Q; ++q) d[0][q] = flat[from[q]];
            if constexpr (MASK)
                for_q<L::Q>([&](auto qc) {
                    constexpr int q = decltype(qc)::value;
                    if constexpr (q != 0) d[0][q] = link_select<q>(lk[0], o[0][L::opp[q]], d[0][q]);
                });
            collide<LAT, SOFT, FORCE>(a.ph, d[0], s, o[0]);
        }
    };
    for (int l = 1; l < steps; l += 2) {  // (an even number of steps after the first)
        step(l, sh[1]);
        step(l + 1, sh[0]);
    }
    const int ox = i - hx * (steps - 1), oy = j - hy * (steps - 1);
    if (more >= 0 && ox >= 0 && ox < ta.p.tx && oy >= 0 && oy < ta.p.ty && txi * ta.p.tx + ox < nx && tyi * ta.p.ty + oy < ny) {
        const uint32_t h[1] = {SR ? sr_node((uint32_t)t.own, ta.last_key) : 0u};
        store_tile<LAT, ST, MASK, 1, SR, false, false>(g, static_cast<T *>(a.dst), t, lk, o, h);
    }
}

template <int ST, bool MASK, bool SOFT, int FORCE, bool SLIP, bool SR>
hipError_t tile_launch(const TileArgs &ta, int threads, hipStream_t st)
{
    hipLaunchKernelGGL((k_tile<ST, MASK, SOFT, FORCE, SLIP, SR>), dim3(ta.p.ntx * ta.p.nty), dim3(threads), 0, st, ta);
    return hipGetLastError();
}

// `steps` time steps (odd, 1 .. p.steps) from a.src into a.dst with the step keys `keys`.
template <int ST, bool SR>
hipError_t tile_st(int force, const StepArgs &a, const TilePlan &p, int steps, const uint32_t *keys, hipStream_t st)
{
    const bool mask = a.links != nullptr, soft = a.g.s != nullptr, slip = a.g.slip != 0;
    TileArgs ta{};
    ta.a = a;
    ta.p = p;
    ta.steps = steps;
    const int rx = p.tx + (p.tx < a.g.nx ? 2 * (steps - 1) : 0), ry = p.ty + (p.ty < a.g.ny ? 2 * (steps - 1) : 0);
    ta.div_rx = make_fastdiv(rx);
    ta.div_ntx = make_fastdiv(p.ntx);
    ta.div_nx = make_fastdiv(a.g.nx);
    ta.div_ny = make_fastdiv(a.g.ny);
    auto first = [&](int halo, int n) { return (halo + n - 1) / n * n - halo; };
    ta.xoff = first((rx - p.tx) / 2, a.g.nx);
    ta.yoff = first((ry - p.ty) / 2, a.g.ny);
    for (int k = 0; k < steps; ++k) ta.keys[k] = ta.last_key = keys[k];
    const int threads = (rx * ry + 63) / 64 * 64;
    if (steps % 2 == 0 || steps < 1 || steps > kTileSteps || threads > kTileThreads) return hipErrorInvalidValue;
#define LBM_TILE(M, S, F) \
    return M && slip ? tile_launch<ST, M, S, F, M, SR>(ta, threads, st) : tile_launch<ST, M, S, F, false, SR>(ta, threads, st)
#define LBM_TILE_F(M, S)                   \
    do {                                   \
        if (force == 0) LBM_TILE(M, S, 0); \
        if (force == 1) LBM_TILE(M, S, 1); \
        if (force == 2) LBM_TILE(M, S, 2); \
        LBM_TILE(M, S, 3);                 \
    } while (0)
    if (mask) {
        if (soft) LBM_TILE_F(true, true); else LBM_TILE_F(true, false);
    } else {
        if (soft) LBM_TILE_F(false, true); else LBM_TILE_F(false, false);
    }
#undef LBM_TILE_F
#undef LBM_TILE
}

}  // namespace
}  // namespace lbm
