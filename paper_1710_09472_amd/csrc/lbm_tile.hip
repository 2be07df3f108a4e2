// lbm_tile.hip -- several steps per launch on tiles of D2V9 grids (lbm_tile_kernels.h): FP32 instances, the
// choice of tiles and the dispatch over storage formats.
#include "lbm_tile_kernels.h"

#include <algorithm>

namespace lbm {

// Tiles by measurement: the most steps whose tiles fit the CUs (256) once (a second block per CU
// takes turns with the first), on the smallest tiles that do (fewer wavefronts per SIMD). us per
// step, FP32 with solids:
//   64 x 32    4 x 4, 9 steps 0.76    8 x 8, 9 steps 0.86    16 x 16, 9 steps 1.04
//   128 x 128  8 x 8, 9 steps 0.92    16 x 16, 9 steps 1.07  8 x 8, 11 steps 0.94
//   256 x 256  16 x 16, 9 steps 1.18  16 x 16, 7 steps 1.25  32 x 16, 5 steps 1.44
//   300 x 290  20 x 18, 7 steps 1.46  16 x 16, 9 steps 1.69  24 x 24, 5 steps 1.58
// and 24 x 24 with 5 steps on every larger grid:
//   512 x 256  24 x 24, 5 steps 1.59  32 x 16, 5 steps 1.63  20 x 18, 7 steps 1.83
//   512 x 512  24 x 24, 5 steps 2.21  32 x 16, 5 steps 2.38  28 x 28, 3 steps 2.91
//   2048^2     24 x 24, 5 steps 23.2  32 x 16, 5 steps 29.3  56 x 8, 5 steps 25.4
// Grids of few rows (columns): the tile spans them, so that only the long axis has a halo and
// more steps fit (4096 x 4: 32 columns, 17 steps 0.54; 9 steps 0.68). Along that axis it is as
// long as one tile per CU makes it, between 32 nodes and a block of 1024 threads: a block holds
// 64 KB of LDS whatever its threads, so many short tiles leave the CUs with a wave or two each.
// us per step, FP32 without solids, tiles of 32 / as planned / single steps: 40000 x 1
// 1.06 / 0.52 / 3.4, 400000 x 2 8.5 / 2.7 / 12.4, 400000 x 8 14.6 / 9.6 / 40, 4 10^6 x 1
// 75 / 9.9 / 50; BF16 with solids, stochastic: 500000 x 2 19.3 / 5.1 / 14.0, 4 10^6 x 1
// 121 / 16.2 / 34.
TilePlan tile_plan(int nx, int ny, int cus)
{
    TilePlan p{};
    auto fits = [&](int steps, int tx, int ty) {
        p.steps = steps;
        p.tx = tx;
        p.ty = ty;
        return (long long)((nx + tx - 1) / tx) * ((ny + ty - 1) / ty) <= cus;
    };
    const int narrow = std::min(nx, ny), wide = std::max(nx, ny);
    if (narrow <= 8 && wide > 64) {
        const int len = std::min(std::max(((wide + cus - 1) / cus + 31) / 32 * 32, 32), kTileThreads / narrow - 32);
        if (nx <= ny)
            fits(17, nx, len);
        else
            fits(17, len, ny);
    } else if (!fits(9, 4, 4) && !fits(9, 8, 8) && !fits(9, 16, 16) && !fits(7, 20, 18)) {
        fits(5, 24, 24);
    }
    p.tx = std::min(p.tx, nx);
    p.ty = std::min(p.ty, ny);
    p.ntx = (nx + p.tx - 1) / p.tx;
    p.nty = (ny + p.ty - 1) / p.ty;
    p.ragged = (float)((double)p.ntx * p.tx * p.nty * p.ty / ((double)nx * ny));
    return p;
}

hipError_t launch_tile(int storage, int force, const StepArgs &a, const TilePlan &p, int steps, const uint32_t *keys,
                       hipStream_t st)
{
    if (storage == LBM_F32) return tile_st<LBM_F32, false>(force, a, p, steps, keys, st);
    return a.sr ? launch_tile_sr(storage, force, a, p, steps, keys, st)
                : launch_tile_16(storage, force, a, p, steps, keys, st);
}

}  // namespace lbm
