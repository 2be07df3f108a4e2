// lbm_tile.hip -- several steps per launch on small D2V9 grids (lbm_tile_kernels.h): FP32 instances, the
// choice of tiles and the dispatch over storage formats.
#include "lbm_tile_kernels.h"

#include <algorithm>

namespace lbm {

// Tiles by measurement (us per step, FP32 with solids): 16 x 16 with 9 steps where such tiles
// fit the 256 CUs once (64 x 32: 1.36, 256 x 256: 1.60; 32 x 16 with 5 steps: 1.7, 2.1),
// 32 x 16 with 5 steps where they do not (300 x 300: 2.4 against 2.9; 512 x 256: 2.5 against
// 2.8). Grids of few rows (columns): the tile spans them, so that only the long axis has a
// halo and more steps fit (4096 x 4, 17 steps on 32 columns: 0.7).
TilePlan tile_plan(int nx, int ny)
{
    TilePlan p{};
    const long long n16 = (long long)((nx + 15) / 16) * ((ny + 15) / 16);
    const int thin = std::min(nx, ny);
    if (thin <= 8 && std::max(nx, ny) > 64) {
        p.steps = 17;
        p.tx = nx <= ny ? nx : 32;
        p.ty = nx <= ny ? 32 : ny;
    } else if (n16 <= 256) {
        p.steps = 9;
        p.tx = p.ty = 16;
    } else {
        p.steps = 5;
        p.tx = 32;
        p.ty = 16;
    }
    p.tx = std::min(p.tx, nx);
    p.ty = std::min(p.ty, ny);
    p.ntx = (nx + p.tx - 1) / p.tx;
    p.nty = (ny + p.ty - 1) / p.ty;
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
