// lbm_tile_sr.hip -- several steps per launch on tiles of D2V9 grids (lbm_tile_kernels.h): 16-bit storage with
// stochastic rounding.
#include "lbm_tile_kernels.h"

namespace lbm {

hipError_t launch_tile_sr(int storage, int force, const StepArgs &a, const TilePlan &p, int steps,
                          const uint32_t *keys, hipStream_t st)
{
    if (storage == LBM_F16) return tile_st<LBM_F16, true>(force, a, p, steps, keys, st);
    if (storage == LBM_BF16) return tile_st<LBM_BF16, true>(force, a, p, steps, keys, st);
    return hipErrorInvalidValue;
}

}  // namespace lbm
