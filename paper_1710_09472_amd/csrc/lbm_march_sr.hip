// lbm_march_sr.hip -- several D2V9 time steps per launch (lbm_march_kernels.h), 16-bit
// storage with stochastic rounding.
#include "lbm_march_kernels.h"

namespace lbm {

hipError_t launch_march_sr(int storage, int force, const StepArgs &a, int cus, int steps, const uint32_t *keys,
                           hipStream_t st)
{
    if (storage == LBM_F16) return march_st<LBM_F16, true>(force, a, cus, steps, keys, st);
    if (storage == LBM_BF16) return march_st<LBM_BF16, true>(force, a, cus, steps, keys, st);
    return hipErrorInvalidValue;
}

}  // namespace lbm
