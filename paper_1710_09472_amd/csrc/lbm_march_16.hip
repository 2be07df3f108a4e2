// lbm_march_16.hip -- several D2V9 time steps per launch (lbm_march_kernels.h), 16-bit
// storage rounded to nearest.
#include "lbm_march_kernels.h"

namespace lbm {

hipError_t launch_march_16(int storage, int force, const StepArgs &a, int cus, int steps, const uint32_t *keys,
                           hipStream_t st)
{
    if (a.sr) return launch_march_sr(storage, force, a, cus, steps, keys, st);
    if (storage == LBM_F16) return march_st<LBM_F16, false>(force, a, cus, steps, keys, st);
    if (storage == LBM_BF16) return march_st<LBM_BF16, false>(force, a, cus, steps, keys, st);
    return hipErrorInvalidValue;
}

}  // namespace lbm
