// lbm_march.hip -- several D2V9 time steps per launch (lbm_march_kernels.h): FP32 instances
// and the dispatch over storage formats.
#include "lbm_march_kernels.h"

namespace lbm {

hipError_t launch_march(int storage, int force, const StepArgs &a, int cus, int steps, const uint32_t *keys,
                        hipStream_t st)
{
    if (steps != 3 && steps != kMarchSteps) return hipErrorInvalidValue;
    if (storage == LBM_F32) return march_st<LBM_F32, false>(force, a, cus, steps, keys, st);
    return launch_march_16(storage, force, a, cus, steps, keys, st);
}

}  // namespace lbm
