// lbm_march3.hip -- two D3V19 time steps per launch (lbm_march3_kernels.h): FP32 instances and
// the dispatch over storage formats.
#include "lbm_march3_kernels.h"

namespace lbm {

hipError_t launch_march3(int storage, int force, const StepArgs &a, const uint32_t *keys, hipStream_t st)
{
    if (storage == LBM_F32) return march3_st<LBM_F32, false>(force, a, keys, st);
    if (storage == LBM_F16) return launch_march3_f16(force, a, keys, st);
    if (storage == LBM_BF16) return launch_march3_bf16(force, a, keys, st);
    return hipErrorInvalidValue;
}

}  // namespace lbm
