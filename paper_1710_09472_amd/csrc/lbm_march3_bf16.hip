// lbm_march3_bf16.hip -- two D3V19 time steps per launch (lbm_march3_kernels.h), BF16 storage
// rounded to nearest.
#include "lbm_march3_kernels.h"

namespace lbm {

hipError_t launch_march3_bf16(int force, const StepArgs &a, const March3Plan &p, const uint32_t *keys, hipStream_t st)
{
    if (a.sr) return launch_march3_bf16_sr(force, a, p, keys, st);
    return march3_st<LBM_BF16, false>(force, a, p, keys, st);
}

}  // namespace lbm
