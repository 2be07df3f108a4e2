// lbm_march3_f16_sr.hip -- two D3V19 time steps per launch (lbm_march3_kernels.h), F16 storage
// with stochastic rounding.
#include "lbm_march3_kernels.h"

namespace lbm {

hipError_t launch_march3_f16_sr(int force, const StepArgs &a, const March3Plan &p, const uint32_t *keys, hipStream_t st)
{
    return march3_st<LBM_F16, true>(force, a, p, keys, st);
}

}  // namespace lbm
