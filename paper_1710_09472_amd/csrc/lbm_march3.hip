// lbm_march3.hip -- two D3V19 time steps per launch (lbm_march3_kernels.h): FP32 instances and
// the dispatch over storage formats.
#include "lbm_march3_kernels.h"

namespace lbm {

// Planes per segment: the grid's columns of blocks times the segments fill the CUs (one block
// each) in as few rounds of as few planes (two of them recomputed) as there are.
March3Plan march3_plan(int nx, int ny, int nz, int cus)
{
    March3Plan p{(nx + kM3Cols - 1) / kM3Cols, (ny + kM3Rows - 3) / (kM3Rows - 2), nz, 0.f, 0.f};
    const long long columns = (long long)p.ntx * p.nty;
    long long cost = 1ll << 60;
    for (int nseg = 1; nseg <= std::max(1, nz / 4); ++nseg) {
        const int planes = (nz + nseg - 1) / nseg, used = (nz + planes - 1) / planes;
        const long long c = (columns * used + cus - 1) / cus * (planes + 3);
        if (c < cost) {
            cost = c;
            p.planes = planes;
        }
    }
    // the waves of rows that a grid of few rows lacks only wait: about half a working wave's time
    // (FP32 512 x 4 x 256 2.2 us per plane, 256 x 256 x 8 4.2 us)
    const double working = 0.5 + 0.5 * (std::min(ny, kM3Rows - 2) + 3) / (kM3Rows + 1);
    p.slots = (float)(working * (double)cost * cus * kM3Threads / ((double)nx * ny * nz));
    const int threads = row_block_threads(nx, 1);
    p.lanes = (float)((nx + threads - 1) / threads * threads) / (float)nx;
    return p;
}

hipError_t launch_march3(int storage, int force, const StepArgs &a, const March3Plan &p, const uint32_t *keys, hipStream_t st)
{
    if (storage == LBM_F32) return march3_st<LBM_F32, false>(force, a, p, keys, st);
    if (storage == LBM_F16) return launch_march3_f16(force, a, p, keys, st);
    if (storage == LBM_BF16) return launch_march3_bf16(force, a, p, keys, st);
    return hipErrorInvalidValue;
}

}  // namespace lbm
