// fdm_stage_f32.hip -- FP32-arithmetic instances of the stage kernels
// (float32 state).
//
// Implicit multiply-add contraction is off: the fused operations are the
// explicit madd() calls of the stage code, the same in every unrolled copy of
// the row loop and in every kernel instance, so results do not depend on the
// tile height or on the batched / plain schedule.
#pragma clang fp contract(off)
#include "fdm_stage.h"

namespace fdm {

hipError_t launch_stage_f32(const InstDev &I, int mode, hipStream_t s)
{
    return launch_stage_r<float, float>(I, mode, s);
}

hipError_t launch_fused_f32(const InstDev &I, int dir, int integ, hipStream_t s)
{
    switch (integ) {
    case FUSED_HEUN: return launch_fused_r<float, float, FUSED_HEUN>(I, dir, s);
    case FUSED_MIDPOINT: return launch_fused_r<float, float, FUSED_MIDPOINT>(I, dir, s);
    default: return launch_fused_r<float, float, FUSED_TWO_STEPS>(I, dir, s);
    }
}

hipError_t launch_fused_batched(const InstDev *d_inst, const int32_t *d_tile_inst, int64_t total_tiles, int dir,
                                bool mid, hipStream_t s)
{
    const int64_t blocks = (total_tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    const int per_xcd = (int)((blocks + 7) / 8);
    const dim3 grid(8 * per_xcd), block(kBlock);
    if (mid) {
        if (dir)
            hipLaunchKernelGGL((fused_kernel_batched<1, FUSED_MIDPOINT>), grid, block, 0, s, d_inst, d_tile_inst, total_tiles,
                               per_xcd);
        else
            hipLaunchKernelGGL((fused_kernel_batched<0, FUSED_MIDPOINT>), grid, block, 0, s, d_inst, d_tile_inst, total_tiles,
                               per_xcd);
    } else {
        if (dir)
            hipLaunchKernelGGL((fused_kernel_batched<1, FUSED_HEUN>), grid, block, 0, s, d_inst, d_tile_inst, total_tiles,
                               per_xcd);
        else
            hipLaunchKernelGGL((fused_kernel_batched<0, FUSED_HEUN>), grid, block, 0, s, d_inst, d_tile_inst, total_tiles,
                               per_xcd);
    }
    return hipGetLastError();
}

hipError_t launch_stage_batched_f32(const InstDev *d_inst, const int32_t *d_tile_inst, int64_t total_tiles,
                                    int mode, bool fd, hipStream_t s)
{
    return launch_batched_r<float, float>(d_inst, d_tile_inst, total_tiles, mode, fd, s);
}

}  // namespace fdm
