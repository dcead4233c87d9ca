// fdm_fused_f64.hip -- FP64-arithmetic instances of the fused two-stage
// kernel (float32 or float64 state), apart from the stage kernels' instances
// so that the two compile side by side.  No multiply-add contraction, as in
// fdm_stage_f64.hip.
#pragma clang fp contract(off)
#include "fdm_stage.h"

namespace fdm {

hipError_t launch_fused_f64(const InstDev &I, int dir, bool mid, bool f64_state, hipStream_t s)
{
    if (f64_state)
        return mid ? launch_fused_r<double, double, true>(I, dir, s) : launch_fused_r<double, double, false>(I, dir, s);
    return mid ? launch_fused_r<double, float, true>(I, dir, s) : launch_fused_r<double, float, false>(I, dir, s);
}

}  // namespace fdm
