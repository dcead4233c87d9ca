// fdm_fused_f64.hip -- FP64-arithmetic instances of the fused two-stage
// kernel (float32 or float64 state), apart from the stage kernels' instances
// so that the two compile side by side.  No multiply-add contraction, as in
// fdm_stage_f64.hip.
#pragma clang fp contract(off)
#include "fdm_stage.h"

namespace fdm {

hipError_t launch_fused_f64(const InstDev &I, int dir, int integ, bool f64_state, hipStream_t s)
{
    if (integ == FUSED_TWO_STEPS) return hipErrorInvalidValue;   // float only
    const bool mid = integ == FUSED_MIDPOINT;
    if (f64_state)
        return mid ? launch_fused_r<double, double, FUSED_MIDPOINT>(I, dir, s)
                   : launch_fused_r<double, double, FUSED_HEUN>(I, dir, s);
    return mid ? launch_fused_r<double, float, FUSED_MIDPOINT>(I, dir, s)
               : launch_fused_r<double, float, FUSED_HEUN>(I, dir, s);
}

}  // namespace fdm
