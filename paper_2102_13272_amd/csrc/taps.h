// The mixed nest's contraction from level-1 taps (taps.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "plan.h"

namespace nwg {

// U [live group][2 k1r + k1c][M][np4(N)] -> Z; V [live group][3 q1r + q1c][M][np4(T)]
// (taps_applies plans)
hipError_t launch_contract_taps(const nwg_plan_info& g, const float* U, const float* V, float* Z,
                                hipStream_t s);
// w -> U and x -> V in those layouts (mixed.hip)
hipError_t launch_kernel_xform_taps(const nwg_plan_info& g, const float* w, float* U,
                                    hipStream_t s);
hipError_t launch_input_xform_taps(const nwg_plan_info& g, const float* x, float* V, float* X4,
                                   hipStream_t s);

}  // namespace nwg
