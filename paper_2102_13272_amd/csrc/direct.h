// Launches of the direct kernels (direct.hip): x and the plain weights w -> y.
#pragma once

#include <hip/hip_runtime.h>

#include "plan.h"

namespace nwg {

// d: direct_route or direct_shape of g, not kDirectNone
hipError_t launch_direct(const nwg_plan_info& g, const DirectShape& d, const float* x,
                         const float* w, float* y, hipStream_t s);
// w copied to U, where a plan keeps the weights its calls read
hipError_t launch_direct_weights(const nwg_plan_info& g, const float* w, float* U, hipStream_t s);
// launch_direct with a status and a message, for entry points that hold no plan
int direct_conv(const nwg_plan_info& g, const DirectShape& d, const float* x, const float* w,
                float* y, hipStream_t s);

}  // namespace nwg
