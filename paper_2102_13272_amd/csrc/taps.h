// The contraction from level-1 taps (taps.hip) and the transforms it reads.
#pragma once

#include <hip/hip_runtime.h>

#include "plan.h"

namespace nwg {

// U [live group][2 k1r + k1c][M][np4(N)] -> Z; V [live group][3 q1r + q1c][M][np4(T)]
// (taps_applies plans)
hipError_t launch_contract_taps(const nwg_plan_info& g, const float* U, const float* V, float* Z,
                                hipStream_t s);
// Work-groups of a kernel that fit on one CU of device dev, asked once per
// (device, kernel); 0 if the query fails.
int taps_occupancy(int dev, const void* kernel, int threads);

// F(3,3) chains at depth 2 (taps5.hip): U 9 taps a group, V with rows of Tp; Z, 9
// values a group, lies behind V (taps5_z), in the memory of V and Z.
hipError_t launch_kernel_xform_taps5(const nwg_plan_info& g, const float* w, float* U,
                                     hipStream_t s);
hipError_t launch_contract_taps5(const nwg_plan_info& g, const float* U, const float* V, float* Z,
                                 hipStream_t s);
float* taps5_z(const nwg_plan_info& g, float* V);

// w -> U and x -> V in those layouts, on the mixed nest (mixed.hip) and on F(2,3)
// chains (kernel_xform.hip, taps_input.hip); X4: the mixed nest's scratch
hipError_t launch_kernel_xform_taps_mix(const nwg_plan_info& g, const float* w, float* U,
                                        hipStream_t s);
hipError_t launch_input_xform_taps_mix(const nwg_plan_info& g, const float* x, float* V, float* X4,
                                       hipStream_t s);
hipError_t launch_kernel_xform_taps_f23(const nwg_plan_info& g, const float* w, float* U,
                                        hipStream_t s);
hipError_t launch_input_xform_taps_f23(const nwg_plan_info& g, const float* x, float* V,
                                       hipStream_t s);
inline hipError_t launch_kernel_xform_taps(const nwg_plan_info& g, const float* w, float* U,
                                           hipStream_t s) {
  return g.tile == NWG_TILE_MIX_F23_F33 ? launch_kernel_xform_taps_mix(g, w, U, s)
                                        : launch_kernel_xform_taps_f23(g, w, U, s);
}
inline hipError_t launch_input_xform_taps(const nwg_plan_info& g, const float* x, float* V,
                                          float* X4, hipStream_t s) {
  return g.tile == NWG_TILE_MIX_F23_F33 ? launch_input_xform_taps_mix(g, x, V, X4, s)
                                        : launch_input_xform_taps_f23(g, x, V, s);
}

}  // namespace nwg
