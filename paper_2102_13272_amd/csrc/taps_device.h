// Device helpers of the transforms that write the tap and point planes of
// taps.hip's contraction.
#pragma once

#include "nwg_internal.h"

namespace nwg {

// Rank of axis prefix i among the live prefixes (the live ones below it),
// branch-free over the four 32-bit words (a 64-bit shift by a lane-varying
// amount became control flow that stopped the transforms' unrolling).
__device__ __forceinline__ int prefix_rank(unsigned long long m0, unsigned long long m1, int i) {
  const unsigned wd[4] = {(unsigned)m0, (unsigned)(m0 >> 32), (unsigned)m1, (unsigned)(m1 >> 32)};
  int r = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = i - 32 * q;
    const unsigned below = k <= 0 ? 0u : (k >= 32 ? 0xffffffffu : (1u << k) - 1u);
    r += __popc(wd[q] & below);
  }
  return r;
}

// The level-1 taps of a branch from its 9 x 9 sub-kernel S (level-1 digit 3
// dead: no tap has level-1 digit 2): G of level 2 along both axes.  put(q2r,
// q2c, 2 k1r + k1c, value).
template <class Put>
__device__ __forceinline__ void taps_xform(const float (&S)[9][9], Put&& put) {
#pragma unroll
  for (int q2r = 0; q2r < 4; ++q2r)
#pragma unroll
    for (int k1r = 0; k1r < 2; ++k1r) {
      float rowv[9];
#pragma unroll
      for (int ic = 0; ic < 9; ++ic) {
        float sacc = 0.0f;
#pragma unroll
        for (int k2 = 0; k2 < 3; ++k2)
          if (g_coef(q2r, k2) != 0.0f) sacc += g_coef(q2r, k2) * S[3 * k2 + k1r][ic];
        rowv[ic] = sacc;
      }
#pragma unroll
      for (int k1c = 0; k1c < 2; ++k1c) {
        float o[4];
        g_one(rowv[k1c], rowv[3 + k1c], rowv[6 + k1c], o);
#pragma unroll
        for (int q2c = 0; q2c < 4; ++q2c) put(q2r, q2c, 2 * k1r + k1c, o[q2c]);
      }
    }
}

// Where a branch's groups (q2r, q2c) lie in the live list (row-prefix rank x np
// + column-prefix rank): br, bc are the digits above level 2 of each axis, and
// group (q2r, q2c) is at base + rows * np + columns with the live nibbles' counts.
struct BranchPlace {
  unsigned nr, nc, live;
  int base, np;
  __device__ __forceinline__ BranchPlace(unsigned long long m0, unsigned long long m1, int np_,
                                         int br, int bc) {
    nr = prefix_nibble(m0, m1, br);
    nc = prefix_nibble(m0, m1, bc);
    live = nibble_live(nr, nc);
    np = np_;
    base = prefix_rank(m0, m1, 4 * br) * np + prefix_rank(m0, m1, 4 * bc);
  }
  __device__ __forceinline__ bool on(int q2r, int q2c) const { return (live >> (4 * q2r + q2c)) & 1u; }
  __device__ __forceinline__ int at(int q2r, int q2c) const {
    return base + __popc(nr & ((1u << q2r) - 1u)) * np + __popc(nc & ((1u << q2c) - 1u));
  }
};

}  // namespace nwg
