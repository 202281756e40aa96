// Inclusive sums over the lanes of a wavefront, restarted where a key changes.
#pragma once

#include "device_utils.h"

namespace gco {

// Cross-lane moves on the data-parallel-primitive path (no LDS): lane l receives the value
// of lane l - N of its 16-lane row (row_shr:N), or rows 1 and 3 receive lane 15 of the row
// before them (row_bcast:15), or rows 2 and 3 receive lane 31 (row_bcast:31); every lane
// without a source keeps `fill`.  The six moves N = 1, 2, 4, 8, bcast 15, bcast 31 make an
// inclusive scan over the 64 lanes.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_move(int fill, int v) {
  return __builtin_amdgcn_update_dpp(fill, v, kCtrl, kRowMask, 0xf, false);
}
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_move(float fill, float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(fill), __float_as_int(v), kCtrl, kRowMask, 0xf, false));
}
#define GCO_SCAN_STEPS(STEP) \
  STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)

// Inclusive sum over the lanes, restarted wherever key changes (equal keys are contiguous).
__device__ __forceinline__ float scan_sum_by_key(float v, int key) {
#define GCO_STEP(C, M)                            \
  {                                               \
    const float ov = dpp_move<C, M>(0.f, v);      \
    const int ok = dpp_move<C, M>(-2, key);       \
    if (ok == key) v += ov;                       \
  }
  GCO_SCAN_STEPS(GCO_STEP)
#undef GCO_STEP
  return v;
}

}  // namespace gco
