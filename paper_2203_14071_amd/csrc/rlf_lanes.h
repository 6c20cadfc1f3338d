// Cross-lane sums by VALU lane swaps.
#pragma once

#include <hip/hip_runtime.h>

namespace rlf {

// Sum the values the wave's two halves (kHalf) or the rows of 16 lanes in
// each half hold, for two quantities at once: the lower half (even rows) of
// the result sums a, the upper half (odd rows) b.
template <bool kHalf>
__device__ __forceinline__ double fold_lanes(double a, double b) {
  const auto lo = kHalf ? __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false)
                        : __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = kHalf ? __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false)
                        : __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

}  // namespace rlf
