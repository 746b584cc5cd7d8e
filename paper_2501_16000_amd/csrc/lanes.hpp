// lanes.hpp -- one-lane shifts across a 64-wide wavefront, shared by the
// register-resident multi-step D2Q9 kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace oreg {
namespace detail {

// lane l <- lane l - 1 (wave_shr:1) and lane l <- lane l + 1 (wave_shl:1).
// Lanes without a source are outside the valid region of the next level: in
// FP32 they read zero (bound_ctrl), which lets the compiler fold the shift
// into the arithmetic instruction that consumes it; in FP64 (two 32-bit
// moves, no folding) they keep their own value.
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ double from_left(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ double from_right(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x130, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(lo, lo, 0x130, 0xF, 0xF, false));
}

}  // namespace detail
}  // namespace oreg
