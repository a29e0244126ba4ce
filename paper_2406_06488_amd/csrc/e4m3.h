// Conversion of the BF16-refined form's low plane.
#pragma once
#include "common.h"

namespace et {

// Four values, at most 448 in size, to fp8 E4M3, the first in the lowest byte: the hardware's
// conversion, which gives f32_to_e4m3's codes but keeps the sign of a zero.
__device__ inline uint32_t pack_e4m3(const float* x) {
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(
      x[2], x[3], __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], 0, false), true);
}

}  // namespace et
