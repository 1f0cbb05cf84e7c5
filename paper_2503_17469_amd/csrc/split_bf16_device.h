// fp32 products on the bf16 matrix instruction: every fp32 operand as the exact sum of three bf16 values.
#pragma once
#include <hip/hip_runtime.h>

#include "bf16.h"

namespace omni {

// x = p[0] + p[1] + p[2] (two values at a time, packed as the matrix instruction's operands hold them): 24 significant bits
// are three times 8, and rounding to nearest makes each remainder exact in fp32.  Not for infinities, NaN and values that
// round up to infinity: a product with one of those comes out as infinity or NaN, which the kernels look for.
__device__ __forceinline__ void split3(float a, float b, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  p0 = pack_bf16(a, b);
  const float ra = a - bf16_lo(p0), rb = b - bf16_hi(p0);
  p1 = pack_bf16(ra, rb);
  const float sa = ra - bf16_lo(p1), sb = rb - bf16_hi(p1);
  p2 = pack_bf16(sa, sb);
}

}  // namespace omni
