// fp32 products on the bf16 matrix instruction: every fp32 operand as the exact sum of three bf16 values.
#pragma once
#include <hip/hip_runtime.h>

#include "bf16.h"

namespace omni {

// 2^24 x = p[0] + p[1] + p[2] (two values at a time, packed as the matrix instruction's operands hold them): 24 significant bits
// are three times 8, and rounding to nearest makes each remainder exact in fp32.  Scaled, because unscaled the third piece of
// what is smaller than 2^-110 would lie below bf16's smallest number (2^-133; of 2^-124 ten bits are left): 2^24 times the
// smallest fp32 number is 2^-125, so that no piece of any number is even subnormal.  A sum of products is to be multiplied by
// kSplitUnscale.  `scale`: plus or minus kSplitScale.  Not for infinities, NaN and what reaches 2^104: their pieces have a NaN among them, which the kernels look for.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;
__device__ __forceinline__ void split3(float a, float b, float scale, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  a *= scale;
  b *= scale;
  p0 = pack_bf16(a, b);
  const float ra = a - bf16_lo(p0), rb = b - bf16_hi(p0);
  p1 = pack_bf16(ra, rb);
  const float sa = ra - bf16_lo(p1), sb = rb - bf16_hi(p1);
  p2 = pack_bf16(sa, sb);
}

}  // namespace omni
