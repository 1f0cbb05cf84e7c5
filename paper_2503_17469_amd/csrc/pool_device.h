// Device code of the 2 x 2 max pooling that the convolution kernels write with their output.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace omni {

// Where the gradient of a 2 x 2 max pooling goes: the first of the four inputs (scan order (0,0),
// (0,1), (1,0), (1,1)) that holds the maximum, or nowhere (4) when a ReLU folded into the pooled
// tensor has zeroed the maximum.  The comparison is on the values as stored (bf16).
__device__ inline uint32_t pool_code_of(float a, float b, float c, float d, bool relu, float& m) {
  m = a;
  uint32_t k = 0;
  if (b > m) { m = b; k = 1; }
  if (c > m) { m = c; k = 2; }
  if (d > m) { m = d; k = 3; }
  return (relu && !(m > 0.f)) ? 4u : k;
}

}  // namespace omni
