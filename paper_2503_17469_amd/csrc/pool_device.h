// Device code of the 2 x 2 max pooling that the convolution kernels write with their output.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "bf16.h"

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

// The pooling's gradient from its output's, 2 D channels (eight or four) at output position m (column `col` of rows of W): the four
// inputs of the window, each the gradient where its code says so and zero elsewhere.  din: the pooled tensor's gradient, rows of 2 W;
// c: the first channel.
template <int D>
__device__ inline void unpool_store(bf16_t* __restrict__ din, size_t m, int col, int W, int N, int c,
                                    uint32_t __attribute__((ext_vector_type(D))) grad, uint32_t __attribute__((ext_vector_type(D / 2))) code) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t Out __attribute__((ext_vector_type(D)));
  const u16x2 one = {1, 1};
  u16x2 k[D];
#pragma unroll
  for (int d = 0; d < D; ++d)
    k[d] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(0u, code[d >> 1], d & 1 ? 0x0C030C02u : 0x0C010C00u));
  bf16_t* const to = din + (4 * m - 2 * (size_t)col) * N + c;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    Out t;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const u16x2 which = {(uint16_t)q, (uint16_t)q};
      t[d] = grad[d] & __builtin_bit_cast(uint32_t, (u16x2)(__builtin_elementwise_min((u16x2)(k[d] ^ which), one) - one));
    }
    *reinterpret_cast<Out*>(to + (size_t)(((q >> 1) * 2 * W + (q & 1)) * N)) = t;
  }
}

}  // namespace omni
