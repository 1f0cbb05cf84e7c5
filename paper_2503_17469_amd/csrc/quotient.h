// Quotients by a divisor that stays the same for a whole launch: a run-time division takes 150 to 300 cycles, and one or two of
// them used to stand in front of a kernel's first load; a multiplication takes a few.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace omni {

// 2^32 / d rounded up where quotient() is then exact for all 0 <= n < below, otherwise (and for d = 1) 0.  With r the rounding up
// (below d), n (2^32 + r) / (d 2^32) exceeds n / d by n r / (d 2^32), which stays below 1 / d while n d is at most 2^32.
inline uint32_t reciprocal_below(uint64_t d, uint64_t below) {
  return d > 1 && d < 1ull << 32 && below <= (1ull << 32) / d ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u;
}

// By a divisor that is 1 or whose reciprocal is known not to be 0: no branch, so that loads are not held up at one.
__host__ __device__ inline int exact_quotient(int n, uint32_t by) { return by ? (int)(((uint64_t)(uint32_t)n * by) >> 32) : n; }

__host__ __device__ inline int quotient(int n, uint32_t by, int d) {
  return by ? (int)(((uint64_t)(uint32_t)n * by) >> 32) : d == 1 ? n : n / d;
}

}  // namespace omni
