// A workgroup's barrier for data that goes through LDS only.
#pragma once
#include <hip/hip_runtime.h>

namespace omni {

// __syncthreads() also waits until every global store and load of the wavefront so far is complete, 1000 to 3000 cycles where
// results have just been stored or operands of a later step are on their way.  This one orders LDS accesses alone; global
// memory written before it must not be read by the workgroup's other wavefronts after it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace omni
