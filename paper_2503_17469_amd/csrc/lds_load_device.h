// Loads from memory that write LDS themselves (global_load_lds_dwordx4 of gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace omni {

// Sixteen bytes per lane from memory to LDS address `to` + 16 * lane (to: the same in the whole wavefront), from base + offset or
// from an address per lane.  Counted by vmcnt like any load; the compiler does not know of it, so whoever reads the data waits
// first.  (Through the builtin it waits for all loads under way before the next LDS read, whichever part of LDS that reads.)
//
// Vector memory must read a scalar register five wait states or more after a vector instruction has written it (v_readfirstlane of a
// base, v_readlane of a spilled one), which the hardware does not see to, and the compiler not in front of assembly: two moves and
// three states of s_nop.  M0 wants one of them in either form.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t offset, uint32_t to) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 2\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
               : "=&s"(m0) : "s"(to), "v"(offset), "s"(base) : "memory");
}
__device__ __forceinline__ void load_to_lds(const void* from, uint32_t to) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
               : "=&s"(m0) : "s"(to), "v"(from) : "memory");
}

// The LDS address of a pointer into shared memory.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p;
}

}  // namespace omni
