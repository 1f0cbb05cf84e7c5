// The transposing LDS read of gfx950 (ds_read_b64_tr_b16): sixteen lanes hand in four rows x sixteen columns of 16-bit values,
// 8 bytes each, and every lane receives one column at those four rows.
#pragma once
#include <hip/hip_runtime.h>

namespace omni {

// Eight rows of one column, from the addresses that this lane hands in for either four: an operand of the 16-bit matrix
// instructions whose reduction index is the slow one in LDS.
__device__ inline auto tr_pair(const unsigned char* a, const unsigned char* b) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) v4s lds_v4s;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)a);
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)b);
  return __builtin_bit_cast(v8bf, v8s{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
}

}  // namespace omni
