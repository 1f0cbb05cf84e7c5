// Per-channel sums of a batch norm's first stage in the epilogues of the convolutions (conv3_wide_bf16.hip, conv_frag_bf16.hip),
// in double throughout as in bn_partial_kernel (bn.hip).  In fp32 over the 32 or 64 positions of a wavefront, dgamma (a sum of
// products of either sign) was off by more than its own rounding to fp32 in a third of the channels, by 900 times that where
// the terms nearly cancel.  (Against sums in fp32: 1.5 per cent of a step of the ResNet-18 shape, 2048 images.)
//
// A lane of a wavefront's half (32 lanes, a position each, lane j) adds its positions' terms for runs of eight channels; a fixed
// tree over the lanes follows in which a lane keeps half of its list and adds what its partner holds of the same half, so that the
// list halves while the positions covered double: 15 additions for 16 sums.  Everything stays in vector registers
// (permlane16_swap, DPP): the same tree through ds_swizzle needs two of them per double.
#pragma once
#include "bf16.h"
#include "common.h"

namespace omni {

// The value of the lane that a DPP control word names; all lanes must be active.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const u32x2 w = __builtin_bit_cast(u32x2, v);
  const u32x2 r = {(uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[0], CTRL, 0xF, 0xF, true),
                   (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[1], CTRL, 0xF, 0xF, true)};
  return __builtin_bit_cast(double, r);
}
constexpr int kDppRotate8 = 0x128, kDppHalfMirror = 0x141, kDppXor2 = 0x4E, kDppXor1 = 0xB1;   // lane ^ 8, ^ 7, ^ 2, ^ 1

// One step of the tree: of `lo` and `hi` the lane keeps `hi` if `upper`, and adds its partner's.
template <int CTRL>
__device__ __forceinline__ double bn_exchange(double lo, double hi, bool upper) {
  const double keep = upper ? hi : lo, send = upper ? lo : hi;
  return keep + dpp_f64<CTRL>(send);
}

// t[0][e], t[1][e]: this lane's sums of channel e's values and products.  Lanes j and j ^ 1 are left with half of the sum t[j >> 4][e]
// each, e's bits being those of j from 8 down to 2 (bn_sums_channel).
__device__ __forceinline__ double bn_sums_tree(const double (&t)[2][8], int j) {
  double s[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // lanes 0-15 of a half get t[0] of both rows, lanes 16-31 t[1]
    const u32x2 a = __builtin_bit_cast(u32x2, t[0][e]), b = __builtin_bit_cast(u32x2, t[1][e]);
    const u32x2 x = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const u32x2 y = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    s[e] = __builtin_bit_cast(double, u32x2{x[0], y[0]}) + __builtin_bit_cast(double, u32x2{x[1], y[1]});
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] = bn_exchange<kDppRotate8>(s[e], s[4 + e], (j & 8) != 0);
#pragma unroll
  for (int e = 0; e < 2; ++e) s[e] = bn_exchange<kDppHalfMirror>(s[e], s[2 + e], (j & 4) != 0);
  return bn_exchange<kDppXor2>(s[0], s[1], (j & 2) != 0);
}
// The last step, for two runs of channels: even lanes end with the sum of the first, odd ones of the second.
__device__ __forceinline__ double bn_sums_pair(double first, double second, int j) {
  return bn_exchange<kDppXor1>(first, second, (j & 1) != 0);
}
// Which of its sixteen channels (second run: 16 on) and which sum lane (j, h) holds after that; h: the wavefront's half, whose
// runs start at channel 8 h.
__device__ __forceinline__ int bn_sums_channel(int j, int h) {
  return (j & 1) * 16 + h * 8 + ((j >> 3) & 1) * 4 + ((j >> 2) & 1) * 2 + ((j >> 1) & 1);
}
__device__ __forceinline__ int bn_sums_which(int j) { return j >> 4; }

// Adds eight stored values (four words of two bf16) and their squares.
__device__ __forceinline__ void bn_sums_add(double (&t)[2][8], u32x4 stored) {
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double v = (double)(i ? bf16_hi(stored[d]) : bf16_lo(stored[d]));
      t[0][2 * d + i] += v;
      t[1][2 * d + i] = fma(v, v, t[1][2 * d + i]);
    }
}
// Adds eight stored values of an output gradient and their products with the batch norm's input less its mean (fp32, a rounding
// each); 1 / deviation, the same for the whole channel, multiplies the sum (one rounding less per term than with the normalised
// value, and one multiplication).
__device__ __forceinline__ void bn_sums_add(double (&t)[2][8], u32x4 stored, u32x4 x, const v4f (&mean)[2]) {
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float v = i ? bf16_hi(stored[d]) : bf16_lo(stored[d]);
      t[0][2 * d + i] += (double)v;
      t[1][2 * d + i] += (double)(v * ((i ? bf16_hi(x[d]) : bf16_lo(x[d])) - mean[d >> 1][2 * (d & 1) + i]));
    }
}

}  // namespace omni
