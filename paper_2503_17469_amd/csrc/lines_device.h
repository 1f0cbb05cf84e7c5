// From the accumulators of a transposed 32 x 32 matrix product (weights left: a lane has one position, and of the channels runs of four)
// to whole lines of memory: after three exchanges within the wavefront a lane has ONE run of eight channels at several positions, and
// the lanes of an instruction cover eight positions' 128 bytes (one block of 32 channels: sixteen positions' 64).
//
// A compute unit takes a load or store apart into the 128-byte lines that it touches, 2 cycles each from the L2 and 4.4 from beyond.
// A run of eight channels of 32 positions per instruction, which is what one exchange leaves, is 32 lines of which a quarter is used:
// 64 to 140 cycles an instruction and not 17 to 35.  The epilogues of the convolutions (outputs; in the input gradients also the share
// to add and the batch norm's input) were bound by that.  It also leaves a batch norm's sums with fewer lanes to meet over.
#pragma once
#include "bf16.h"
#include "bn_sums_device.h"
#include "common.h"

namespace omni {

typedef float lines_v16f __attribute__((ext_vector_type(16)));

// Where a lane's run of eight channels begins in its tile of 32 NB channels, and its positions: position base + lines_position(r) of the
// block of 32, counted as the lanes that held them, for r = 0 .. 2 NB - 1.
template <int NB>
__device__ __forceinline__ int lines_channel(int lane) {
  return (NB == 2 ? (lane >> 3 & 1) * 32 : 0) + (lane >> 4 & 1) * 16 + (lane >> 5) * 8;
}
template <int NB>
__device__ __forceinline__ int lines_base(int lane) { return lane & (NB == 2 ? 7 : 15); }
// r's bits: the upper one is bit 3 of the position (NB == 2), the lower one bit 4.
template <int NB>
constexpr int lines_position(int r) { return (NB == 2 ? (r >> 1) * 8 : 0) + (r & 1) * 16; }

// Of `low` and `high` (two blocks of channels at a lane's position) lanes whose bit 3 is 0 keep `low` and lanes whose bit 3 is 1 `high`:
// at the position with bit 3 = 0 in `low`, at the other in `high`.
__device__ __forceinline__ void lines_exchange8(uint32_t& low, uint32_t& high) {
  const uint32_t was = low;
  low = (uint32_t)__builtin_amdgcn_update_dpp((int)low, (int)high, kDppRotate8, 0xF, 0xC, false);
  high = (uint32_t)__builtin_amdgcn_update_dpp((int)high, (int)was, kDppRotate8, 0xF, 0x3, false);
}
__device__ __forceinline__ void lines_exchange16(uint32_t& low, uint32_t& high) {
  const u32x2 s = __builtin_amdgcn_permlane16_swap(low, high, false, false);
  low = s[0];
  high = s[1];
}
__device__ __forceinline__ void lines_exchange32(uint32_t& low, uint32_t& high) {
  const u32x2 s = __builtin_amdgcn_permlane32_swap(low, high, false, false);
  low = s[0];
  high = s[1];
}

// Of fp32 accumulators: val[r] = eight channels at position r.
template <int NB>
__device__ __forceinline__ void lines_of(const lines_v16f (&acc)[NB], float (&val)[2 * NB][8]) {
  uint32_t w[NB][2][8];   // [block][half][channel]
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        w[b][q][e] = __float_as_uint(acc[b][8 * q + e]);
        w[b][q][4 + e] = __float_as_uint(acc[b][8 * q + 4 + e]);
        lines_exchange32(w[b][q][e], w[b][q][4 + e]);
      }
      lines_exchange16(w[b][0][e], w[b][1][e]);
      lines_exchange16(w[b][0][4 + e], w[b][1][4 + e]);
    }
  if constexpr (NB == 2) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) lines_exchange8(w[0][q][e], w[NB - 1][q][e]);
  }
#pragma unroll
  for (int r = 0; r < 2 * NB; ++r)
#pragma unroll
    for (int e = 0; e < 8; ++e) val[r][e] = __uint_as_float(w[r >> 1][r & 1][e]);
}

// Of values already rounded to bf16, in the order of the accumulators: w[b][d] = registers 2 d and 2 d + 1 of block b.
template <int NB>
__device__ __forceinline__ void lines_of(uint32_t (&w)[NB][8], u32x4 (&out)[2 * NB]) {
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int d = 0; d < 2; ++d) lines_exchange32(w[b][4 * q + d], w[b][4 * q + 2 + d]);
#pragma unroll
    for (int d = 0; d < 4; ++d) lines_exchange16(w[b][d], w[b][4 + d]);
  }
  if constexpr (NB == 2) {
#pragma unroll
    for (int d = 0; d < 8; ++d) lines_exchange8(w[0][d], w[NB - 1][d]);
  }
#pragma unroll
  for (int r = 0; r < 2 * NB; ++r)
#pragma unroll
    for (int d = 0; d < 4; ++d) out[r][d] = w[r >> 1][(r & 1) * 4 + d];
}

// The sums of a batch norm over a wavefront's positions (bn_sums_device.h), from what lanes have added for their eight channels: over the
// eight lanes that share them, as the tree there.  A lane is left with sum lines_sum(lane) of channels lines_sum_channel(lane) and
// the next one of a tile of 64.
__device__ __forceinline__ void lines_sums(const double (&t)[2][8], int lane, double (&sum)[2]) {
  double s[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) s[e] = bn_exchange<kDppHalfMirror>(t[0][e], t[1][e], (lane & 4) != 0);
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] = bn_exchange<kDppXor2>(s[e], s[4 + e], (lane & 2) != 0);
#pragma unroll
  for (int e = 0; e < 2; ++e) sum[e] += bn_exchange<kDppXor1>(s[e], s[2 + e], (lane & 1) != 0);
}
__device__ __forceinline__ int lines_sum(int lane) { return lane >> 2 & 1; }
__device__ __forceinline__ int lines_sum_channel(int lane) { return lines_channel<2>(lane) + (lane >> 1 & 1) * 4 + (lane & 1) * 2; }

}  // namespace omni
