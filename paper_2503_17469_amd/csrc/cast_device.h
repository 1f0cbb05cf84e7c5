// bf16 copies of a network's weights: the work of one workgroup, for the launch of their own (pointwise_bf16.hip) and for the
// first layer's forward launch, which takes them along (conv_bf16.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "bf16.h"
#include "common.h"
#include "kernels.h"

namespace omni {

// All layers' weight copies in one launch: with a few thousand weights per layer a launch per layer is pure launch latency
// (4 x 4.6 us at the three-layer CNN).  The table travels in the kernel arguments.
// Bound by HBM (4 bytes read, 2 or 4 written per weight).  A workgroup takes 64 x 64 weights of one filter
// tap through LDS, so that the transposed copy leaves in 32-byte pieces of whole rows; one thread per weight
// scattered it as 2-byte stores a row apart: 87 us for the 11.2 M weights of the ResNet-18 shape, 17 us for
// the 4.2 M of the 3072-1024-1024 MLP.
constexpr int kCastTile = 64;
constexpr int kCastStride = kCastTile + 2;   // halfwords; odd in words, so a column of the tile spreads over the banks

// Offset of the piece of eight channels that starts at c of output n in a copy laid out as matrix operands
// (conv_frag_bf16): blocks [n/32][tap][c/16] of 64 lanes x 8 elements.
__device__ inline long frag_offset(int n, int tap, int c, int taps, int channels) {
  return (((long)(n >> 5) * taps + tap) * (channels >> 4) + (c >> 4)) * 512 + ((n & 31) + 32 * ((c >> 3) & 1)) * 8;
}

// (256 threads; `tile` is kCastTile * kCastStride halfwords of LDS; the lanes look through the table at once)
__device__ __forceinline__ void cast_weights_body(const CastTable& tab, const float* __restrict__ params,
                                                  bf16_t* __restrict__ shadow, uint32_t* __restrict__ zero_page, int block,
                                                  bf16_t* tile) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (zero_page && block == 0 && tid < kZeroPageWords) zero_page[tid] = 0u;
  const int first = lane < tab.n ? tab.e[lane].first_block : 0x7fffffff;
  const int e = (int)__popcll(__ballot(block >= first)) - 1;
  const CastEntry t = tab.e[e];
  const int ci_tiles = (t.cin_pad + kCastTile - 1) / kCastTile;
  int local = block - t.first_block;
  const int ci0 = local % ci_tiles * kCastTile;
  local /= ci_tiles;
  const int tap = local % t.taps, co0 = local / t.taps * kCastTile;

  const int cl = (tid & 15) * 4, ci = ci0 + cl, r = tid >> 4;
  v4f v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int co = co0 + r + 16 * i;
    v[i] = v4f{0.f, 0.f, 0.f, 0.f};
    if (co < t.cout) {
      const float* src = params + t.src + ((long)co * t.taps + tap) * t.cin_real + ci;
      if (ci + 3 < t.cin_real) {
        v[i] = *reinterpret_cast<const v4f_a4*>(src);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (ci + q < t.cin_real) v[i][q] = src[q];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int co = co0 + r + 16 * i;
    const u32x2 w = {pack_bf16(v[i][0], v[i][1]), pack_bf16(v[i][2], v[i][3])};
    if (co < t.cout && ci < t.cin_pad)
      *reinterpret_cast<u32x2*>(shadow + t.dst_fwd +
                                (t.frag_fwd ? frag_offset(co, tap, ci, t.taps, t.cin_pad) + (ci & 7)
                                            : ((long)co * t.taps + tap) * t.cin_pad + ci)) = w;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      tile[(cl + q) * kCastStride + r + 16 * i] = (bf16_t)(w[q >> 1] >> (16 * (q & 1)));
  }
  if (t.dst_t < 0) return;
  __syncthreads();
  // rows of the transposed copy: output channels are a multiple of 8 wherever there is one
  const int tr = tid >> 2, tc = (tid & 3) * 16;
  if (ci0 + tr >= t.cin_pad) return;
  const uint32_t* row = reinterpret_cast<const uint32_t*>(tile + tr * kCastStride + tc);
  bf16_t* dst = shadow + t.dst_t + (t.frag_t ? frag_offset(ci0 + tr, tap, co0 + tc, t.taps, t.cout)
                                             : ((long)(ci0 + tr) * t.taps + tap) * t.cout + co0 + tc);
  const int second = t.frag_t ? 32 * 8 : 8;   // from one piece of eight channels to the next
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (co0 + tc + 8 * h < t.cout)
      *reinterpret_cast<u32x4*>(dst + second * h) = u32x4{row[4 * h], row[4 * h + 1], row[4 * h + 2], row[4 * h + 3]};
}

}  // namespace omni
