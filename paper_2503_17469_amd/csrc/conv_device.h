// Device code that the general implicit-GEMM kernels of conv_bf16.hip and conv_wgrad_bf16.hip share: how a reduction piece
// and a GEMM row find their element of the gathered tensor.
#pragma once
#include <hip/hip_runtime.h>

#include "bf16.h"
#include "kernels.h"

namespace omni {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

constexpr int kThreads = 256;
constexpr int kMaxPieces = 1024;   // reduction pieces (8 channels of one tap) a kernel can index: K <= 8192

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// q-th 8-channel piece of the reduction -> (filter row u, filter column v, first channel)
__device__ inline void build_tap_table(int* tab, const ConvGeom& g, int tid) {
  for (int q = tid; q * 8 < g.K && q < kMaxPieces; q += kThreads) {
    const int k = q * 8;
    const int tap = k / g.Cs, ci = k - tap * g.Cs;
    const int u = tap / g.ks, v = tap - u * g.ks;
    tab[q] = u | (v << 4) | (ci << 8);
  }
}

// Source element offset of (sample n, position h,w, tap u,v, channel ci); -1 if it falls in the padding.
__device__ inline long gather_offset(const ConvGeom& g, int n, int h, int w, int u, int v, int ci) {
  // written without early exits: the callers' loads must not sit behind divergent branches
  const int th = g.transposed ? h + g.pad - u : h * g.stride + u - g.pad;
  const int tw = g.transposed ? w + g.pad - v : w * g.stride + v - g.pad;
  const bool strided = g.transposed && g.stride > 1;
  const int hs = strided ? th / g.stride : th, ws = strided ? tw / g.stride : tw;
  bool ok = th >= 0 && tw >= 0 && hs < g.Hs && ws < g.Ws;
  ok = ok && (!strided || (hs * g.stride == th && ws * g.stride == tw));
  const long o = (((long)n * g.Hs + hs) * g.Ws + ws) * g.Cs + ci;
  return ok ? o : -1;
}

// position index m -> (n, h, w); m < 2^24 so the float quotient is exact after one correction
__device__ inline void decode_pos(const ConvGeom& g, int m, int& n, int& h, int& w) {
  const int hw = g.Hp * g.Wp;
  n = (int)((float)m * (1.0f / (float)hw));
  if (n * hw > m) --n;
  if ((n + 1) * hw <= m) ++n;
  const int r = m - n * hw;
  h = (int)((float)r * (1.0f / (float)g.Wp));
  if (h * g.Wp > r) --h;
  if ((h + 1) * g.Wp <= r) ++h;
  w = r - h * g.Wp;
}

}  // namespace
}  // namespace omni
