// Bandwidth-bound kernels of the step: softmax cross-entropy over the ragged
// batch, and the fused weighted gradient aggregation + SGD update.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "update_device.h"

namespace omni {

namespace {

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Worker that owns row s (segments are few; a linear scan over kernel arguments).
__device__ inline int owner(const Segments& seg, int s) {
  int k = 0;
  while (k + 1 < seg.K && s >= seg.off[k + 1]) ++k;
  return k;
}

// One wavefront per row.  loss_row = logsumexp(z) - z[y]; dz = (softmax - onehot) / b_k:
// the 1/|b_k| of equation bspweightedgrads, so that the backward pass yields
// each worker's MEAN gradient.
__global__ __launch_bounds__(256) void softmax_xent_kernel(const float* __restrict__ z,
                                                           const int32_t* __restrict__ labels, int C,
                                                           Segments seg, float* __restrict__ dz,
                                                           float* __restrict__ loss_rows,
                                                           uint32_t* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int rows = seg.off[seg.K];
  if (row >= rows) return;
  const int k = owner(seg, row);
  const float inv_b = 1.0f / (float)(seg.off[k + 1] - seg.off[k]);
  const float* zr = z + (size_t)row * C;
  float* dr = dz + (size_t)row * C;
  const int y = labels[row];
  if (y < 0 || y >= C) {
    if (lane == 0) {
      atomicOr(status, 1u);
      loss_rows[row] = 0.f;
    }
    for (int c = lane; c < C; c += 64) dr[c] = 0.f;
    return;
  }
  float m = -INFINITY;
  for (int c = lane; c < C; c += 64) m = fmaxf(m, zr[c]);
  m = wave_max(m);
  float s = 0.f;
  for (int c = lane; c < C; c += 64) s += expf(zr[c] - m);
  s = wave_sum(s);
  const float lse = logf(s);
  if (lane == 0) loss_rows[row] = lse - (zr[y] - m);
  for (int c = lane; c < C; c += 64) {
    float p = expf(zr[c] - m - lse);
    if (c == y) p -= 1.0f;
    dr[c] = p * inv_b;
  }
}

// One workgroup.  L_k = (1/b_k) sum of the worker's row losses (fixed-order tree,
// so results repeat bit for bit), loss = sum_k (b_k/B) L_k.
__global__ __launch_bounds__(256) void loss_reduce_kernel(const float* __restrict__ loss_rows, Segments seg,
                                                          float* __restrict__ loss_per_worker,
                                                          float* __restrict__ loss) {
  __shared__ float red[256];
  const int t = threadIdx.x;
  const float invB = 1.0f / (float)seg.off[seg.K];
  float total = 0.f;
  for (int k = 0; k < seg.K; ++k) {
    float a = 0.f;
    for (int s = seg.off[k] + t; s < seg.off[k + 1]; s += 256) a += loss_rows[s];
    red[t] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (t < w) red[t] += red[t + w];
      __syncthreads();
    }
    if (t == 0) {
      const float bk = (float)(seg.off[k + 1] - seg.off[k]);
      const float Lk = red[0] / bk;
      loss_per_worker[k] = Lk;
      total += bk * invB * Lk;
    }
    __syncthreads();
  }
  if (t == 0) loss[0] = total;
}

__device__ inline uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// The last P % 4 parameters of the update below.
template <bool SHADOW, bool MOM, bool KEEPG>
__device__ inline void weighted_sgd_tail(float* params, float* velocity, const float* grads, size_t stride, size_t P, int K,
                                         const Lambdas& lam, const Optim& opt, uint16_t* shadow, float* gout) {
  if (threadIdx.x < (P & 3)) {
    const size_t j = P / 4 * 4 + threadIdx.x;
    float g = 0.f;
    for (int k = 0; k < K; ++k) g += lam.v[k] * grads[(size_t)k * stride + j];
    if (KEEPG) gout[j] = g;
    float th = params[j], v = MOM ? velocity[j] : 0.f;
    apply_update<MOM>(th, v, g, opt);
    params[j] = th;
    if (MOM) velocity[j] = v;
    if (SHADOW) shadow[j] = bf16_rne(th);
  }
}

// theta[j] -= lr * sum_k lambda_k G[k][j]  (equations bspweightedgrads and
// bspvariableSGD fused: the K gradient rows and theta are each read once, theta
// written once).  Rows of G are 256-byte aligned, so 16-byte loads throughout.
// The gradient rows are read exactly once (streaming, non-temporal loads); two
// 16-byte columns per thread are in flight together so that 2*(K+1) loads cover
// the HBM latency.
// MOM: the momentum / weight-decay update of the paper's experiments (velocity is read and
// written beside the parameters: (K+4)*4 bytes per parameter instead of (K+2)*4):
//   d = g + wd*theta;  v = mu*v + d;  theta -= lr*v.
// KEEPG: the aggregated gradient g itself is also written to gout (4 more bytes per parameter; for
// callers that want to look at it: the update alone never stores it).
template <bool SHADOW, bool MOM, bool KEEPG>
__global__ __launch_bounds__(256) void weighted_sgd_kernel(float* __restrict__ params, float* __restrict__ velocity,
                                                           const float* __restrict__ grads, size_t stride,
                                                           size_t P, int K, Lambdas lam, Optim opt,
                                                           uint16_t* __restrict__ shadow, float* __restrict__ gout) {
  const size_t n4 = P / 4;
  const size_t nthreads = (size_t)gridDim.x * blockDim.x;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t i0 = t; i0 < n4; i0 += 2 * nthreads) {
    const size_t i1 = i0 + nthreads;
    const bool has1 = i1 < n4;
    const size_t j1 = has1 ? i1 : i0;          // the second column re-reads the first when past the end
    v4f g0 = {0.f, 0.f, 0.f, 0.f}, g1 = {0.f, 0.f, 0.f, 0.f};
    v4f th0 = *reinterpret_cast<const v4f*>(params + 4 * i0);
    v4f th1 = *reinterpret_cast<const v4f*>(params + 4 * j1);
    v4f v0 = {0.f, 0.f, 0.f, 0.f}, v1 = {0.f, 0.f, 0.f, 0.f};
    if (MOM) {
      v0 = *reinterpret_cast<const v4f*>(velocity + 4 * i0);
      v1 = *reinterpret_cast<const v4f*>(velocity + 4 * j1);
    }
    int k = 0;
    for (; k + 4 <= K; k += 4) {
      v4f a[4], c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(grads + (size_t)(k + u) * stride + 4 * i0));
        c[u] = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(grads + (size_t)(k + u) * stride + 4 * j1));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        g0 += lam.v[k + u] * a[u];
        g1 += lam.v[k + u] * c[u];
      }
    }
    for (; k < K; ++k) {
      g0 += lam.v[k] * __builtin_nontemporal_load(reinterpret_cast<const v4f*>(grads + (size_t)k * stride + 4 * i0));
      g1 += lam.v[k] * __builtin_nontemporal_load(reinterpret_cast<const v4f*>(grads + (size_t)k * stride + 4 * j1));
    }
    if (KEEPG) {
      *reinterpret_cast<v4f*>(gout + 4 * i0) = g0;
      if (has1) *reinterpret_cast<v4f*>(gout + 4 * i1) = g1;
    }
    apply_update<MOM>(th0, v0, g0, opt);
    apply_update<MOM>(th1, v1, g1, opt);
    *reinterpret_cast<v4f*>(params + 4 * i0) = th0;
    if (has1) *reinterpret_cast<v4f*>(params + 4 * i1) = th1;
    if (MOM) {
      *reinterpret_cast<v4f*>(velocity + 4 * i0) = v0;
      if (has1) *reinterpret_cast<v4f*>(velocity + 4 * i1) = v1;
    }
    if (SHADOW) {
      ushort4 s;
      s.x = bf16_rne(th0[0]); s.y = bf16_rne(th0[1]); s.z = bf16_rne(th0[2]); s.w = bf16_rne(th0[3]);
      *reinterpret_cast<ushort4*>(shadow + 4 * i0) = s;
      if (has1) {
        s.x = bf16_rne(th1[0]); s.y = bf16_rne(th1[1]); s.z = bf16_rne(th1[2]); s.w = bf16_rne(th1[3]);
        *reinterpret_cast<ushort4*>(shadow + 4 * i1) = s;
      }
    }
  }
  if (blockIdx.x == 0) weighted_sgd_tail<SHADOW, MOM, KEEPG>(params, velocity, grads, stride, P, K, lam, opt, shadow, gout);
}

// The same for few parameters, which are one round of workgroups that wait for memory: a column per thread, and the rows'
// loads of DEEP workers on their way together (four at a time are sixteen round trips one after the other for 64
// workers).  Same sums in the same order.  10,000 to 100,000 parameters: 64 workers 11.4 -> 6.7 us, 16 and fewer
// 4.3 -> 3.8 us (of which the launch itself is 3.5).
template <int DEEP, bool SHADOW, bool MOM, bool KEEPG>
__global__ __launch_bounds__(256) void weighted_sgd_few_kernel(float* __restrict__ params, float* __restrict__ velocity,
                                                               const float* __restrict__ grads, size_t stride,
                                                               size_t P, int K, Lambdas lam, Optim opt,
                                                               uint16_t* __restrict__ shadow, float* __restrict__ gout) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P / 4) {
    v4f th = *reinterpret_cast<const v4f*>(params + 4 * i);
    v4f g = {0.f, 0.f, 0.f, 0.f}, v = {0.f, 0.f, 0.f, 0.f};
    if (MOM) v = *reinterpret_cast<const v4f*>(velocity + 4 * i);
    const float* src = grads + 4 * i;
    for (int k0 = 0; k0 < K; k0 += DEEP) {
      v4f a[DEEP];
#pragma unroll
      for (int u = 0; u < DEEP; ++u)
        a[u] = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(src + (size_t)min(k0 + u, K - 1) * stride));
      __builtin_amdgcn_sched_barrier(0);   // all of them before the first is waited for
#pragma unroll
      for (int u = 0; u < DEEP; ++u)
        g += lam.v[min(k0 + u, K - 1)] * (k0 + u < K ? a[u] : v4f{0.f, 0.f, 0.f, 0.f});
    }
    if (KEEPG) *reinterpret_cast<v4f*>(gout + 4 * i) = g;
    apply_update<MOM>(th, v, g, opt);
    *reinterpret_cast<v4f*>(params + 4 * i) = th;
    if (MOM) *reinterpret_cast<v4f*>(velocity + 4 * i) = v;
    if (SHADOW) {
      ushort4 s;
      s.x = bf16_rne(th[0]); s.y = bf16_rne(th[1]); s.z = bf16_rne(th[2]); s.w = bf16_rne(th[3]);
      *reinterpret_cast<ushort4*>(shadow + 4 * i) = s;
    }
  }
  if (blockIdx.x == 0) weighted_sgd_tail<SHADOW, MOM, KEEPG>(params, velocity, grads, stride, P, K, lam, opt, shadow, gout);
}

// The same for ranges of the parameters, 1024 columns of one range at a time; four loads of each of four workers on their way.
constexpr int kRangesMax = 32;
struct RangeTable {
  int n, pieces;
  int32_t first[kRangesMax];   // range i has the pieces first[i] on, 1024 columns each
  uint32_t beg[kRangesMax], end[kRangesMax];
};
template <bool MOM>
__global__ __launch_bounds__(256) void weighted_sgd_ranges_kernel(float* __restrict__ params, float* __restrict__ velocity,
                                                                  const float* __restrict__ grads, size_t stride, RangeTable tab,
                                                                  int K, Lambdas lam, Optim opt) {
  const int lane = threadIdx.x & (kRangesMax - 1), mine = tab.first[lane];   // (all lanes at once)
  for (int piece = blockIdx.x; piece < tab.pieces; piece += gridDim.x) {
    const int at = __popcll(__ballot((int)(threadIdx.x & 63) < tab.n && mine <= piece)) - 1;
    const int part = piece - __builtin_amdgcn_readlane(mine, at);
    const size_t beg = tab.beg[at], n = tab.end[at] - beg, n4 = n / 4, c0 = (size_t)part * 1024 + threadIdx.x;
    float* const th_at = params + beg;
    float* const ve_at = MOM ? velocity + beg : nullptr;
    const float* const g_at = grads + beg;
    if (n4 > 0) {
      size_t j[4];
      v4f th[4], ve[4], g[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        j[u] = 4 * min(c0 + 256 * u, n4 - 1);
        th[u] = *reinterpret_cast<const v4f*>(th_at + j[u]);
        ve[u] = MOM ? *reinterpret_cast<const v4f*>(ve_at + j[u]) : v4f{0.f, 0.f, 0.f, 0.f};
        g[u] = v4f{0.f, 0.f, 0.f, 0.f};
      }
      int k = 0;
      for (; k + 4 <= K; k += 4) {
        v4f a[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            a[q][u] = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(g_at + (size_t)(k + q) * stride + j[u]));
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 4; ++u) g[u] += lam.v[k + q] * a[q][u];
      }
      for (; k < K; ++k)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          g[u] += lam.v[k] * __builtin_nontemporal_load(reinterpret_cast<const v4f*>(g_at + (size_t)k * stride + j[u]));
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (c0 + 256 * u >= n4) continue;
        apply_update<MOM>(th[u], ve[u], g[u], opt);
        *reinterpret_cast<v4f*>(th_at + j[u]) = th[u];
        if (MOM) *reinterpret_cast<v4f*>(ve_at + j[u]) = ve[u];
      }
    }
    if (part == 0) weighted_sgd_tail<false, MOM, false>(th_at, ve_at, g_at, stride, n, K, lam, opt, nullptr, nullptr);
  }
}

// g = sum_k lambda_k G[k] alone (equation bspweightedgrads without the update), same summation order.
__global__ __launch_bounds__(256) void weighted_reduce_kernel(const float* __restrict__ grads, size_t stride, size_t P,
                                                              int K, Lambdas lam, float* __restrict__ gout) {
  for (size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x; j < P; j += (size_t)gridDim.x * blockDim.x) {
    float g = 0.f;
    for (int k = 0; k < K; ++k) g += lam.v[k] * grads[(size_t)k * stride + j];
    gout[j] = g;
  }
}

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace

void softmax_xent_f32(hipStream_t st, const float* z, const int32_t* labels, int C, const Segments& seg,
                      float* dz, float* loss_rows, float* loss_per_worker, float* loss, uint32_t* status) {
  const int rows = seg.off[seg.K];
  hipLaunchKernelGGL(softmax_xent_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, z, labels, C, seg, dz,
                     loss_rows, status);
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(256), 0, st, loss_rows, seg, loss_per_worker, loss);
}

void weighted_sgd_f32(hipStream_t st, float* params, const float* grads, size_t stride, size_t P,
                      const Segments& seg, float lr, uint16_t* shadow_bf16, float* velocity, float momentum,
                      float weight_decay, const KernelTimer* timer, float* gout) {
  const Lambdas lam = lambdas_of(seg);
  const Optim opt{lr, momentum, weight_decay};
  const size_t n4 = P / 4;
  size_t blocks = (n4 + 511) / 512;          // two columns per thread per trip
  // Two workgroups per compute unit, each thread walking its columns: measured at P = 11.2 M, K = 8 (449 MB per
  // launch): 512 workgroups 71.8 us, 256: 73.8, 2048: 77.0, one trip per thread (5479): 74.7; counts that are no
  // multiple of the 256 compute units lose to the uneven last round (384: 78.5, 640: 80.6).
  if (blocks > 512) blocks = 512;
  if (blocks < 1) blocks = 1;
  const bool few = n4 <= 256 * 256;          // one workgroup per compute unit; beyond, 64 workers are 4 to 8 per cent slower with it
  if (few) blocks = std::max<size_t>((n4 + 255) / 256, 1);
  const dim3 grid((unsigned)blocks), block(256);
#define OMNI_UPD_(KERNEL)                                                                                      \
  if (timer)                                                                                                   \
    hipExtLaunchKernelGGL(KERNEL, grid, block, 0, st, timer->start, timer->stop, 0, params, velocity, grads,   \
                          stride, P, seg.K, lam, opt, shadow_bf16, gout);                                      \
  else                                                                                                         \
    hipLaunchKernelGGL(KERNEL, grid, block, 0, st, params, velocity, grads, stride, P, seg.K, lam, opt,        \
                       shadow_bf16, gout)
#define OMNI_UPD(SH, MO, KG) \
  if (!few) { OMNI_UPD_((weighted_sgd_kernel<SH, MO, KG>)); }                \
  else if (seg.K <= 4) { OMNI_UPD_((weighted_sgd_few_kernel<4, SH, MO, KG>)); } \
  else if (seg.K <= 8) { OMNI_UPD_((weighted_sgd_few_kernel<8, SH, MO, KG>)); } \
  else { OMNI_UPD_((weighted_sgd_few_kernel<16, SH, MO, KG>)); }
#define OMNI_UPD2(SH, MO)                                 \
  if (gout) { OMNI_UPD(SH, MO, true); } else { OMNI_UPD(SH, MO, false); }
  if (velocity) {
    if (shadow_bf16) { OMNI_UPD2(true, true) } else { OMNI_UPD2(false, true) }
  } else {
    if (shadow_bf16) { OMNI_UPD2(true, false) } else { OMNI_UPD2(false, false) }
  }
#undef OMNI_UPD2
#undef OMNI_UPD
#undef OMNI_UPD_
}

void weighted_sgd_ranges_f32(hipStream_t st, const SgdArgs& sgd, const float* grads, size_t stride, const ParamRange* ranges, int n,
                             const Segments& seg, int workgroups) {
  const Lambdas lam = lambdas_of(seg);
  const Optim opt{sgd.lr, sgd.momentum, sgd.weight_decay};
  for (int base = 0; base < n; base += kRangesMax) {
    RangeTable tab{};
    tab.n = std::min(n - base, kRangesMax);
    for (int i = 0; i < tab.n; ++i) {
      const ParamRange& r = ranges[base + i];
      tab.first[i] = tab.pieces;
      tab.beg[i] = (uint32_t)r.beg;
      tab.end[i] = (uint32_t)r.end;
      tab.pieces += (int)std::max<size_t>((r.end - r.beg + 4095) / 4096, 1);
    }
    const auto kernel = sgd.velocity ? weighted_sgd_ranges_kernel<true> : weighted_sgd_ranges_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(std::min(tab.pieces, workgroups)), dim3(256), 0, st, sgd.params, sgd.velocity, grads, stride, tab, seg.K, lam, opt);
  }
}

void weighted_reduce_f32(hipStream_t st, const float* grads, size_t stride, size_t P, const Segments& seg,
                         float* gout) {
  size_t blocks = (P + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(weighted_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, grads, stride, P, seg.K,
                     lambdas_of(seg), gout);
}

void fill_u32(hipStream_t st, uint32_t* p, size_t n, uint32_t v) {
  if (n == 0) return;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
}

}  // namespace omni
