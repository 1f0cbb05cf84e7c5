// Device code of the classifier head that more than one kernel uses: the wavefront
// reductions and the body of the head's parameter-gradient kernel (a kernel of its own
// in head.hip; a role of the launches of input gradients in gemm_f32*.hip and gemm_bf16.hip
// and of the first convolution's weight gradient in conv_wgrad_bf16.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "bf16.h"
#include "common.h"
#include "kernels.h"

namespace omni {

// Wavefront-wide reductions on the vector ALU's data-parallel primitives: two quad
// permutes and two row mirrors leave every lane with the result of its row of 16, four
// lane reads combine the rows.  (A butterfly of __shfl_xor goes through the LDS crossbar:
// six dependent round trips of ~170 cycles each per reduction; with one wavefront per SIMD
// nothing hides them, and the ten per-class sums of the classifier were most of this
// kernel's time.)
template <int CTRL>
__device__ inline float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ inline float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ inline float wave_sum(float v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
// Losses and label check, one workgroup of any number of wavefronts, one wavefront per worker:
// L_k = mean of the worker's row losses, loss = sum_k lambda_k L_k, status bit 0 if a label lies outside [0, C).
constexpr int kHeadLossLdsFloats = OMNI_MAX_WORKERS;
__device__ __forceinline__ void head_loss_body(const HeadLossParams& h, const Segments& seg, float* part) {
  const int tid = threadIdx.x, nthreads = blockDim.x, lane = tid & 63;
  const int rows = seg.off[seg.K];
  const float invB = 1.0f / (float)rows;
  for (int k = tid >> 6; k < seg.K; k += nthreads >> 6) {
    float a = 0.f;
    const int end = seg.off[k + 1];
    for (int s = seg.off[k] + lane; s < end; s += 512) {   // eight loads in flight, added in order
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = h.loss_rows[min(s + 64 * u, end - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) a += s + 64 * u < end ? v[u] : 0.f;
    }
    a = wave_sum(a);
    if (lane == 0) {
      const float bk = (float)(seg.off[k + 1] - seg.off[k]);
      const float Lk = a / bk;
      h.loss_per_worker[k] = Lk;
      part[k] = bk * invB * Lk;   // lambda_k L_k
    }
  }
  int badl = 0;
  for (int s = tid; s < rows; s += 4 * nthreads) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int y = h.labels[min(s + u * nthreads, rows - 1)];
      badl |= (y < 0 || y >= h.C) ? 1 : 0;
    }
  }
  const int anybad = __syncthreads_or(badl);
  if (tid == 0) {
    float total = 0.f;
    for (int k = 0; k < seg.K; ++k) total += part[k];
    h.loss[0] = total;
    h.status[0] = anybad ? 1u : 0u;
  }
}

// LDS: the row groups' sums of 256 / JC groups x 16 classes x JC columns (rows of JC + 1), and 256 rows of dz.
constexpr int kHeadWgradLdsFloats = 64 * 16 * 5 + 256 * 16;
// Input columns per workgroup: 16, or 8 or 4 where that leaves most of the chip idle (a worker's rows are walked by one
// workgroup per 16 classes and JC columns: one worker with 4096 rows of 1024 columns took 66 us in 64 workgroups).
inline int head_wgrad_columns(int cin, int classes, int K) {
  const long groups = (long)K * ((classes + 15) / 16);
  for (int jc = 16; jc > 4; jc /= 2)
    if (groups * ((cin + jc - 1) / jc) >= 256) return jc;
  return 4;
}
inline dim3 head_wgrad_grid(int cin, int classes, int K) {
  const int jc = head_wgrad_columns(cin, classes, K);
  return dim3(K * ((cin + jc - 1) / jc) + 1, (classes + 15) / 16, 1);
}

// One worker, JC input columns, 16 classes; 256 threads.  Each thread walks one column and every (256 / JC)-th row: of 256
// rows at a time all its elements are on their way before the rows' dz (16 classes of them) is staged in LDS (fetched
// per thread they would be 16 global loads per row, and the vector cache, not the arithmetic, would set the pace).
template <typename T, int JC>
__device__ __forceinline__ void head_wgrad_columns_body(const HeadWgradParams& h, const Segments& seg, int bx, int by,
                                                        float* smem) {
  constexpr int RS = 256 / JC;
  float (*red)[16][JC + 1] = reinterpret_cast<float (*)[16][JC + 1]>(smem);
  float (*dzs)[16] = reinterpret_cast<float (*)[16]>(smem + RS * 16 * (JC + 1));
  const float* __restrict__ dz = h.dz;
  const T* __restrict__ x = static_cast<const T*>(h.x);
  const int cin = h.cin, C = h.C;
  float* __restrict__ gw = h.gw;
  float* __restrict__ gb = h.gb;
  const size_t worker_stride = h.worker_stride;
  const int tid = threadIdx.x;
  const int jchunks = (cin + JC - 1) / JC;
  const int wk = bx / jchunks, jc = bx % jchunks;
  const int jl = tid % JC, rs = tid / JC;
  const int j = min(jc * JC + jl, cin - 1);   // a column past the end shadows the last one and is not stored
  const int c0 = by * 16;
  const int nc = min(16, C - c0);
  const int s_end = seg.off[wk + 1];
  const bool want_bias = jc == 0 && gb != nullptr;
  float acc[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) acc[c] = 0.f;
  float bsum = 0.f;   // class tid % 16, rows tid / 16, + 16, ...

  for (int base = seg.off[wk]; base < s_end; base += 256) {
    const int n = min(256, s_end - base);
    // (a worker often has fewer rows than that: groups of four loads that would all lie past the end are left out)
    const T* xb = x + (size_t)base * cin;          // (uniform bases and 32-bit offsets: half the address registers)
    const float* dzb = dz + (size_t)base * C + c0;
    float av[JC];
#pragma unroll
    for (int u = 0; u < JC; ++u) {
      if (u % 4 == 0 && RS * u >= n) break;
      av[u] = Piece<T>::get(xb + (min(rs + RS * u, n - 1) * cin + j));   // (dz of rows past the end: 0)
    }
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += 8) {          // (eight at a time: registers)
      if (16 * i0 >= n) break;
      float dv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int rr = (tid >> 4) + 16 * (i0 + i), c = tid & 15;
        const bool ok = rr < n && c < nc;
        const float v = dzb[ok ? rr * C + c : 0];
        dv[i] = ok ? v : 0.f;
      }
      if (i0 == 0) __syncthreads();               // the previous 256 rows have been consumed
#pragma unroll
      for (int i = 0; i < 8; ++i) dzs[(tid >> 4) + 16 * (i0 + i)][tid & 15] = dv[i];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < JC; ++u) {
      if (u % 4 == 0 && RS * u >= n) break;
      // (a row of the group that the staged rows do not reach is not counted)
      const bool live = rs + RS * u < n;
      const v4f* d = reinterpret_cast<const v4f*>(&dzs[live ? rs + RS * u : 0][0]);
      const float a = live ? av[u] : 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v4f t = d[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * q + e] += t[e] * a;
      }
    }
    if (want_bias)
      for (int r2 = tid >> 4; r2 < n; r2 += 16) bsum += dzs[r2][tid & 15];
  }

#pragma unroll
  for (int c = 0; c < 16; ++c) red[rs][c][jl] = acc[c];
  __syncthreads();
  if (tid < 16 * JC) {
    const int c = tid / JC, jj = tid % JC;
    float part[4] = {0.f, 0.f, 0.f, 0.f};   // (four short chains: smaller rounding errors, and the reads need not wait for each other)
#pragma unroll 4
    for (int r = 0; r < RS; r += 4)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[q] += red[r + q][c][jj];
    const float t = (part[0] + part[1]) + (part[2] + part[3]);
    if (c < nc && jc * JC + jj < cin)
      gw[(size_t)wk * worker_stride + (size_t)(c0 + c) * cin + jc * JC + jj] = t;
  }
  if (want_bias) {
    // bias gradient: column sums of dz over the worker's rows, 16 row groups x 16 classes
    __syncthreads();
    float* r2 = &red[0][0][0];
    r2[(tid >> 4) * 16 + (tid & 15)] = bsum;
    __syncthreads();
    if (tid < 16 && tid < nc) {
      float u[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 16; ++r) u[r & 3] += r2[r * 16 + tid];
      gb[(size_t)wk * worker_stride + c0 + tid] = (u[0] + u[1]) + (u[2] + u[3]);
    }
  }
}

// Workgroup (bx, by) of a head_wgrad_grid, 256 threads, kHeadWgradLdsFloats floats of LDS at smem (16-byte aligned).  The
// one past the last column computes the losses.
template <typename T>
__device__ __forceinline__ void head_wgrad_loss_body(const HeadWgradParams& h, const Segments& seg, int bx, int by,
                                                     float* smem) {
  const int jchunks = (h.cin + h.columns - 1) / h.columns;
  if (bx == seg.K * jchunks) {
    if (by == 0)
      head_loss_body(HeadLossParams{h.labels, h.C, h.loss_rows, h.loss_per_worker, h.loss, h.status}, seg, smem);
    return;
  }
  if (h.columns == 16) head_wgrad_columns_body<T, 16>(h, seg, bx, by, smem);
  else if (h.columns == 8) head_wgrad_columns_body<T, 8>(h, seg, bx, by, smem);
  else head_wgrad_columns_body<T, 4>(h, seg, bx, by, smem);
}

// The classifier's part of a launch it shares with a matrix product: its workgroups come first (they are short but wait for
// memory most of the time, so they should not be left for the end).
struct HeadRole {
  HeadWgradParams p;
  int gx, blocks;   // blocks = 0: no such part
};
inline HeadRole head_role(const HeadWgradParams* h, const Segments& seg) {
  HeadRole r{};
  if (!h) return r;
  const dim3 g = head_wgrad_grid(h->cin, h->C, seg.K);
  r.p = *h;
  r.gx = (int)g.x;
  r.blocks = (int)(g.x * g.y);
  return r;
}

}  // namespace omni
