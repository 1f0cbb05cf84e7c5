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

// LDS: the four wavefronts' 16 x 64 (16) tiles and their sums of dz.
constexpr int kHeadWgradLdsFloats = 4 * (16 * 64 + 16);
// Input columns per workgroup: 64, or 16 where that leaves at most 24 workgroups, whose walk is then the launch (four matrix
// instructions per four rows and 64 columns), or where a wavefront walks 24 blocks of 16 rows and more and there are fewer workgroups than
// compute units.  bf16, 64 / 16 columns: step of 512-128-10 with one worker, 96 rows 20.9 / 19.9 us, 1500 rows 52.3 / 43.8; 512-512-37,
// 1000 rows 47.1 / 41.7; with more workgroups it is the product or the convolution beside it that waits: 512-512-512-10, six workers, 3000
// rows (48) 80.9 / 83.5, 3-32-64-64-10, three workers, 600 images (48) 132.2 / 133.5, eight workers, 512 (128) 114.3 / 116.0.
inline int head_wgrad_columns(int cin, int classes, const Segments& seg) {
  const long groups = (long)seg.K * ((classes + 15) / 16) * ((cin + 63) / 64);
  return groups <= 24 || (groups < 256 && seg.off[seg.K] / seg.K > 4 * 24 * 16) ? 16 : 64;
}
inline dim3 head_wgrad_grid(const HeadWgradParams& h, const Segments& seg) {
  return dim3(seg.K * ((h.cin + h.columns - 1) / h.columns) + 1, (h.C + 15) / 16, 1);
}

// One worker, 16 WB input columns, 16 classes; 256 threads: gw = dz^T x on the fp32 matrix instruction (bf16 inputs are exact in
// fp32).  The four wavefronts take blocks of 16 rows in turn, operands straight from global memory (their layout is the
// instruction's: one class, WB columns and every fourth row per lane), DEPTH blocks in flight (as many as
// the registers of the launch it is in allow), eight rows summed by themselves, into two or four running totals; their tiles are added in a fixed order.  A block that would run past the end of the worker's rows is moved back to end there; rows that are not its
// own count zero in both operands.  Columns past the end are the last ones again and are not stored.
// (A thread per column with dz staged in LDS read 64 bytes of LDS per row: 1024 rows of 2048 inputs, eight workers, 10 classes
// in a launch of its own 7.5 -> 5.3 us, beside the first convolution's weight gradient 6.7 -> 2.3 us more.)
template <typename T, int WB> struct HeadInputs;
template <> struct HeadInputs<float, 4> {
  typedef v4f raw;
  __device__ static inline raw load(const float* p) { return *reinterpret_cast<const v4f_a4*>(p); }
  __device__ static inline float get(const raw& v, int e) { return v[e]; }
};
template <> struct HeadInputs<float, 1> {
  typedef float raw;
  __device__ static inline raw load(const float* p) { return *p; }
  __device__ static inline float get(raw v, int) { return v; }
};
template <> struct HeadInputs<bf16_t, 4> {       // (widths are multiples of 8: aligned)
  typedef u32x2 raw;
  __device__ static inline raw load(const bf16_t* p) { return *reinterpret_cast<const u32x2*>(p); }
  __device__ static inline float get(const raw& v, int e) { return e & 1 ? bf16_hi(v[e >> 1]) : bf16_lo(v[e >> 1]); }
};
template <> struct HeadInputs<bf16_t, 1> {
  typedef bf16_t raw;
  __device__ static inline raw load(const bf16_t* p) { return *p; }
  __device__ static inline float get(raw v, int) { return bf16_to_f32(v); }
};

template <typename T, int WB, int DEPTH>
__device__ __forceinline__ void head_wgrad_tile_body(const HeadWgradParams& h, const Segments& seg, int wk, int jc, int by, float* smem) {
  typedef HeadInputs<T, WB> In;
  constexpr int TN = 16 * WB, kTile = 16 * TN + 16, D = WB == 1 ? 4 : DEPTH, NS = WB == 1 ? 4 : 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int s0 = seg.off[wk], s1 = seg.off[wk + 1], last = seg.off[seg.K] - 1;
  const int cin = h.cin, C = h.C, c0 = by * 16, j0 = jc * TN;
  const int col = min(j0 + WB * r, cin - WB);
  const T* const x = static_cast<const T*>(h.x) + col;
  const float* const dz = h.dz + min(c0 + r, C - 1);
  const bool want_bias = jc == 0 && h.gb != nullptr;
  const int blocks = (s1 - s0 + 63 - 16 * wave) >> 6;       // of this wavefront
  float a[D][4];
  typename In::raw b[D][4];
  auto start = [&](int i) { return max(min(s0 + 16 * wave + 64 * i, s1 - 16), 0); };
  auto load = [&](int d, int i) {
    const int at = start(min(i, blocks - 1));
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = min(at + 4 * t + g, last);            // (fewer than 16 rows in all)
      a[d][t] = dz[(size_t)row * C];
      b[d][t] = In::load(x + (size_t)row * cin);
    }
  };
  v4f acc[NS][WB];                                          // (in turn: short chains)
  float bsum[NS];
#pragma unroll
  for (int d = 0; d < NS; ++d) {
    bsum[d] = 0.f;
#pragma unroll
    for (int e = 0; e < WB; ++e) acc[d][e] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  if (blocks > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, d);
    for (int i0 = 0; i0 < blocks; i0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int i = i0 + d;
        if (i < blocks) {
          const int lo = s0 + 16 * wave + 64 * i, at = start(i);
#pragma unroll
          for (int half = 0; half < 2; ++half) {            // eight rows by themselves
            v4f sum[WB];
            float bs = 0.f;
#pragma unroll
            for (int t = 2 * half; t < 2 * half + 2; ++t) {
              const int row = at + 4 * t + g;
              const bool own = row >= lo && row < s1;
              const float av = own ? a[d][t] : 0.f;
              bs += av;
#pragma unroll
              for (int e = 0; e < WB; ++e)
                sum[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, own ? In::get(b[d][t], e) : 0.f,
                                                              t % 2 == 0 ? v4f{0.f, 0.f, 0.f, 0.f} : sum[e], 0, 0, 0);
            }
            const int set = (2 * d + half) % NS;
#pragma unroll
            for (int e = 0; e < WB; ++e) acc[set][e] += sum[e];
            bsum[set] += bs;
          }
          if (i + D < blocks) load(d, i + D);
        }
      }
    }
  }
  float* const mine = smem + wave * kTile;
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int e = 0; e < WB; ++e) mine[(4 * g + v) * TN + WB * r + e] = NS == 2 ? acc[0][e][v] + acc[1][e][v] : (acc[0][e][v] + acc[1][e][v]) + (acc[NS - 2][e][v] + acc[NS - 1][e][v]);
  if (want_bias) {
    float t = NS == 2 ? bsum[0] + bsum[1] : (bsum[0] + bsum[1]) + (bsum[NS - 2] + bsum[NS - 1]);
    t += __shfl_xor(t, 16, 64);
    t += __shfl_xor(t, 32, 64);
    if (g == 0) mine[16 * TN + r] = t;
  }
  __syncthreads();
  float* const gw = h.gw + (size_t)wk * h.worker_stride + (size_t)c0 * cin;
#pragma unroll
  for (int q = 0; q < WB; ++q) {
    const int e = q * 256 + tid, c = e / TN, nom = j0 + e % TN / WB * WB, cc = min(nom, cin - WB) + e % WB;
    const float t = (smem[e] + smem[kTile + e]) + (smem[2 * kTile + e] + smem[3 * kTile + e]);
    if (c0 + c < C && cc >= nom) gw[(size_t)c * cin + cc] = t;   // (of a group moved back, what the group before it also holds is left to that one)
  }
  if (want_bias && tid < 16 && c0 + tid < C) {
    const float* const q = smem + 16 * TN + tid;
    h.gb[(size_t)wk * h.worker_stride + c0 + tid] = (q[0] + q[kTile]) + (q[2 * kTile] + q[3 * kTile]);
  }
}

// Workgroup b of a head_wgrad_grid (rows of gx), 256 threads, kHeadWgradLdsFloats floats of LDS at smem (16-byte aligned).  The
// one past the last column computes the losses.
template <typename T, int DEPTH>
__device__ __forceinline__ void head_wgrad_loss_body(const HeadWgradParams& h, const Segments& seg, int b, int gx, float* smem) {
  int bx = b, by = 0;
  while (bx >= gx) { bx -= gx; ++by; }
  if (bx == gx - 1) {
    if (by == 0)
      head_loss_body(HeadLossParams{h.labels, h.C, h.loss_rows, h.loss_per_worker, h.loss, h.status}, seg, smem);
    return;
  }
  const int chunks = (h.cin + h.columns - 1) / h.columns, wk = bx / chunks, jc = bx - wk * chunks;
  if (h.columns == 64) head_wgrad_tile_body<T, 4, DEPTH>(h, seg, wk, jc, by, smem);
  else head_wgrad_tile_body<T, 1, DEPTH>(h, seg, wk, jc, by, smem);
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
  const dim3 g = head_wgrad_grid(*h, seg);
  r.p = *h;
  r.gx = (int)g.x;
  r.blocks = (int)(g.x * g.y);
  return r;
}

}  // namespace omni
