// Fully connected layers of bf16 networks (v_mfma_f32_32x32x16_bf16, fp32 accumulation):
//   forward   Y  = X W^T + bias, optional ReLU        (W: the step's bf16 copy, [cout][cin])
//   dgrad     dX = dY W, optional ReLU mask           (W: the transposed copy, [cin][cout]: the same product)
//   wgrad     G_k = dY_k^T X_k for every worker, several layers in one launch, with the update where the step applies it
//
// These layers are short: a few GFLOP spread over a chip that does 2.5 in a microsecond, so what counts is how many compute
// units take part and how little each of them waits.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>

#include "bf16.h"
#include "common.h"
#include "head_device.h"
#include "kernels.h"
#include "lds_transpose_device.h"
#include "update_device.h"
#include "xcd_tiles.h"

namespace omni {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

// ------------------------------------------------------------------ forward and input gradient
struct BfGemm {
  const bf16_t* A;     // [M][K]
  const bf16_t* B;     // [N][K]
  bf16_t* C;           // [M][N]
  int M, N, K;         // K and N multiples of 8
  const float* bias;   // [N], may be null
  const bf16_t* mask;  // [M][N], the value passes where mask > 0, may be null
  int relu;
  XcdTiles tiles;
};

// A workgroup owns a tile of 32 WB x 32 WB outputs; its four wavefronts split the reduction, each with the whole tile in
// registers, and their partial tiles are added in wavefront order at the end.  Wavefronts share no operand data, so the main
// loop has no barrier: a chunk of 64 reduction elements arrives in 128-byte lines (8 lanes per row) and turns into the
// instruction's layout through wavefront-private LDS (36-word rows: conflict-free both ways).
// Bound by LDS bandwidth: WB = 2 moves 32 KB per 16 matrix instructions of 32 cycles.  1024 rows, 3072 -> 1024 -> 1024: both
// products 23.6 us, 364 TFLOP/s.
constexpr int kLine = 64;          // reduction elements of a chunk: 128 bytes
constexpr int kLineWords = 36;

template <int WB> constexpr int bf16_gemm_words() { return 4 * 2 * 32 * WB * kLineWords; }

template <int WB>
__device__ __forceinline__ void bf16_gemm_body(const BfGemm& p, int block, uint32_t* lds) {
  constexpr int T = 32 * WB, NL = 4 * WB, D = 2;     // NL: 16-byte pieces of an operand's chunk per lane
  constexpr int kWave = 2 * T * kLineWords;          // words of a wavefront's LDS block
  static_assert(kWave >= T * T, "the partial tile reuses the staging block");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5, lrow = lane >> 3, lp = lane & 7;
  const int M = p.M, N = p.N, K = p.K;
  int tile_m, tile_n;
  if (!xcd_tile(p.tiles, block, tile_m, tile_n)) return;
  const int row0 = tile_m * T, col0 = tile_n * T;
  uint32_t* la = lds + wave * kWave;
  uint32_t* lb = la + T * kLineWords;

  // rows past the end shadow the last ones (their results are not stored); a piece past the end of a row shadows its last
  // piece and counts zero, in both operands (0 * infinity is no zero)
  const bf16_t* a0 = p.A + (size_t)row0 * K;
  const bf16_t* b0 = p.B + (size_t)col0 * K;
  uint32_t aoff[NL], boff[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    aoff[i] = (uint32_t)min(lrow + 8 * i, M - 1 - row0) * (uint32_t)K;
    boff[i] = (uint32_t)min(lrow + 8 * i, N - 1 - col0) * (uint32_t)K;
  }
  const int nc = (K + kLine - 1) / kLine;
  const int cb = wave * nc / 4, ce = (wave + 1) * nc / 4;
  u32x4 ga[D][NL], gb[D][NL];
  auto fetch = [&](int d, int ch) {
    const uint32_t k = (uint32_t)min(ch * kLine + lp * 8, K - 8);
#pragma unroll
    for (int i = 0; i < NL; ++i) ga[d][i] = *reinterpret_cast<const u32x4*>(a0 + (aoff[i] + k));
#pragma unroll
    for (int i = 0; i < NL; ++i) gb[d][i] = *reinterpret_cast<const u32x4*>(b0 + (boff[i] + k));
  };
  v16f acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto stage = [&](int d, int ch) {
    if (__builtin_expect((ch + 1) * kLine > K, 0)) {
      const bool beyond = ch * kLine + lp * 8 >= K;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        ga[d][i] = beyond ? u32x4{0u, 0u, 0u, 0u} : ga[d][i];
        gb[d][i] = beyond ? u32x4{0u, 0u, 0u, 0u} : gb[d][i];
      }
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(la + (lrow + 8 * i) * kLineWords + lp * 4) = ga[d][i];
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4*>(lb + (lrow + 8 * i) * kLineWords + lp * 4) = gb[d][i];
  };
  auto multiply = [&]() {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      bf16x8 fa[WB], fb[WB];
#pragma unroll
      for (int i = 0; i < WB; ++i) {
        fa[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(la + (32 * i + r) * kLineWords + 8 * ks + 4 * h));
        fb[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(lb + (32 * i + r) * kLineWords + 8 * ks + 4 * h));
      }
#pragma unroll
      for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < WB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  };
  // What the results are combined with at the end travels beside the last products.
  constexpr int kOut = (T * T / 8 + 255) / 256;   // eight neighbouring results each of a thread, all in the same columns
  static_assert(256 % (T / 8) == 0, "the same columns");
  float bias[8];
  u32x4 mask[kOut];
  auto fetch_rest = [&]() {
    const int col = min(col0 + tid % (T / 8) * 8, N - 8);
#pragma unroll
    for (int q = 0; q < 8; ++q) bias[q] = p.bias ? p.bias[col + q] : 0.f;
#pragma unroll
    for (int o = 0; o < kOut; ++o)
      mask[o] = p.mask ? *reinterpret_cast<const u32x4*>(p.mask + (size_t)min(row0 + (o * 256 + tid) / (T / 8), M - 1) * N + col)
                       : u32x4{0u, 0u, 0u, 0u};
  };
  if (ce <= cb) fetch_rest();
  if (ce > cb) {
    // (a chunk past this wavefront's last one is that one again, unused: loads are never conditional)
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d, min(cb + d, ce - 1));
    int ch = cb;
    for (; ch + D < ce; ch += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        stage(d, ch + d);
        fetch(d, min(ch + d + D, ce - 1));
        multiply();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (ch + d < ce) {
        stage(d, ch + d);
        if (ch + d == ce - 1) fetch_rest();   // (not earlier: the chunks under way take all registers)
        multiply();
      }
  }

  // register v of lane (r, h): row 8 (v / 4) + 4 h + v % 4 of its block, column r
  float* part = reinterpret_cast<float*>(la);
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) part[(32 * i + 8 * (v >> 2) + 4 * h + (v & 3)) * T + 32 * j + r] = acc[i][j][v];
  __syncthreads();
  const float* all = reinterpret_cast<const float*>(lds);
#pragma unroll
  for (int e0 = 0; e0 < T * T / 8; e0 += 256) {
    const int e = e0 + tid;
    if (T * T / 8 < 256 && e >= T * T / 8) break;
    const int lr = e / (T / 8), lc = e % (T / 8) * 8, row = row0 + lr, col = col0 + lc;
    if (row >= M || col >= N) continue;
    float y[8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      v4f t = *reinterpret_cast<const v4f*>(all + lr * T + lc + 4 * q);
#pragma unroll
      for (int w = 1; w < 4; ++w) t += *reinterpret_cast<const v4f*>(all + w * kWave + lr * T + lc + 4 * q);
#pragma unroll
      for (int q2 = 0; q2 < 4; ++q2) y[4 * q + q2] = t[q2];
    }
    const size_t idx = (size_t)row * N + col;
    if (p.bias) {
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] += bias[q];
    }
    if (p.relu) {
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = y[q] > 0.f ? y[q] : 0.f;
    }
    if (p.mask) {
      float m[8];
      for (int q = 0; q < 4; ++q) {
        m[2 * q] = bf16_lo(mask[e0 / 256][q]);
        m[2 * q + 1] = bf16_hi(mask[e0 / 256][q]);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = m[q] > 0.f ? y[q] : 0.f;
    }
    Piece<bf16_t>::store(p.C + idx, y);
  }
}

template <int WB>
__global__ __launch_bounds__(256, 2) void bf16_gemm_kernel(BfGemm p) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[bf16_gemm_words<WB>()];
  bf16_gemm_body<WB>(p, (int)blockIdx.x, lds);
}

// An input gradient and, in front of its tiles, the classifier's parameter gradients and losses.
template <int WB>
__global__ __launch_bounds__(256, 2) void bf16_dgrad_head_kernel(BfGemm p, HeadRole head, Segments seg) {
  constexpr int kWords = bf16_gemm_words<WB>() > kHeadWgradLdsFloats ? bf16_gemm_words<WB>() : kHeadWgradLdsFloats;
  __shared__ __attribute__((aligned(16))) uint32_t lds[kWords];
  const int b = (int)blockIdx.x;
  if (b < head.blocks) head_wgrad_loss_body<bf16_t, WB == 2 ? 4 : 2>(head.p, seg, b, head.gx, reinterpret_cast<float*>(lds));
  else bf16_gemm_body<WB>(p, b - head.blocks, lds);
}

// ------------------------------------------------------------------ weight gradients
constexpr int kThreads = 256;
constexpr int kTile = 64;                 // outputs per side of a workgroup's tile
constexpr int kRows = 64;                 // reduction rows of a slab
constexpr int kSlabStride = 160;          // bytes per slab row: 128 of data; four consecutive rows start in different bank octets
constexpr int kSlab = kRows * kSlabStride;
constexpr int kFlushStride = kTile + 4;
static_assert(kTile * (kFlushStride + 4) * 4 <= 2 * kSlab, "the staged output tile and bias sums must fit one LDS stage");

struct BfWgradJob {
  const bf16_t* dy;    // [rows][M]
  const bf16_t* x;     // [rows][N]
  float* gw;           // worker 0's [M][N]
  float* gb;           // worker 0's [M], may be null
  float* theta;        // with the update: the layer's weights, bias and their velocities
  float* theta_bias;
  float* vel;
  float* vel_bias;
  int M, N;
};
constexpr int kBfJobs = 8;
struct BfWgrad {
  int n;
  int start[kBfJobs + 1];
  size_t worker_stride;
  long head_n;             // classifier: parameters, where they start, and worker 0's gradients of them
  float* head_theta;
  float* head_vel;
  const float* head_grad;
  BfWgradJob job[kBfJobs];
};

// A workgroup owns a 64 x 64 tile of one layer's weights and walks through all workers' rows, 64 at a time, both operands in
// LDS as they arrive ([row][column]); where a worker's rows end the tile goes out to G[k], and with UPD (1 SGD, 2 momentum)
// sum_k lambda_k G[k] of the pieces a thread stores stays in its registers for the update of the tile's parameters at the
// end.  APART: a workgroup per tile and worker instead (UPD = 0), see wgrad_workers_apart.  Bound by the gradient rows it writes
// (K x 4 bytes per weight), with few tiles by the walk: 3072-1024-1024, eight workers, 1024 rows, momentum: 39.4 us
// for 201 MB, 5.1 TB/s, which is what a large copy reaches.
template <int UPD, bool APART>
__global__ __launch_bounds__(kThreads, 4) void bf16_wgrad_kernel(BfWgrad b, Segments seg, Lambdas lam, Optim opt) {
  constexpr bool MOM = UPD == 2;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][2 * kSlab];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (UPD != 0 && (int)blockIdx.x >= b.start[b.n]) {
    const long j = (long)((int)blockIdx.x - b.start[b.n]) * kThreads + tid;
    if (j >= b.head_n) return;
    float g = 0.f;
#pragma unroll 4
    for (int k = 0; k < seg.K; ++k) g += lam.v[k] * b.head_grad[(size_t)k * b.worker_stride + j];
    float th = b.head_theta[j], ve = MOM ? b.head_vel[j] : 0.f;
    apply_update<MOM>(th, ve, g, opt);
    b.head_theta[j] = th;
    if (MOM) b.head_vel[j] = ve;
    return;
  }
  static_assert(!APART || UPD == 0, "the update needs all workers");
  const int wbeg = APART ? (int)((unsigned)blockIdx.x / (unsigned)b.start[b.n]) : 0, wend = APART ? wbeg + 1 : seg.K;
  const int bx = (int)blockIdx.x - wbeg * b.start[b.n];
  int ji = 0;
  for (int i = 1; i < b.n; ++i)
    if (bx >= b.start[i]) ji = i;
  const BfWgradJob& J = b.job[ji];
  const int M = J.M, N = J.N;
  const int tiles_n = (N + kTile - 1) / kTile;
  const int local = bx - b.start[ji];
  const int tile_m = local / tiles_n, tile_n = local - tile_m * tiles_n;
  const int i0 = tile_m * kTile, j0 = tile_n * kTile;
  const bool want_bias = J.gb != nullptr && tile_n == 0;

  // staging: thread = row tid / 8 (+ 32), 16-byte piece tid % 8; a piece past the last column shadows the last one (its
  // outputs are not stored), rows past a worker's end are stored as zeros in both operands
  const int lrow = tid >> 3, lp = (tid & 7) * 8;
  const bf16_t* dyp = J.dy + min(i0 + lp, M - 8);
  const bf16_t* xp = J.x + min(j0 + lp, N - 8);
  const int last_row = seg.off[seg.K] - 1;
  u32x4 ra[2], rb[2];
  auto fetch = [&](int k) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const size_t row = (size_t)min(k + lrow + 32 * t, last_row);
      ra[t] = *reinterpret_cast<const u32x4*>(dyp + row * M);
      rb[t] = *reinterpret_cast<const u32x4*>(xp + row * N);
    }
  };
  auto stage = [&](unsigned char* s, int live) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      u32x4 a = ra[t], c = rb[t];
      if (live < kRows && lrow + 32 * t >= live) a = c = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(s + (lrow + 32 * t) * kSlabStride + lp * 2) = a;
      *reinterpret_cast<u32x4*>(s + kSlab + (lrow + 32 * t) * kSlabStride + lp * 2) = c;
    }
  };

  // fragment addresses: lane group g = lane / 16 hands in row 8 (g / 2) + s / 4 (+ 4 for the second read) and columns
  // 16 (g % 2) + 4 (s % 4) .. + 3 of a step of 16 rows, s = lane % 16
  const int g = lane >> 4, s = lane & 15;
  const int frow = 8 * (g >> 1) + (s >> 2), fcol = 16 * (g & 1) + 4 * (s & 3);
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
  const int aofs = frow * kSlabStride + (wi + fcol) * 2, bofs = kSlab + frow * kSlabStride + (wj + fcol) * 2;

  // Four slabs are summed by themselves, then added to the worker's sum: one chain over all rows had up to 3.5 times the error
  // against float64 that chunks of 256 rows have.
  constexpr int kGroup = 4;
  v16f acc, slab;
  int slabs = 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = slab[v] = 0.f;
  v4f gsum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) gsum[q] = v4f{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f, bgsum = 0.f;

  int w = wbeg, k = APART ? seg.off[wbeg] : 0, end = seg.off[wbeg + 1], cur = 0;
  fetch(k);
  for (;;) {
    unsigned char* st = lds[cur];
    const int live = min(kRows, end - k);
    stage(st, live);
    // the slab after this one
    int w2 = w, k2 = k + kRows, end2 = end;
    if (k2 >= end) {
      ++w2;
      if (w2 < wend) { k2 = seg.off[w2]; end2 = seg.off[w2 + 1]; }
    }
    fetch(min(k2, last_row));
    __syncthreads();
    const int steps = (live + 15) / 16;
#pragma unroll
    for (int ks = 0; ks < kRows / 16; ++ks) {
      if (ks < steps) {
        const unsigned char* pa = st + aofs + 16 * ks * kSlabStride;
        const unsigned char* pb = st + bofs + 16 * ks * kSlabStride;
        const bf16x8 fa = tr_pair(pa, pa + 4 * kSlabStride);
        const bf16x8 fb = tr_pair(pb, pb + 4 * kSlabStride);
        slab = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, slab, 0, 0, 0);
      }
    }
    if (++slabs == kGroup || w2 != w) {
      slabs = 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc[v] += slab[v]; slab[v] = 0.f; }
    }
    if (want_bias) {
#pragma unroll
      for (int rr = 0; rr < kRows / 4; ++rr)
        bsum += bf16_to_f32(*reinterpret_cast<const bf16_t*>(st + (wave * (kRows / 4) + rr) * kSlabStride + lane * 2));
    }
    if (w2 != w) {
      // this worker's rows are done: its tile goes out through the stage that was just multiplied, in 16-byte pieces
      float* G = J.gw + (size_t)w * b.worker_stride;
      float* tile = reinterpret_cast<float*>(st);
      float (*bred)[kTile] = reinterpret_cast<float (*)[kTile]>(tile + kTile * kFlushStride);
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v)
        tile[(wi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * kFlushStride + wj + (lane & 31)] = acc[v];
      if (want_bias) bred[wave][lane] = bsum;
      __syncthreads();
      const float l = UPD ? lam.v[w] : 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int idx = tid + kThreads * q, r = idx >> 4, c4 = (idx & 15) * 4;
        const v4f t = *reinterpret_cast<const v4f*>(tile + r * kFlushStride + c4);
        if (i0 + r < M && j0 + c4 < N) *reinterpret_cast<v4f_a4*>(G + (size_t)(i0 + r) * N + j0 + c4) = t;
        if (UPD) gsum[q] += l * t;
      }
      if (want_bias && tid < kTile) {
        const float t = ((bred[0][tid] + bred[1][tid]) + bred[2][tid]) + bred[3][tid];
        if (i0 + tid < M) J.gb[(size_t)w * b.worker_stride + i0 + tid] = t;
        if (UPD) bgsum += l * t;
      }
      bsum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
      if (w2 >= wend) break;
    }
    w = w2; k = k2; end = end2;
    cur ^= 1;
  }

  if constexpr (UPD != 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = tid + kThreads * q, r = idx >> 4, c4 = (idx & 15) * 4;
      if (i0 + r >= M || j0 + c4 >= N) continue;
      const size_t at = (size_t)(i0 + r) * N + j0 + c4;
      v4f th = *reinterpret_cast<const v4f_a4*>(J.theta + at), ve = {0.f, 0.f, 0.f, 0.f};
      if (MOM) ve = *reinterpret_cast<const v4f_a4*>(J.vel + at);
      apply_update<MOM>(th, ve, gsum[q], opt);
      *reinterpret_cast<v4f_a4*>(J.theta + at) = th;
      if (MOM) *reinterpret_cast<v4f_a4*>(J.vel + at) = ve;
    }
    if (want_bias && tid < kTile && i0 + tid < M) {
      float th = J.theta_bias[i0 + tid], ve = MOM ? J.vel_bias[i0 + tid] : 0.f;
      apply_update<MOM>(th, ve, bgsum, opt);
      J.theta_bias[i0 + tid] = th;
      if (MOM) J.vel_bias[i0 + tid] = ve;
    }
  }
}

// Whether every worker has workgroups of its own (APART), and the update is a launch of its own behind them: the walk through the
// workers, a microsecond and more each, against that launch (4 us and the reading of G).  Step in us, together / apart:
//    24 tiles  2 workers,  200 rows 27.7 / 28.2   4, 480 32.1 / 29.7    16, 600 45.6 / 33.3   32, 3000 94.7 / 50.7
//    51 tiles  4 workers,  170 rows 42.0 / 43.1
//    88 tiles  2 workers,  200 rows 30.5 / 30.9   4, 480 35.4 / 33.5    16, 600 50.0 / 40.5   32, 3000 104 / 65.1
//   160 tiles  4 workers,  480 rows 34.8 / 34.9   8,  64 35.5 / 38.6  8, 1500 57.8 / 46.8   16, 128 47.1 / 45.7   32, 3000 104 / 80.2
//   512 tiles  8 workers, 1500 rows 70.2 / 76.0  16, 600 58.0 / 79.4
bool wgrad_workers_apart(long tiles, const Segments& seg) {
  const int rows = seg.off[seg.K];
  if (tiles <= 96) return seg.K >= 5 || (seg.K == 4 && (tiles <= 24 || rows >= 400));
  return tiles <= 160 && (seg.K >= 16 || (seg.K >= 8 && rows >= 1024));
}

inline int tiles_of(int rows, int cols, int t) { return ((rows + t - 1) / t) * ((cols + t - 1) / t); }

}  // namespace

void linear_bf16(hipStream_t st, const bf16_t* a, const bf16_t* b, bf16_t* c, int M, int N, int K, const float* bias,
                 bool relu, const bf16_t* mask, const HeadWgradParams* head, const Segments& seg) {
  BfGemm p{a, b, c, M, N, K, bias, mask, relu ? 1 : 0, {}};
  // 64 x 64 tiles need half the operand traffic of 32 x 32 ones; they are taken once they cover the compute units
  const int t64 = tiles_of(M, N, 64);
  const int T = t64 >= 192 ? 64 : 32;
  p.tiles = xcd_tiles((M + T - 1) / T, (N + T - 1) / T);
  if (head) {
    const HeadRole role = head_role(head, seg);
    const dim3 grid(p.tiles.grid() + role.blocks);
    if (T == 64) hipLaunchKernelGGL(bf16_dgrad_head_kernel<2>, grid, dim3(256), 0, st, p, role, seg);
    else hipLaunchKernelGGL(bf16_dgrad_head_kernel<1>, grid, dim3(256), 0, st, p, role, seg);
    return;
  }
  if (T == 64)
    hipLaunchKernelGGL((bf16_gemm_kernel<2>), dim3(p.tiles.grid()), dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((bf16_gemm_kernel<1>), dim3(p.tiles.grid()), dim3(256), 0, st, p);
}

bool linear_wgrad_bf16(hipStream_t st, const LinearWgradBf16Job* jobs, int n, size_t worker_stride, const Segments& seg,
                       const LinearWgradBf16Job* head, const SgdArgs* sgd, const KernelTimer* timer) {
  const bool one = n <= kBfJobs;
  long tiles = 0;
  for (int i = 0; i < n; ++i) tiles += tiles_of(jobs[i].cout, jobs[i].cin, kTile);
  const bool apart = one && tiles > 0 && wgrad_workers_apart(tiles, seg);
  if (apart) sgd = nullptr;
  const int upd = sgd ? (sgd->velocity ? 2 : 1) : 0;
  const Lambdas lam = lambdas_of(seg);
  const Optim opt = sgd ? Optim{sgd->lr, sgd->momentum, sgd->weight_decay} : Optim{0.f, 0.f, 0.f};
  if (timer && !one) (void)hipEventRecord(timer->start, st);
  int base = 0;
  do {
    BfWgrad p{};
    p.n = std::min(n - base, kBfJobs);
    p.worker_stride = worker_stride;
    for (int i = 0; i < p.n; ++i) {
      const LinearWgradBf16Job& j = jobs[base + i];
      BfWgradJob& q = p.job[i];
      q.dy = j.dy; q.x = j.x; q.gw = j.gw; q.gb = j.gb; q.M = j.cout; q.N = j.cin;
      if (sgd) {
        q.theta = sgd->params + j.w_off; q.theta_bias = sgd->params + j.b_off;
        if (sgd->velocity) { q.vel = sgd->velocity + j.w_off; q.vel_bias = sgd->velocity + j.b_off; }
      }
      p.start[i + 1] = p.start[i] + tiles_of(j.cout, j.cin, kTile);
    }
    if (sgd && head && base + kBfJobs >= n) {
      p.head_n = (long)head->cout * head->cin + (head->gb ? head->cout : 0);   // (the bias follows the weight)
      p.head_theta = sgd->params + head->w_off;
      if (sgd->velocity) p.head_vel = sgd->velocity + head->w_off;
      p.head_grad = head->gw;
    }
    const dim3 grid(p.start[p.n] * (apart ? seg.K : 1) + (unsigned)((p.head_n + kThreads - 1) / kThreads)), block(kThreads);
#define OMNI_BF_WGRAD(U, A)                                                                                         \
  if (timer && one)                                                                                                 \
    hipExtLaunchKernelGGL((bf16_wgrad_kernel<U, A>), grid, block, 0, st, timer->start, timer->stop, 0, p, seg, lam, opt); \
  else                                                                                                              \
    hipLaunchKernelGGL((bf16_wgrad_kernel<U, A>), grid, block, 0, st, p, seg, lam, opt)
    if (apart) { OMNI_BF_WGRAD(0, true); }
    else if (upd == 0) { OMNI_BF_WGRAD(0, false); }
    else if (upd == 1) { OMNI_BF_WGRAD(1, false); }
    else { OMNI_BF_WGRAD(2, false); }
#undef OMNI_BF_WGRAD
    base += kBfJobs;
  } while (base < n);
  if (timer && !one) (void)hipEventRecord(timer->stop, st);
  return sgd != nullptr;
}

}  // namespace omni
