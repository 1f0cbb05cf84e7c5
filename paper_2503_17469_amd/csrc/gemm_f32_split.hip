// Large fp32 matrix products on the bf16 matrix instruction (v_mfma_f32_32x32x16_bf16).
//
// The contractions of gemm_f32.hip (Algorithm 1, procedure Train, the gradient line, fully connected layers):
//   forward   Y  = X W^T + bias,  dgrad  dX = dY W,  wgrad  G_k = dY_k^T X_k (with the update, as there)
// where the output has enough 128 x 128 tiles to fill the chip.  The fp32 instruction's pipe is what bounds those (154 TFLOP/s; 104
// were reached, staging instructions between); the bf16 one is sixteen times as fast.  Every operand element is taken as the
// exact sum of three bf16 values, scaled (split_bf16_device.h), and of the nine products the six that reach 2^-24 of the whole are
// formed, exactly, and added in fp32.  What is left out is at most 2^-24 of a product, with random signs: a sum of one
// product is off by up to 2.5 x 2^-24 (0.58 in the root mean square), where the fp32 instruction rounds once (1, 0.43).
//
// Measured, 3072-1024-1024-10, 4096 rows, against the fp32 instruction: forward 222 -> 149 and 75 -> 54 us, input gradient 85 -> 63,
// weight gradients of sixteen workers with the update 346 -> 270 (all of them 2.5 % longer since operands are scaled); 160 to 167
// TFLOP/s in whole steps, that is 1.0 PFLOP/s of bf16 products, where a loop of nothing but these matrix instructions reaches 1.40 on
// the same data (the clock falls under the load).  Error against float64 (2-norm), as a part of the fp32 kernels': forward 0.4 to 0.7 (32 to 8192
// elements), input gradients 0.5 to 0.9, weight gradients 0.35 to 0.75 from 8 rows of a worker on, the same at 4, but 1.2 at 2 and
// 1.4 at one.
//
// A workgroup has a 128 x 128 tile and eight wavefronts: a 2 x 2 grid of 64 x 64 blocks, twice; the two wavefronts of a block take
// the two halves of every slab of 32 reduction elements, and their sums are added at the end.  (Four wavefronts with the
// whole slab each have one wavefront per SIMD and no partner to fill the gaps: 144 instead of 180 TFLOP/s.  64 x 32 blocks read
// half as much again from LDS per instruction.)  Elements are split once, on their way to LDS.  Smaller tiles split too often for
// what they multiply: 64 x 64 and 64 x 32 tiles, with the reduction cut four or eight ways, were no faster than the fp32 kernels
// at 480 to 1500 rows.
//
// The instruction rounds down: products that share a sum, and the sum they are added to, are cut off at 2^-24 of the largest
// product, towards minus infinity (0.085 x 2^-24 of the absolute products' sum, all outputs alike, however long the reduction).  So
// the second half of every slab is summed with the opposite sign, and subtracted.
//
// The pipeline: while a slab is multiplied from registers, the next one's fragments are read from LDS, the one after that is
// split and written where the present one lay, and the fourth is sent for.  One barrier per slab.
//
// Infinities and NaN, and operands from 2^104 on, come out of the products as infinity or NaN, never as a number, and so do sums
// from 2^80 on; sums that are not finite are formed again with the fp32 instruction, whose results then stand.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "head_device.h"
#include "kernels.h"
#include "lds_limit.h"
#include "split_bf16_device.h"
#include "update_device.h"
#include "xcd_tiles.h"

namespace omni {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8s __attribute__((ext_vector_type(8)));

namespace {

constexpr int kTile = 128, kThreads = 512;
constexpr int BK = 32;              // reduction elements per slab
constexpr int kShares = 2;          // wavefronts per 64 x 64 block
// A weight gradient adds at most so many rows of a worker in one chain of slabs; longer ones go to G in pieces (4096 rows of
// one worker: 0.35 instead of 0.71 times the fp32 kernel's error, for 5 us per piece).
constexpr int kChunkRows = 512;

enum { MODE_FWD = 0, MODE_DGRAD = 1, MODE_WGRAD = 2 };

// LDS, in 16-byte pieces of 8 reduction elements: a row of an operand has 4 per plane and 3 planes, and every fourth row is
// followed by one more, so that the pieces of 16 rows (reads; writes of both kinds) lie in 16 different parts of the banks.
__host__ __device__ __forceinline__ constexpr int row_piece(int r) { return 12 * r + (r >> 2); }
constexpr int kOperand = row_piece(kTile), kStage = 2 * kOperand;
// Two stages, and between them what the flush of a weight gradient needs beyond one of them: both shares' tiles, 64 rows at a time.
constexpr int kFlushRows = 64, kFlushPitch = kTile + 4;
constexpr int kExtra = kShares * kFlushRows * kFlushPitch / 4 - kStage;
constexpr size_t kGemmLds = (size_t)kShares * kTile * kTile * sizeof(float);           // (the shares' tiles at the end)
constexpr size_t kWgradLds = (size_t)(2 * kStage + kExtra) * 16 + BK / 8 * kTile * sizeof(float);
static_assert(kExtra > 0 && kGemmLds >= (size_t)2 * kStage * 16 && kGemmLds <= kLdsOfComputeUnit && kWgradLds <= kLdsOfComputeUnit,
              "LDS of a workgroup");

// One operand's slab, 128 rows x 32 reduction elements: a piece of 8 elements per thread.  MC: rows are contiguous in memory
// (element (r, k) at base[k * ld + r]), else the reduction is.
template <bool MC>
struct Operand {
  float v[8];
  const float* ptr;

  __device__ static __forceinline__ int row_of(int tid) { return MC ? tid % kTile : tid / (BK / 8); }
  __device__ static __forceinline__ int k8_of(int tid) { return MC ? tid / kTile : tid % (BK / 8); }
  __device__ __forceinline__ void prepare(const float* base, int ld, int row0, int rows, int tid) {
    const int r = min(row0 + row_of(tid), rows - 1);   // (rows past the end feed outputs that are not stored)
    ptr = base + (MC ? (size_t)(k8_of(tid) * 8) * ld + r : (size_t)r * ld + k8_of(tid) * 8);
  }
  __device__ static __forceinline__ int share_of(int tid) { return k8_of(tid) / (BK / 8 / kShares); }
  // (16-byte loads from any multiple of 4 bytes)
  __device__ __forceinline__ void load(int ld, int ks) {
    if (!MC) {
      const v4f lo = *reinterpret_cast<const v4f_a4*>(ptr + ks), hi = *reinterpret_cast<const v4f_a4*>(ptr + ks + 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) { v[q] = lo[q]; v[4 + q] = hi[q]; }
    } else {
      const float* p = ptr + (size_t)ks * ld;
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = p[(size_t)q * ld];
    }
  }
  // clears what lies outside [lo, hi) of the slab
  __device__ __forceinline__ void clear_outside(int lo, int hi, int tid) {
    if (lo > 0 || hi < BK) {
      const int k = k8_of(tid) * 8;
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = (k + q >= lo && k + q < hi) ? v[q] : 0.f;
    }
  }
  __device__ __forceinline__ void store(u32x4* lds, int tid, float scale) const {
    uint32_t w[3][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) split3(v[2 * q], v[2 * q + 1], scale, w[0][q], w[1][q], w[2][q]);
    u32x4* at = lds + row_piece(row_of(tid)) + k8_of(tid);
#pragma unroll
    for (int p = 0; p < 3; ++p) at[4 * p] = u32x4{w[p][0], w[p][1], w[p][2], w[p][3]};
  }
  // waits for the loads on their way
  __device__ __forceinline__ void arrived() {
#pragma unroll
    for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(v[q]));
  }
};

struct SplitParams {
  const float* A;
  const float* B;
  float* C;
  int M, N;            // rows of A / rows of B = rows / columns of C
  int lda, ldb, ldc;
  int kred;            // reduction length (forward, input gradient)
  const float* bias;   // forward, may be null
  const float* mask;   // input gradient, [M][ldc], may be null: the value passes where mask > 0
  int relu, accumulate;
  XcdTiles xcd;        // forward, input gradient
  // weight gradient: as in gemm_f32.hip
  size_t c_worker_stride;
  float* bias_grad;
  float* theta;
  float* theta_bias;
  float* velocity;
  float* velocity_bias;
};

// The whole workgroup program.  UPD (weight gradient): 1 / 2 with the SGD / momentum update of the tile's parameters.
template <bool A_MC, bool B_MC, int MODE, int UPD>
__device__ __forceinline__ void split_body(const SplitParams& p, const Segments& seg, const int bx, u32x4* lds,
                                           const Lambdas* lam = nullptr, const Optim* opt = nullptr) {
  constexpr bool WGRAD = MODE == MODE_WGRAD;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int share = wave >> 2, r32 = lane & 31, h = lane >> 5;
  const int wrow = (wave >> 1 & 1) * 64, wcol = (wave & 1) * 64;
  int tile_m, tile_n;
  if (WGRAD) {
    const int tiles_n = (p.N + kTile - 1) / kTile;
    tile_m = bx / tiles_n; tile_n = bx % tiles_n;
  } else if (!xcd_tile(p.xcd, bx, tile_m, tile_n)) {
    return;
  }
  const int row0 = tile_m * kTile, col0 = tile_n * kTile;
  auto stage = [&](int s) { return lds + s * (kStage + kExtra); };

  // The reduction is a stream of slabs over chunks (weight gradient: of the workers' rows; else one); w == nrange marks the end.
  // A slab that would run past the end of its chunk is moved back to end there, and what is not its own is cleared in both operands.
  enum { kCont = 1, kMore = 2 };                  // the worker has chunks before this one, behind it
  struct Slab { int c, w, k0, kend, pieces; };    // chunk, worker, first reduction element, end of the chunk, the two above
  const int nrange = WGRAD ? seg.K : 1;
  auto chunk = [&](Slab s) {              // its end
    const int end = seg.off[s.w + 1];
    s.kend = min(s.k0 + kChunkRows, end);
    if (s.kend < end) s.pieces |= kMore;
    return s;
  };
  auto first = [&]() { return WGRAD ? chunk(Slab{0, 0, seg.off[0], 0, 0}) : Slab{0, 0, 0, p.kred, 0}; };
  auto after = [&](Slab s) {
    if (s.w >= nrange) return s;
    Slab t{s.c, s.w, s.k0 + BK, s.kend, s.pieces};
    if (t.k0 < s.kend) return t;
    ++t.c;
    t.k0 = s.kend;
    t.pieces = kCont;
    if (!WGRAD || !(s.pieces & kMore)) {
      if (++t.w >= nrange) return t;
      t.k0 = seg.off[t.w];
      t.pieces = 0;
    }
    return chunk(t);
  };
  auto live = [&](Slab s) { return s.w < nrange ? s : first(); };
  auto start = [&](Slab s) { return s.k0 + BK <= s.kend ? s.k0 : max(s.kend - BK, 0); };

  Operand<A_MC> a;
  Operand<B_MC> b;
  const float scale_a = Operand<A_MC>::share_of(tid) == 0 ? kSplitScale : -kSplitScale;    // (the second share sums -A B)
  a.prepare(p.A, p.lda, row0, p.M, tid);
  b.prepare(p.B, p.ldb, col0, p.N, tid);
  const bool want_bias_grad = WGRAD && p.bias_grad != nullptr && tile_n == 0;
  float (*bred)[kTile] = reinterpret_cast<float (*)[kTile]>(lds + 2 * kStage + kExtra);
  float bsum = 0.f, bnext = 0.f, bpart = 0.f;   // of the chunk up to slab s0, of s1, of s2 (below); this thread's row and k8

  v16f tot[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) tot[i][j][v] = 0.f;
  // sum_k lambda_k G[k] of the 16-byte pieces this thread stores
  constexpr int kPieces = kTile * kTile / 4 / kThreads, kParts = kTile / kFlushRows;
  v4f gsum[WGRAD && UPD ? kPieces : 1];
#pragma unroll
  for (int q = 0; q < (WGRAD && UPD ? kPieces : 1); ++q) gsum[q] = v4f{0.f, 0.f, 0.f, 0.f};
  float bgsum = 0.f;
  v4f theta[WGRAD && UPD ? kPieces : 1], vel[WGRAD && UPD == 2 ? kPieces : 1];   // of those pieces
  bool notfinite = false;

  auto take = [&](Slab s) {       // registers of slab s made ready for LDS
    const int st = start(s);
    a.clear_outside(s.k0 - st, s.kend - st, tid);
    b.clear_outside(s.k0 - st, s.kend - st, tid);
    if (want_bias_grad) bpart = ((a.v[0] + a.v[1]) + (a.v[2] + a.v[3])) + ((a.v[4] + a.v[5]) + (a.v[6] + a.v[7]));
  };
  // (past the end: the first slab again, dropped; loads are never conditional)
  auto send = [&](Slab s) {
    const int st = start(live(s));
    a.load(p.lda, st);
    b.load(p.ldb, st);
  };
  // Slab s0 is being multiplied (its fragments are in registers), s1 is in LDS, s2 on its way to registers.
  Slab s0 = first(), s1 = after(s0), s2 = after(s1);
  send(s0);
  take(s0);
  a.store(stage(0), tid, scale_a);
  b.store(stage(0) + kOperand, tid, kSplitScale);
  bsum = bpart;
  send(s1);
  take(live(s1));
  a.store(stage(1), tid, scale_a);
  b.store(stage(1) + kOperand, tid, kSplitScale);
  bnext = bpart;
  send(s2);
  if (WGRAD) { a.arrived(); b.arrived(); }      // (see the loop)
  __syncthreads();

  // Lane l of the instruction's operands: row l % 32, reduction elements 8 (l / 32) .. + 7 of the share's sixteen.
  constexpr int kBlock = row_piece(32);
  const int fragA = row_piece(wrow + r32) + 2 * share + h, fragB = kOperand + row_piece(wcol + r32) + 2 * share + h;
  bf16x8s fa[2][3], fb[2][3];
  auto read_a = [&](const u32x4* st, int i, int q) { return __builtin_bit_cast(bf16x8s, st[fragA + i * kBlock + 4 * q]); };
  auto read_b = [&](const u32x4* st, int j, int q) { return __builtin_bit_cast(bf16x8s, st[fragB + j * kBlock + 4 * q]); };
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      fa[i][q] = read_a(stage(0), i, q);
      fb[i][q] = read_b(stage(0), i, q);
    }
  __syncthreads();
  int cur = 0;
  // One slab; true when it was the last of a chunk (done: that slab).  Forward and input gradient keep the sums of two slabs
  // in acc before they join the total (fresh: the first of the two); a weight gradient has no registers for that (it holds
  // gsum) and adds every block's sixteen elements to the total by themselves.
  v16f acc[WGRAD ? 1 : 2][WGRAD ? 1 : 2];
  Slab done = s0;
  auto step = [&](auto fresh) {
    const Slab s3 = after(s2);
    const u32x4* rst = stage(cur ^ 1);
    u32x4* wst = stage(cur);
    bf16x8s na[2][3], nb[2][3];
    take(live(s2));
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};   // smallest products first
    if constexpr (!WGRAD) {
#pragma unroll
      for (int t = 0; t < 6; ++t) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (decltype(fresh)::value && t == 0) {
              v16f z;
#pragma unroll
              for (int v = 0; v < 16; ++v) z[v] = 0.f;
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][pa[t]], fb[j][pb[t]], z, 0, 0, 0);
            } else {
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][pa[t]], fb[j][pb[t]], acc[i][j], 0, 0, 0);
            }
          }
        if (t == 0) a.store(wst, tid, scale_a);
        if (t == 1) { b.store(wst + kOperand, tid, kSplitScale); send(s3); }
        // fragments that no later product needs make room for the next slab's
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (t == 0) na[i][2] = read_a(rst, i, 2);
          if (t == 1) nb[i][2] = read_b(rst, i, 2);
          if (t == 3) { na[i][1] = read_a(rst, i, 1); na[i][0] = read_a(rst, i, 0); }
          if (t == 4) { nb[i][1] = read_b(rst, i, 1); nb[i][0] = read_b(rst, i, 0); }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      // block by block, the second row from the right, so that fragments are done with early
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const int i = blk >> 1, j = (blk & 1) ^ i;
        v16f c;
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] = 0.f;
#pragma unroll
        for (int t = 0; t < 6; ++t) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][pa[t]], fb[j][pb[t]], c, 0, 0, 0);
        if (blk == 0) a.store(wst, tid, scale_a);
        if (blk == 1) { b.store(wst + kOperand, tid, kSplitScale); send(s3); }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          if (i == 1) nb[j][q] = read_b(rst, j, q);
          if (blk & 1) na[i][q] = read_a(rst, i, q);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) tot[i][j][v] += c[v];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i][q] = na[i][q];
        fb[i][q] = nb[i][q];
      }
    __syncthreads();
    cur ^= 1;
    done = s0;
    const bool ended = s1.c != s0.c;
    if (want_bias_grad && !ended) { bsum += bnext; bnext = bpart; }
    s0 = s1; s1 = s2; s2 = s3;
    return ended;
  };
  auto flush = [&](auto last) {
    constexpr bool LAST = decltype(last)::value;
    // The chunk's tile goes out through the stage that is free (slab s0's, whose fragments are in registers) and the extra area.
    a.arrived();
    b.arrived();
    int ft = tid;
    asm volatile("" : "+v"(ft));      // (addresses are worked out here, not kept in registers through the loop)
    float* C = p.C + (size_t)done.w * p.c_worker_stride;
    float* out = reinterpret_cast<float*>(cur == 1 ? lds + kStage : lds);
    if (want_bias_grad) bred[Operand<A_MC>::k8_of(ft)][Operand<A_MC>::row_of(ft)] = bsum;
    const bool cont = done.pieces & kCont;       // added to the worker's earlier chunks
    const bool whole = !cont && row0 + kTile <= p.M && col0 + kTile <= p.N;
    // The update takes G once it is complete, as one in a launch of its own does: the same bits.
    const bool complete = !(done.pieces & kMore);
    const float weight = UPD ? lam->v[done.w] : 0.f;
    // The update's parameters set out in front of the last chunk's stores: behind them they would wait for those.  Step of the 3072
    // net in us, behind / in front: one worker, 500 rows 106 / 103; four, 480 rows 111.2 / 109.4, with momentum 118.2 / 114.0; eight, 1000 rows
    // 213.9 / 213.4; sixteen, 4096 rows 568 / 561.  (This copy of the flush stands behind the loop: inside it they spilled.)
    if constexpr (UPD != 0 && LAST) {
#pragma unroll
      for (int q = 0; q < kPieces; ++q) {
        const int part = q / (kPieces / kParts), idx = ft + kThreads * (q % (kPieces / kParts));
        const int row = row0 + part * kFlushRows + idx / (kTile / 4), col = col0 + (idx % (kTile / 4)) * 4;
        const size_t e0 = row < p.M && col + 4 <= p.N ? (size_t)row * p.ldc + col : 0;
        theta[q] = *reinterpret_cast<const v4f_a4*>(p.theta + e0);
        if (UPD == 2) vel[UPD == 2 ? q : 0] = *reinterpret_cast<const v4f_a4*>(p.velocity + e0);
      }
    }
#pragma unroll
    for (int part = 0; part < kParts; ++part) {
      __syncthreads();
      if (wrow / kFlushRows == part) {
        float* o = out + share * kFlushRows * kFlushPitch;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              o[(32 * i + 4 * (ft >> 5 & 1) + 8 * (v / 4) + (v % 4)) * kFlushPitch + wcol + 32 * j + (ft & 31)] = tot[i][j][v];
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPieces / kParts; ++q) {
        const int idx = ft + kThreads * q, r = idx / (kTile / 4), c4 = (idx % (kTile / 4)) * 4;
        const float* o = out + r * kFlushPitch + c4;
        v4f g = *reinterpret_cast<const v4f*>(o) * kSplitUnscale -
                *reinterpret_cast<const v4f*>(o + kFlushRows * kFlushPitch) * kSplitUnscale;   // (each: the sum may be large)
        const int row = row0 + part * kFlushRows + r;
        float* dst = C + (size_t)row * p.ldc + col0 + c4;
        if (whole) {
          *reinterpret_cast<v4f_a4*>(dst) = g;
        } else if (row < p.M) {
          // (16 bytes at a time as well: element by element, 1021 x 3400 outputs of 32 workers took 54 us longer, and the eight
          // pieces of a worker with 4096 rows 37)
          if (col0 + c4 + 4 <= p.N) {
            v4f_a4* const to = reinterpret_cast<v4f_a4*>(dst);
            if (cont) g += *to;
            *to = g;
          } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
              if (col0 + c4 + e < p.N) {
                if (cont) g[e] += dst[e];
                dst[e] = g[e];
              }
          }
        }
        if (UPD && complete) gsum[part * (kPieces / kParts) + q] += weight * g;
      }
    }
    if (want_bias_grad && ft < kTile) {
      float g = (bred[0][ft] + bred[1][ft]) + (bred[2][ft] + bred[3][ft]);
      if (row0 + ft < p.M) {
        float* dst = p.bias_grad + (size_t)done.w * p.c_worker_stride + row0 + ft;
        if (cont) g += *dst;
        *dst = g;
      }
      if (UPD && complete) bgsum += weight * g;
    }
  };
  for (;;) {
    if constexpr (!WGRAD) {
      for (bool ended = false; !ended;) {
        ended = step(std::true_type());
        if (!ended) ended = step(std::false_type());
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) tot[i][j] += acc[i][j];
      }
    } else {
      // The first step of a chunk is a copy of its own: its loads are older than the previous chunk's stores and have
      // arrived; a wait shared with the steps that follow no stores would wait for the stores too.
      bool ended = step(std::true_type());
      while (!ended) ended = step(std::true_type());
    }

    float bad = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) bad += tot[i][j][v] * 0.f;
    notfinite = notfinite || bad != bad;

    if (!WGRAD || s0.w >= nrange) break;
    if constexpr (WGRAD) {
      flush(std::false_type{});
      __syncthreads();      // (the free stage is written again)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) tot[i][j][v] = 0.f;
      bsum = bnext;
      bnext = bpart;
    }
  }
  if constexpr (WGRAD) flush(std::true_type{});

  // Sums that are not finite once more, from memory, in pieces of 32 elements; what is finite stays (a row's results do not depend
  // on other rows).  Here, where nothing else is in registers: beside the loop it spilled, and the spills' waits were the stores'.
  const int ri = wrow + 32 * share;      // 32 of the block's rows by each wavefront
  auto again = [&](int j, int kb, int ke) {
    const int ra = min(row0 + ri + r32, p.M - 1), rb = min(col0 + wcol + 32 * j + r32, p.N - 1);
    v16f sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.f;
#pragma unroll 1
    for (; kb < ke; kb += BK) {
      v16f c;
#pragma unroll
      for (int v = 0; v < 16; ++v) c[v] = 0.f;
#pragma unroll 4
      for (int k = kb; k < min(kb + BK, ke); k += 2) {
        const int kk = min(k + h, ke - 1);
        float x = A_MC ? p.A[(size_t)kk * p.lda + ra] : p.A[(size_t)ra * p.lda + kk];
        float y = B_MC ? p.B[(size_t)kk * p.ldb + rb] : p.B[(size_t)rb * p.ldb + kk];
        if (k + h >= ke) x = y = 0.f;
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, c, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[v] += c[v];
    }
    return sum;
  };
  auto row_of = [&](int v) { return ri + 4 * h + 8 * (v >> 2) + (v & 3); };
  const bool repair = __syncthreads_or(notfinite);
  if (WGRAD && repair) {
    for (int w = 0; w < seg.K; ++w) {
      float* C = p.C + (size_t)w * p.c_worker_stride;
#pragma unroll 1
      for (int j = 0; j < 2; ++j) {
        const v16f c = again(j, seg.off[w], seg.off[w + 1]);
        const int col = col0 + wcol + 32 * j + r32;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (row0 + row_of(v) < p.M && col < p.N) {
            float* dst = C + (size_t)(row0 + row_of(v)) * p.ldc + col;
            const float z = *dst * 0.f;
            if (z != z) *dst = c[v];
          }
      }
    }
    __syncthreads();
    if (UPD) {
#pragma unroll
      for (int q = 0; q < kPieces; ++q) {
        const int part = q / (kPieces / kParts), idx = tid + kThreads * (q % (kPieces / kParts));
        const int row = row0 + part * kFlushRows + idx / (kTile / 4), col = col0 + (idx % (kTile / 4)) * 4;
        gsum[q] = v4f{0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < seg.K; ++w)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (row < p.M && col + e < p.N)
              gsum[q][e] += lam->v[w] * p.C[(size_t)w * p.c_worker_stride + (size_t)row * p.ldc + col + e];
      }
    }
  }

  if constexpr (WGRAD && UPD != 0) {
    constexpr bool MOM = UPD == 2;
#pragma unroll
    for (int q = 0; q < kPieces; ++q) {
      const int part = q / (kPieces / kParts), idx = tid + kThreads * (q % (kPieces / kParts));
      const int row = row0 + part * kFlushRows + idx / (kTile / 4), col = col0 + (idx % (kTile / 4)) * 4;
      if (row >= p.M || col >= p.N) continue;
      const size_t e0 = (size_t)row * p.ldc + col;
      if (col + 4 <= p.N) {
        v4f th = theta[q], ve = vel[MOM ? q : 0];
        apply_update<MOM>(th, ve, gsum[q], *opt);
        *reinterpret_cast<v4f_a4*>(p.theta + e0) = th;
        if (MOM) *reinterpret_cast<v4f_a4*>(p.velocity + e0) = ve;
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          if (col + e >= p.N) continue;
          float th = p.theta[e0 + e], ve = MOM ? p.velocity[e0 + e] : 0.f;
          const float g = gsum[q][e];
          apply_update<MOM>(th, ve, g, *opt);
          p.theta[e0 + e] = th;
          if (MOM) p.velocity[e0 + e] = ve;
        }
      }
    }
    if (want_bias_grad && tid < kTile && row0 + tid < p.M) {
      float th = p.theta_bias[row0 + tid], ve = MOM ? p.velocity_bias[row0 + tid] : 0.f;
      apply_update<MOM>(th, ve, bgsum, *opt);
      p.theta_bias[row0 + tid] = th;
      if (MOM) p.velocity_bias[row0 + tid] = ve;
    }
  }
  if constexpr (!WGRAD) {
    // both shares' tiles to LDS; each wavefront adds and stores half of its block's registers
    float* out = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) out[(wave * 64 + (i * 2 + j) * 16 + v) * 64 + lane] = tot[i][j][v];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      v16f sum;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int slot = ((wave & 3) * 64 + (share * 2 + j) * 16 + v) * 64 + lane;
        sum[v] = out[slot] * kSplitUnscale - out[slot + 4 * 64 * 64] * kSplitUnscale;   // (each: the sum may be large)
      }
      if (repair) {
        const v16f c = again(j, 0, p.kred);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float z = sum[v] * 0.f;
          sum[v] = z != z ? c[v] : sum[v];
        }
      }
      const int col = col0 + wcol + 32 * j + r32;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + row_of(v);
        if (row < p.M && col < p.N) {
          float val = sum[v];
          const size_t idx = (size_t)row * p.ldc + col;
          if (MODE == MODE_FWD) {
            if (p.bias) val += p.bias[col];
            if (p.relu) val = val > 0.f ? val : 0.f;
          } else {
            if (p.mask) val = p.mask[idx] > 0.f ? val : 0.f;
            if (p.accumulate) val += p.C[idx];
          }
          p.C[idx] = val;
        }
      }
    }
  }
}

template <bool B_MC, int MODE>
__global__ __launch_bounds__(kThreads, 1) void split_gemm_kernel(SplitParams p) {
  extern __shared__ __attribute__((aligned(16))) u32x4 smem_split[];
  split_body<false, B_MC, MODE, 0>(p, Segments{}, (int)blockIdx.x, smem_split);
}

// Weight gradients of several layers in one launch, and with the update the classifier's parameters behind them: as in
// gemm_f32.hip.
constexpr int kMaxBatch = 8;
struct SplitWgradBatch {
  int n;
  int start[kMaxBatch + 1];
  size_t worker_stride;
  long head_n;
  float* head_theta;
  float* head_velocity;
  const float* head_grad;
  SplitParams prob[kMaxBatch];
};

template <int UPD>
__global__ __launch_bounds__(kThreads, 1) void split_wgrad_kernel(SplitWgradBatch b, Segments seg, Lambdas lam, Optim opt) {
  extern __shared__ __attribute__((aligned(16))) u32x4 smem_split[];
  if (UPD != 0 && (int)blockIdx.x >= b.start[b.n]) {
    const long j = (long)((int)blockIdx.x - b.start[b.n]) * kThreads + threadIdx.x;
    if (j >= b.head_n) return;
    float g = 0.f;
#pragma unroll 4
    for (int k = 0; k < seg.K; ++k) g += lam.v[k] * b.head_grad[(size_t)k * b.worker_stride + j];
    float th = b.head_theta[j], ve = UPD == 2 ? b.head_velocity[j] : 0.f;
    apply_update<UPD == 2>(th, ve, g, opt);
    b.head_theta[j] = th;
    if (UPD == 2) b.head_velocity[j] = ve;
    return;
  }
  int pi = 0;
  for (int i = 1; i < b.n; ++i)
    if ((int)blockIdx.x >= b.start[i]) pi = i;
  split_body<true, true, MODE_WGRAD, UPD>(b.prob[pi], seg, (int)blockIdx.x - b.start[pi], smem_split, &lam, &opt);
}

long tiles_of(int rows, int cols) { return (long)((rows + kTile - 1) / kTile) * ((cols + kTile - 1) / kTile); }

// A compute unit holds one workgroup.  A round of 256 whole tiles takes 0.69 to 0.78 of the time the fp32 kernel needs for as much,
// so the rounds have to be useful to four fifths: 4096 rows, 1024 -> 1024 54 / 75 us; with half the rows 53 / 42.
bool fills_rounds(long tiles, long outputs) { return outputs * 5 >= (tiles + 255) / 256 * 256 * kTile * kTile * 4; }

template <bool B_MC, int MODE>
void launch(hipStream_t st, SplitParams& p) {
  p.xcd = xcd_tiles((p.M + kTile - 1) / kTile, (p.N + kTile - 1) / kTile);
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&split_gemm_kernel<B_MC, MODE>), kGemmLds);
  hipLaunchKernelGGL((split_gemm_kernel<B_MC, MODE>), dim3(p.xcd.grid()), dim3(kThreads), kGemmLds, st, p);
}

}  // namespace

bool linear_f32_split(int rows, int cols, int kred) { return kred >= BK && fills_rounds(tiles_of(rows, cols), (long)rows * cols); }

void linear_fwd_f32_split(hipStream_t st, const float* x, const float* w, const float* bias, float* y, int rows, int cin,
                          int cout, bool relu) {
  SplitParams p{};
  p.A = x; p.B = w; p.C = y; p.M = rows; p.N = cout; p.lda = cin; p.ldb = cin; p.ldc = cout;
  p.kred = cin; p.bias = bias; p.relu = relu ? 1 : 0;
  launch<false, MODE_FWD>(st, p);
}

void linear_dgrad_f32_split(hipStream_t st, const float* dy, const float* w, const float* mask, float* dx, int rows, int cin,
                            int cout, bool accumulate) {
  SplitParams p{};
  p.A = dy; p.B = w; p.C = dx; p.M = rows; p.N = cin; p.lda = cout; p.ldb = cin; p.ldc = cin;
  p.kred = cout; p.mask = mask; p.accumulate = accumulate ? 1 : 0;
  launch<true, MODE_DGRAD>(st, p);
}

// Every worker costs a slab that its rows seldom fill and a flush through LDS with five barriers, so that it is rows per worker that
// count, a hundred of them on average; and few rows are bound by the writing of G either way, so at least 400 in all.  Steps, split /
// fp32, in us:
//   3072-1024-1024-10    1 worker,   256 rows  74 /  74    512 rows 107 / 113   1024 rows 200 / 213
//                        4 workers,  256 rows  80 /  75    400 rows 111 / 114   1024 rows 198 / 212
//                       16 workers,  512 rows 141 / 126   1024 rows 225 / 224   2048 rows 354 / 378
//                       32 workers, 1024 rows 275 / 259   2048 rows 405 / 411   4096 rows 603 / 644
//   3400-1021-10         4 workers,  256 rows  70 /  64    400 rows 104 / 103   1024 rows 160 / 170
//                       16 workers, 1024 rows 202 / 188   1536 rows 278 / 270   2048 rows 306 / 309
// No worker of fewer than four rows: sums of one to three products are nearer to float64 on the fp32 instruction (see above).
bool linear_wgrad_f32_split_shape(const LinearWgradJob* jobs, int n, const Segments& seg) {
  if (seg.off[seg.K] < 100 * std::max((int)seg.K, 4)) return false;
  for (int k = 0; k < seg.K; ++k)
    if (seg.off[k + 1] - seg.off[k] < 4) return false;
  long tiles = 0, outputs = 0;
  for (int i = 0; i < n; ++i) {
    tiles += tiles_of(jobs[i].cout, jobs[i].cin);
    outputs += (long)jobs[i].cout * jobs[i].cin;
  }
  return n <= kMaxBatch && fills_rounds(tiles, outputs);
}

void linear_wgrad_f32_split(hipStream_t st, const LinearWgradJob* jobs, int n, size_t worker_stride,
                            const Segments& seg, const LinearWgradJob* head, const SgdArgs* sgd, const KernelTimer* timer) {
  const int upd = sgd ? (sgd->velocity ? 2 : 1) : 0;
  const Lambdas lam = lambdas_of(seg);
  const Optim opt = sgd ? Optim{sgd->lr, sgd->momentum, sgd->weight_decay} : Optim{0.f, 0.f, 0.f};
  SplitWgradBatch b{};
  b.n = n;
  b.worker_stride = worker_stride;
  for (int i = 0; i < n; ++i) {
    const LinearWgradJob& j = jobs[i];
    SplitParams& p = b.prob[i];
    p.A = j.dy; p.B = j.x; p.C = j.gw; p.M = j.cout; p.N = j.cin; p.lda = j.cout; p.ldb = j.cin; p.ldc = j.cin;
    p.c_worker_stride = worker_stride; p.bias_grad = j.gb;
    if (sgd) {
      p.theta = sgd->params + j.w_off; p.theta_bias = sgd->params + j.b_off;
      if (sgd->velocity) { p.velocity = sgd->velocity + j.w_off; p.velocity_bias = sgd->velocity + j.b_off; }
    }
    b.start[i + 1] = b.start[i] + (int)tiles_of(p.M, p.N);
  }
  if (sgd && head) {
    b.head_n = (long)head->cout * head->cin + (head->gb ? head->cout : 0);   // (the bias follows the weight)
    b.head_theta = sgd->params + head->w_off;
    if (sgd->velocity) b.head_velocity = sgd->velocity + head->w_off;
    b.head_grad = head->gw;
  }
  const dim3 grid(b.start[n] + (unsigned)((b.head_n + kThreads - 1) / kThreads)), block(kThreads);
#define OMNI_WGRAD(U)                                                                                                  \
  {                                                                                                                    \
    static LdsLimit limit;                                                                                             \
    limit.raise(reinterpret_cast<const void*>(&split_wgrad_kernel<U>), kWgradLds);                                     \
    if (timer)                                                                                                         \
      hipExtLaunchKernelGGL((split_wgrad_kernel<U>), grid, block, kWgradLds, st, timer->start, timer->stop, 0, b, seg, \
                            lam, opt);                                                                                 \
    else                                                                                                               \
      hipLaunchKernelGGL((split_wgrad_kernel<U>), grid, block, kWgradLds, st, b, seg, lam, opt);                       \
  }
  if (upd == 0) OMNI_WGRAD(0)
  else if (upd == 1) OMNI_WGRAD(1)
  else OMNI_WGRAD(2)
#undef OMNI_WGRAD
}

}  // namespace omni
