// Forward and input gradient of bf16 convolutions as implicit GEMMs on the CDNA4
// matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation), and which kernel
// takes which layer (conv_gemm_bf16).
//
// These are the contractions inside the per-worker gradient of Algorithm 1
// (procedure Train, gradient line) for the convolutional networks:
//   forward  Y[m][co]  = sum_{u,v,ci} X[n, h*s+u-p, w*s+v-p, ci] * W[co][u][v][ci]
//   dgrad    dX[m][ci] = sum_{u,v,co} dY[n, (h+p-u)/s, (w+p-v)/s, co] * Wt[ci][u][v][co]
// with channels-last activations, m = (n, h, w); both see all workers' rows in one
// launch.  The weight gradients are in conv_wgrad_bf16.hip.
//
// Kernel A (any shape): 128 x (64*TN) output tile per workgroup, 4
// wavefronts in a 2x2 grid, each 64 x (32*TN).  The left operand is gathered
// on the fly (no im2col buffer): a 16-byte piece holds 8 consecutive channels of
// one filter tap, so it is contiguous in memory.  Slabs of 64 reduction
// elements go through LDS (double buffered, next slab prefetched to registers).
// The output width must be a multiple of 8 (16-byte output pieces).  It has a mode
// for the dgrad of stride-2 layers that multiplies only the filter taps an input
// position can meet (a quarter of a 3x3 filter).
//
// Kernel D (3x3 / pad 1 / stride 1, channels a multiple of 32): 256 positions x 64 (32 for
// narrow layers) channels per workgroup; the input patch of the positions stays in LDS, so
// the nine taps are row offsets into it and cost no extra global loads.
//
// Kernel F (3 input channels stored as 8, forward): the filter bank in registers.
//
// In files of their own: few positions (conv_frag_bf16.hip, asked first), 3x3 / stride 1
// (conv3_wide_bf16.hip; kernel D has what it leaves: pooling without a ReLU or on maps other than 16 and 8
// wide, narrow layers with a mask, few units), a residual block's entry (conv3s2_dgrad_bf16.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "bf16.h"
#include "bn_sums_device.h"
#include "cast_device.h"
#include "common.h"
#include "conv_device.h"
#include "kernels.h"
#include "lds_limit.h"
#include "pool_device.h"
#include "quotient.h"

namespace omni {

namespace {

constexpr int BM = 128;

// the same with explicit extents: m -> (n, h, w) over planes of hw positions, rows of wd
__device__ inline void decode_pos2(int hw, int wd, int m, int& n, int& h, int& w) {
  n = (int)((float)m * (1.0f / (float)hw));
  if (n * hw > m) --n;
  if ((n + 1) * hw <= m) ++n;
  const int r = m - n * hw;
  h = (int)((float)r * (1.0f / (float)wd));
  if (h * wd > r) --h;
  if ((h + 1) * wd <= r) ++h;
  w = r - h * wd;
}

// ------------------------------------------------------------------ kernel A
struct ConvParams {
  const bf16_t* src;   // gathered tensor [rows][Hs][Ws][Cs]
  const bf16_t* wgt;   // [N][K]
  bf16_t* out;         // [M][N]
  int M, N;
  ConvGeom g;
  const float* bias;   // [N] or null
  const bf16_t* mask;  // [M][N] or null: the value passes where mask > 0
  int relu, accumulate;
  const bf16_t* addend;   // [M][N] or null: added to the product before the mask (a second gradient contribution)
};

// Balance of kernel A: the vector ALU shares issue slots with the matrix pipe, and
// a first version (32-element slabs, per-piece gather arithmetic, 2-byte stores)
// spent three quarters of them away from the matrix pipe.  Hence
//   * a slab is 64 reduction elements (16 MFMAs per wavefront per barrier);
//   * FAST (channels a multiple of 64, filter <= 3x3, dgrad only for stride 1): a
//     slab lies inside one filter tap, so the tap is wavefront-uniform; each
//     thread keeps the pixel offset of its four rows and a 9-bit "tap inside the
//     image" mask, and a piece address is two adds;
//   * the output tile is staged through LDS as fp32 and leaves as 16-byte pieces
//     (bias, ReLU, mask, accumulate applied there).
//   * PHASED (dgrad of a stride-2 convolution, channels a multiple of 64): an input
//     position (h, w) only meets the filter taps whose parity matches (h+pad-u and
//     w+pad-v even), a quarter of a 3x3 filter on average.  Rows are enumerated
//     parity class by parity class (each class padded to whole tiles), so the set
//     of live taps is uniform over a workgroup and dead taps are never multiplied.
constexpr int BK2 = 64;
enum { GEN = 0, FASTM = 1, PHASED = 2 };

// (Launch bounds cap the kernels at 256 registers: the compiler then issues the MFMAs on ordinary
// registers; with accumulation registers it copied every accumulator in around the MFMAs of each slab.)
template <int TN, int MODE>
__global__ __launch_bounds__(kThreads, 2) void conv_gemm2_kernel(ConvParams p) {
  constexpr bool FAST = MODE != GEN;
  constexpr int BN = 64 * TN;
  constexpr int NB = 2 * TN;                 // right-operand pieces per thread per slab
  constexpr int kRow = BK2 + 8;              // 144-byte rows: 16-byte reads, rows 4 banks apart
  constexpr int kA = BM * kRow, kB = BN * kRow;
  constexpr int kOutPitch = BN + 4;          // fp32 staging of the output tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* lds = reinterpret_cast<bf16_t*>(smem);
  int* tab = reinterpret_cast<int*>(smem + (size_t)2 * (kA + kB) * sizeof(bf16_t));
  auto sA = [&](int s) { return lds + s * (kA + kB); };
  auto sB = [&](int s) { return lds + s * (kA + kB) + kA; };

  __shared__ int outrow[BM];   // PHASED: output row of every tile row (-1: none)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_n = (p.N + BN - 1) / BN;
  const int tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x % tiles_n;
  const int col0 = tile_n * BN;
  const int wrow = (wave >> 1) * 64, wcol = (wave & 1) * 32 * TN;
  const ConvGeom g = p.g;
  const int kc = tid & 7, rbase = tid >> 3;   // piece within a slab; rows rbase + 32*i

  // PHASED: this tile's parity class, its rows within the class, its live taps
  int row0 = tile_m * BM;
  int cls_size = 0, ph = 0, pw = 0, H2 = 1, W2 = 1;
  int u0 = 0, v0 = 0, nv = 1, nlive = 0;   // live taps: u = u0 + 2i, v = v0 + 2j, enumerated i-major
  if (MODE == PHASED) {
    H2 = g.Hp >> 1; W2 = g.Wp >> 1;
    cls_size = g.rows * H2 * W2;
    const int tiles_per_class = (cls_size + BM - 1) / BM;
    const int cls = tile_m / tiles_per_class;
    row0 = (tile_m - cls * tiles_per_class) * BM;   // first row within the class
    ph = cls >> 1; pw = cls & 1;
    u0 = (ph + g.pad) & 1; v0 = (pw + g.pad) & 1;
    const int nu = u0 < g.ks ? (g.ks - u0 + 1) >> 1 : 0;
    nv = v0 < g.ks ? (g.ks - v0 + 1) >> 1 : 0;
    nlive = nu * nv;
    if (nv == 0) nv = 1;
  }
  // t-th live tap -> filter tap (u, v) and source displacement (du, dv) in the half-resolution grid
  auto live_tap = [&](int t, int& u, int& v, int& du, int& dv) {
    const int i = t / nv, j = t - i * nv;
    u = u0 + 2 * i; v = v0 + 2 * j;
    du = (ph + g.pad - u) >> 1;   // arithmetic shift: -2 -> -1
    dv = (pw + g.pad - v) >> 1;
  };

  if (!FAST) build_tap_table(tab, g, tid);

  // ---- per-thread invariants of the left operand
  long rowbase[4];
  uint32_t tapmask[4];
  int an[4], ah[4], aw[4];
  uint32_t arow_ok = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = row0 + rbase + 32 * i;
    const bool ok = MODE == PHASED ? m < cls_size : m < p.M;
    arow_ok |= (ok ? 1u : 0u) << i;
    int n, h, w;
    if (MODE == PHASED) decode_pos2(H2 * W2, W2, ok ? m : 0, n, h, w);
    else decode_pos(g, ok ? m : 0, n, h, w);
    an[i] = n; ah[i] = h; aw[i] = w;
    rowbase[i] = 0;
    tapmask[i] = 0;
    if (MODE == PHASED) {
      // (h, w) are the half-resolution coordinates: the output position is (2h+ph, 2w+pw)
      rowbase[i] = (((long)n * g.Hs + h) * g.Ws + w) * g.Cs + kc * 8;
      for (int t = 0; t < nlive; ++t) {
        int u, v, du, dv;
        live_tap(t, u, v, du, dv);
        const int hs = h + du, ws = w + dv;
        const bool in = ok && hs >= 0 && hs < g.Hs && ws >= 0 && ws < g.Ws;
        tapmask[i] |= (in ? 1u : 0u) << t;
      }
    } else if (MODE == GEN) {
      // (unless the source is strided: then ah/aw stay the position and gather_offset divides)
      if (!(g.transposed && g.stride > 1)) {
        ah[i] = g.transposed ? h + g.pad : h * g.stride - g.pad;
        aw[i] = g.transposed ? w + g.pad : w * g.stride - g.pad;
        rowbase[i] = (((long)n * g.Hs + ah[i]) * g.Ws + aw[i]) * g.Cs;
      }
    } else if (FAST) {
      const int hb = g.transposed ? h + g.pad : h * g.stride - g.pad;
      const int wb = g.transposed ? w + g.pad : w * g.stride - g.pad;
      rowbase[i] = (((long)n * g.Hs + hb) * g.Ws + wb) * g.Cs + kc * 8;
      for (int u = 0; u < g.ks; ++u)
        for (int v = 0; v < g.ks; ++v) {
          const int hs = g.transposed ? hb - u : hb + u, ws = g.transposed ? wb - v : wb + v;
          const bool in = ok && hs >= 0 && hs < g.Hs && ws >= 0 && ws < g.Ws;
          tapmask[i] |= (in ? 1u : 0u) << (u * g.ks + v);
        }
    }
  }
  // ---- and of the right operand
  long brow[NB];
  uint32_t brow_ok = 0;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int r = col0 + rbase + 32 * i;
    brow[i] = (long)r * g.K + kc * 8;
    brow_ok |= (r < p.N ? 1u : 0u) << i;
  }
  if (MODE == PHASED && tid < BM) {
    const int m = row0 + tid;
    int n, h, w;
    decode_pos2(H2 * W2, W2, m < cls_size ? m : 0, n, h, w);
    outrow[tid] = m < cls_size ? (n * g.Hp + 2 * h + ph) * g.Wp + 2 * w + pw : -1;
  }
  if (!FAST || MODE == PHASED) __syncthreads();   // tap table / row map ready

  v16f acc[2][TN];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  u32x4 ra[4], rb[NB];
  // Loads of absent pieces (padding, ragged tile edges) are pointed at a page of zeros: one pointer
  // select instead of a select per loaded register, and the load itself stays unconditional.
  const bf16_t* const zp = static_cast<const bf16_t*>(g.zero);
  // FAST: (tap, channel base) of the slab advance uniformly
  int tap = 0, cb = 0;
  auto load_slab = [&](int k0, int tap_, int cb_) {
    if (FAST) {
      long tapoff;
      if (MODE == PHASED) {
        int u, v, du, dv;
        live_tap(tap_, u, v, du, dv);   // tap_ counts the live taps
        tapoff = ((long)du * g.Ws + dv) * g.Cs + cb_;
      } else {
        const int u = tap_ / g.ks, v = tap_ - u * g.ks;
        tapoff = (g.transposed ? -1L : 1L) * ((long)u * g.Ws + v) * g.Cs + cb_;
      }
      const bool kin = k0 < g.K;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = kin && ((tapmask[i] >> tap_) & 1u);
        ra[i] = *reinterpret_cast<const u32x4*>(in ? p.src + (rowbase[i] + tapoff) : zp);
      }
    } else {
      const int q = (k0 >> 3) + kc;
      const bool kin = q * 8 < g.K;
      const int t = tab[kin ? q : 0];
      const int u = t & 15, v = (t >> 4) & 15, ci = t >> 8;
      if (g.transposed && g.stride > 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const long o = gather_offset(g, an[i], ah[i], aw[i], u, v, ci);
          const bool in = kin && ((arow_ok >> i) & 1u) && o >= 0;
          ra[i] = *reinterpret_cast<const u32x4*>(in ? p.src + o : zp);
        }
      } else {
        // ah/aw hold the source coordinates of tap (0, 0); a tap is a displacement
        const int su = g.transposed ? -u : u, sv = g.transposed ? -v : v;
        const long tapoff = ((long)su * g.Ws + sv) * g.Cs + ci;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool in = kin && ((arow_ok >> i) & 1u) && (unsigned)(ah[i] + su) < (unsigned)g.Hs &&
                          (unsigned)(aw[i] + sv) < (unsigned)g.Ws;
          ra[i] = *reinterpret_cast<const u32x4*>(in ? p.src + (rowbase[i] + tapoff) : zp);
        }
      }
    }
    const bool bkin = k0 + kc * 8 < g.K;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const bool in = bkin && ((brow_ok >> i) & 1u);
      rb[i] = *reinterpret_cast<const u32x4*>(in ? p.wgt + (brow[i] + k0) : zp);
    }
  };
  auto store_a = [&](int s, int i) {
    *reinterpret_cast<u32x4*>(sA(s) + (rbase + 32 * i) * kRow + kc * 8) = ra[i];
  };
  auto store_b = [&](int s, int i) {
    *reinterpret_cast<u32x4*>(sB(s) + (rbase + 32 * i) * kRow + kc * 8) = rb[i];
  };
  auto advance = [&]() {
    cb += BK2;
    if (cb >= g.Cs) { cb = 0; ++tap; }
  };

  const int nslab = MODE == PHASED ? nlive * (g.Cs / BK2) : (g.K + BK2 - 1) / BK2;
  // first reduction element of a slab (the right operand's column); g.K = none
  auto slab_k0 = [&](int s_, int tap_, int cb_) {
    if (s_ >= nslab) return g.K;
    if (MODE != PHASED) return s_ * BK2;
    int u, v, du, dv;
    live_tap(tap_, u, v, du, dv);
    return (u * g.ks + v) * g.Cs + cb_;
  };
  load_slab(slab_k0(0, 0, 0), 0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) store_a(0, i);
#pragma unroll
  for (int i = 0; i < NB; ++i) store_b(0, i);
  __syncthreads();
  for (int s = 0; s < nslab; ++s) {
    const int cur = s & 1;
    if (FAST) advance();
    // always issued (past the end it re-reads element 0 and is dropped): a load
    // issued on one path only would make every later wait drain the queue
    load_slab(slab_k0(s + 1, tap, cb), s + 1 < nslab ? tap : 0, cb);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < BK2 / 16; ++ks) {
      bf16x8 fa[2], fb[TN];
      const int ko = ks * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int a = 0; a < 2; ++a)
        fa[a] = as_bf16x8(*reinterpret_cast<const u32x4*>(sA(cur) + (wrow + a * 32 + (lane & 31)) * kRow + ko));
#pragma unroll
      for (int b = 0; b < TN; ++b)
        fb[b] = as_bf16x8(*reinterpret_cast<const u32x4*>(sB(cur) + (wcol + b * 32 + (lane & 31)) * kRow + ko));
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    if (s + 1 < nslab) {
#pragma unroll
      for (int i = 0; i < 4; ++i) store_a(cur ^ 1, i);
#pragma unroll
      for (int i = 0; i < NB; ++i) store_b(cur ^ 1, i);
    }
    __syncthreads();
  }

  // ---- output tile -> LDS (fp32) -> 16-byte pieces.  Accumulator layout of a 32x32
  // block: register v of lane l holds row 8*(v/4) + 4*(l/32) + v%4, column l%32.
  float* so = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int jl = wcol + b * 32 + (lane & 31);
    const int j = col0 + jl;
    const float bj = (p.bias && j < p.N) ? p.bias[j] : 0.f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int il = wrow + a * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4);
        float val = acc[a][b][v] + bj;
        if (p.relu) val = val > 0.f ? val : 0.f;
        so[il * kOutPitch + jl] = val;
      }
  }
  __syncthreads();
  constexpr int kPiecesPerRow = BN / 8;
#pragma unroll
  for (int it = 0; it < BM * kPiecesPerRow / kThreads; ++it) {
    const int c = tid + kThreads * it;
    const int il = c / kPiecesPerRow, jl = (c % kPiecesPerRow) * 8;
    const int i = MODE == PHASED ? outrow[il] : row0 + il, j = col0 + jl;
    if (i < 0 || i >= p.M || j >= p.N) continue;   // N is a multiple of 8: a piece is wholly inside or outside
    float v[8];
    const v4f lo = *reinterpret_cast<const v4f*>(so + il * kOutPitch + jl);
    const v4f hi = *reinterpret_cast<const v4f*>(so + il * kOutPitch + jl + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
    const size_t idx = (size_t)i * p.N + j;
    if (p.addend) {
      float av[8];
      Piece<bf16_t>::load(p.addend + idx, av);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += av[e];
    }
    if (p.mask) {
      float mv[8];
      Piece<bf16_t>::load(p.mask + idx, mv);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = mv[e] > 0.f ? v[e] : 0.f;
    }
    if (p.accumulate) {
      float ov[8];
      Piece<bf16_t>::load(p.out + idx, ov);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += ov[e];
    }
    Piece<bf16_t>::store(p.out + idx, v);
  }
}

// ------------------------------------------------------------------ kernel D
// Forward and stride-1 dgrad of 3x3 / pad-1 convolutions with a channel count that
// is a multiple of 64 (most of a residual net).  Kernel A gathers the left operand
// once per filter tap: nine global loads, nine LDS stores of every input element.
// Here a workgroup owns 256 output positions (a strip of rows of one image, or a few
// whole small images) x 64 output channels:
//   * the input patch of those positions, halo included, is staged in LDS once per
//     64-channel slice ([patch position][64 channels], 144-byte rows);
//   * the left operand of tap (u, v) is that patch read at a row offset: no data
//     moves between taps, only the 8 KB weight slab of the tap streams through LDS
//     (double buffered, prefetched to registers);
//   * each wavefront owns 64 positions x 64 channels (2 x 2 accumulator blocks).
// For dgrad the gathered tensor is dY, the weights are the transposed copy and the
// taps are mirrored (dX(p) meets tap (u, v) at p + (1-u, 1-v)).
struct Conv3Params {
  const bf16_t* src;   // [rows][H][W][Cs]
  const bf16_t* wgt;   // [N][9][Cs]
  bf16_t* out;         // [rows*H*W][N]
  int rows, H, W, Cs, N;
  int R, nimg;         // a unit is nimg images x R rows; nimg * R * W = 256
  int units, upw;      // units in all, units per workgroup
  int flip;            // 1: dgrad (mirrored taps)
  const void* zero;    // page of zeros for absent pieces
  const float* bias;
  const bf16_t* mask;
  int relu, accumulate;
  bf16_t* pool;        // forward only, may be null: [rows*(H/2)*(W/2)][N], the 2 x 2 max pooling of `out`
  uint8_t* pool_code;  // with pool: one byte per pooled element, which of the four inputs the gradient goes to
  const bf16_t* addend;   // may be null: [rows*H*W][N] added to the product before the mask
};
constexpr int kUnitD = 256;

__device__ inline float as_stored(float v) { return bf16_to_f32(f32_to_bf16(v)); }
constexpr int kMaxPatchPieces = 13;   // 16-byte pieces of the patch per thread (up to 416 patch positions)

// A workgroup walks `upw` consecutive units of one channel tile: the next unit's patch
// and first weight slab travel to registers during the last taps of the current one,
// so only the first unit of a workgroup waits for memory before it can multiply.
// NB: 32-channel blocks of output per workgroup (2: a 64-channel tile; 1: layers with at most 32
// output channels, which would leave half of every fragment read and MFMA of the wide tile empty).
// KC: channels of the reduction staged at a time (64; 32 for layers with 32, 96, ... input channels, whose
// patch rows are then 80 bytes: sixteen lanes still cover all 64 banks).
// W8: maps 8 wide with units of whole groups of 8 map rows (see the fragment addresses below).
template <int NP, int NB, int KC, bool W8>   // NP: 16-byte patch pieces per thread
__global__ __launch_bounds__(kThreads, 2) void conv3_gemm_kernel(Conv3Params p) {
  constexpr int TN = 32 * NB;   // output channels per workgroup
  constexpr int OC = KC / 8;    // 16-byte pieces per patch position and per weight row
  constexpr int kRow = KC + 8;  // elements per LDS row
  constexpr int RP = kThreads / OC;               // weight rows staged per pass
  constexpr int WP = (TN + RP - 1) / RP;          // passes
  extern __shared__ __attribute__((aligned(16))) unsigned char smemD[];
  const int W = p.W, H = p.H, R = p.R;
  const int PW = W + 2, PR = R + 2;
  const int npatch = p.nimg * PR * PW;                    // patch positions
  bf16_t* sP = reinterpret_cast<bf16_t*>(smemD);          // [npatch][kRow]
  bf16_t* sW = sP + (size_t)npatch * kRow;                // 2 x [TN][kRow]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 31, h = lane >> 5;
  const int tiles_n = (p.N + TN - 1) / TN;
  const int group = blockIdx.x / tiles_n, tile_n = blockIdx.x - group * tiles_n;
  const int col0 = tile_n * TN;
  const int K = 9 * p.Cs;
  const int ubeg = group * p.upw, uend = min(p.units, ubeg + p.upw);

  // ---- patch staging tasks: piece x = tid + 256 t -> patch position x / OC, channel octet x % OC.
  // Relative to the unit's first image and row; which pieces exist depends on the unit.
  int prel[NP];                // element offset relative to the unit (the host checks the tensor has fewer than 2^31)
  uint32_t col_ok = 0, top = 0, bottom = 0;   // piece t: inside the image's columns / in the first / last patch row
  uint64_t img4 = 0;                           // piece t: image within the unit, 4 bits each
  const int npieces = npatch * OC;
#pragma unroll
  for (int t = 0; t < NP; ++t) {
    const int x = tid + t * kThreads;
    const int pp = min(x, npieces - 1) / OC, oct = x % OC;
    const int il = pp / (PR * PW), rem = pp - il * (PR * PW);
    const int pr = rem / PW, pc = rem - pr * PW;
    prel[t] = ((il * H + pr - 1) * W + pc - 1) * p.Cs + oct * 8;
    col_ok |= (x < npieces && pc >= 1 && pc <= W ? 1u : 0u) << t;
    top |= (pr == 0 ? 1u : 0u) << t;
    bottom |= (pr == PR - 1 ? 1u : 0u) << t;
    img4 |= (uint64_t)il << (4 * t);
  }
  // ---- weight staging: rows tid/OC (+ RP per pass) of the channel tile, octet tid % OC
  const int wr = tid / OC, woct = tid % OC;
  long woff[WP];
  uint32_t wvalid = 0;
#pragma unroll
  for (int i = 0; i < WP; ++i) {
    const int r = col0 + wr + RP * i;
    const bool in = r < p.N && wr + RP * i < TN;
    woff[i] = in ? (long)r * K + woct * 8 : 0;
    wvalid |= (in ? 1u : 0u) << i;
  }
  // ---- fragment addresses: this wavefront's positions wave*64 + a*32 + j
  // On maps 8 wide, sixteen consecutive lanes of a fragment read would cover two consecutive map
  // rows, whose patch rows (10 positions apart) share two of the sixteen bank groups (measured: 40 %
  // of this kernel's LDS cycles were conflicts there, against 15 % on wider maps).  Map rows 4 apart
  // are exactly complementary, so the wavefront takes the 8 map rows of its 64 positions in the order
  // 0 4 1 5 2 6 3 7; the epilogue puts every result back in its place.
  constexpr bool w8 = W8;
  auto row_order = [](int t) { return (t >> 1) + 4 * (t & 1); };   // t: 0..7
  int pbase[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    int pos = wave * 64 + a * 32 + j;
    if (w8) pos = wave * 64 + row_order(a * 4 + (j >> 3)) * 8 + (j & 7);
    const int rr = pos / W, w = pos - rr * W;
    const int il = rr / R, r = rr - il * R;
    pbase[a] = ((il * PR + r) * PW + w) * kRow + h * 8;   // patch origin is (-1, -1): tap (u, v) adds u*PW + v
  }
  const int bfrag = j * kRow + h * 8;

  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);   // absent pieces are read from a page of zeros
  u32x4 rp[NP], rw[WP];
  uint32_t pvalid = 0;
  // unit -> first image, first row, images present
  auto unit_geom = [&](int unit, int& n0, int& r0, int& nvalid) {
    if (p.nimg == 1) {
      const int upi = H / R, img = unit / upi;
      n0 = img; r0 = (unit - img * upi) * R; nvalid = 1;
    } else {
      n0 = unit * p.nimg; r0 = 0; nvalid = min(p.nimg, p.rows - n0);
    }
  };
  // loads are unconditional
  auto load_patch = [&](int unit, int cs) {
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const int ubase = (n0 * H + r0) * W * p.Cs + cs * KC;
    // the first / last patch row lies outside the image when the unit touches its top / bottom edge
    pvalid = col_ok & ~(r0 == 0 ? top : 0u) & ~(r0 + R == H ? bottom : 0u);
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const int il = (int)(img4 >> (4 * t)) & 15;
      if (il >= nvalid) pvalid &= ~(1u << t);
      rp[t] = *reinterpret_cast<const u32x4*>(((pvalid >> t) & 1u) ? p.src + (ubase + prel[t]) : zp);
    }
  };
  auto store_patch = [&]() {
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const int x = tid + t * kThreads;
      if (x < npieces)
        *reinterpret_cast<u32x4*>(sP + (x / OC) * kRow + (x % OC) * 8) = rp[t];
    }
  };
  auto load_w = [&](int k0) {
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      rw[i] = *reinterpret_cast<const u32x4*>(((wvalid >> i) & 1u) ? p.wgt + (woff[i] + k0) : zp);
    }
  };
  auto store_w = [&](int buf) {
#pragma unroll
    for (int i = 0; i < WP; ++i)
      if (wr + RP * i < TN)   // (a pass may cover more rows than the tile has)
        *reinterpret_cast<u32x4*>(sW + buf * TN * kRow + (wr + RP * i) * kRow + woct * 8) = rw[i];
  };

  const int nslice = p.Cs / KC;   // the patch is re-staged per KC-channel slice
  load_patch(min(ubeg, p.units - 1), 0);
  load_w(0);
  for (int unit = ubeg; unit < uend; ++unit) {
    // the unit's first patch slice and first weight slab are in registers
    store_patch();
    store_w(0);
    __syncthreads();
    v16f acc[2][NB];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    for (int cs = 0; cs < nslice; ++cs) {
      const bool last_slice = cs + 1 == nslice;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int cur = tap & 1 ? 1 - (cs & 1) : (cs & 1);   // step cs*9 + tap, odd/even (9 taps per slice)
        const int u = tap / 3, v = tap - u * 3;
        // next step's weights (always issued): next tap, next slice, or the next unit's first slab
        if (tap < 8) load_w((tap + 1) * p.Cs + cs * KC);
        else load_w(last_slice ? 0 : (cs + 1) * KC);
        // the next slice's patch (or the next unit's first) starts its way to registers a few taps early
        if (tap == 4) load_patch(last_slice ? min(unit + 1, uend - 1) : unit, last_slice ? 0 : cs + 1);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay here, a whole tap ahead of their use
        const int toff = (p.flip ? (2 - u) * PW + (2 - v) : u * PW + v) * kRow;
        const bf16_t* wb = sW + cur * TN * kRow + bfrag;
#pragma unroll
        for (int kk = 0; kk < KC / 16; ++kk) {
          bf16x8 fa[2], fb[NB];
#pragma unroll
          for (int a = 0; a < 2; ++a)
            fa[a] = as_bf16x8(*reinterpret_cast<const u32x4*>(sP + pbase[a] + toff + kk * 16));
#pragma unroll
          for (int b = 0; b < NB; ++b)
            fb[b] = as_bf16x8(*reinterpret_cast<const u32x4*>(wb + b * 32 * kRow + kk * 16));
#pragma unroll
          for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);   // nothing that touches the loaded registers moves above the MFMAs
        if (tap < 8 || !last_slice) store_w(cur ^ 1);
        __syncthreads();
        if (tap == 8 && !last_slice) {
          store_patch();       // every wavefront is past its last read of the old slice
          __syncthreads();
        }
      }
    }

    // ---- output tile -> LDS (fp32) -> 16-byte pieces (the staging area is free: the taps ended with a barrier)
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const long out_base = ((long)n0 * H + r0) * W;   // the unit's positions are contiguous rows of `out`
    const int npos = nvalid * R * W;                 // live positions of this unit
    constexpr int kOutPitch = TN + 4;
    float* so = reinterpret_cast<float*>(smemD);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int jl = b * 32 + j;
      const int c = col0 + jl;
      const float bj = (p.bias && c < p.N) ? p.bias[c] : 0.f;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          // accumulator register v of lane (j, h) is row 8 (v/4) + 4 h + v%4 of the block: map row a*4 + v/4 of the wavefront's eight
          const int il = wave * 64 + (w8 ? row_order(a * 4 + v / 4) * 8 : a * 32 + 8 * (v / 4)) + 4 * h + (v % 4);
          float val = acc[a][b][v] + bj;
          if (p.relu) val = val > 0.f ? val : 0.f;
          so[il * kOutPitch + jl] = val;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kUnitD * (TN / 8) / kThreads; ++it) {
      const int c = tid + kThreads * it;
      const int il = c / (TN / 8), jl = (c % (TN / 8)) * 8;
      const int jg = col0 + jl;
      if (il >= npos || jg >= p.N) continue;   // N is a multiple of 8: a piece is wholly inside or outside
      float v[8];
      const v4f lo = *reinterpret_cast<const v4f*>(so + il * kOutPitch + jl);
      const v4f hi = *reinterpret_cast<const v4f*>(so + il * kOutPitch + jl + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
      const size_t idx = (size_t)(out_base + il) * p.N + jg;
      if (p.addend) {
        float av[8];
        Piece<bf16_t>::load(p.addend + idx, av);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += av[e];
      }
      if (p.mask) {
        float mv[8];
        Piece<bf16_t>::load(p.mask + idx, mv);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = mv[e] > 0.f ? v[e] : 0.f;
      }
      if (p.accumulate) {
        float ov[8];
        Piece<bf16_t>::load(p.out + idx, ov);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += ov[e];
      }
      Piece<bf16_t>::store(p.out + idx, v);
    }
    if (p.pool) {
      // 2 x 2 max pooling of the unit straight from the staged tile (rounding to bf16 is monotonic:
      // the maximum of the rounded values is the rounded maximum).  A unit is whole rows of whole
      // images, so its pooled positions are a contiguous run of the pooled tensor too.
      const int Wh = W >> 1, Rh = R >> 1;
      const long pool_base = ((long)n0 * (H >> 1) + (r0 >> 1)) * Wh;
      const int npool = nvalid * Rh * Wh;
#pragma unroll
      for (int it = 0; it < (kUnitD / 4) * (TN / 8) / kThreads; ++it) {
        const int c = tid + kThreads * it;
        const int q = c / (TN / 8), jl = (c % (TN / 8)) * 8;
        const int jg = col0 + jl;
        if (q >= npool || jg >= p.N) continue;
        const int img = q / (Rh * Wh), rem = q - img * (Rh * Wh);
        const int pr = rem / Wh, pw = rem - pr * Wh;
        const float* s0 = so + ((img * R + 2 * pr) * W + 2 * pw) * kOutPitch + jl;
        float m[8];
        u32x2 code = {0u, 0u};
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const v4f a = *reinterpret_cast<const v4f*>(s0 + 4 * half);
          const v4f b = *reinterpret_cast<const v4f*>(s0 + kOutPitch + 4 * half);
          const v4f cc = *reinterpret_cast<const v4f*>(s0 + W * kOutPitch + 4 * half);
          const v4f d = *reinterpret_cast<const v4f*>(s0 + (W + 1) * kOutPitch + 4 * half);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            code[half] |= pool_code_of(as_stored(a[e]), as_stored(b[e]), as_stored(cc[e]), as_stored(d[e]),
                                       p.relu != 0, m[4 * half + e]) << (8 * e);
        }
        Piece<bf16_t>::store(p.pool + (size_t)(pool_base + q) * p.N + jg, m);
        *reinterpret_cast<u32x2*>(p.pool_code + (size_t)(pool_base + q) * p.N + jg) = code;
      }
    }
    __syncthreads();   // the staging area is about to be refilled
  }
}

// ------------------------------------------------------------------ kernel F
// Forward of the FIRST layer: 3x3 / pad 1 / stride 1 on 8 stored channels (3 real ones), at most
// 64 output channels.  The reduction is 9 taps x 8 channels = 72: one 16-byte piece per tap, so a
// k-step of 16 is two taps, and the lane halves of an MFMA operand simply read the patch at two
// different tap offsets.  All weights (at most 64 x 80 values) live in registers for the whole
// kernel; per unit of 256 positions the patch is 5 KB of LDS and the work is 10-20 MFMAs per
// wavefront: the kernel is bound by reading the input and writing the output once.
struct Conv1Params {
  const bf16_t* src;   // [rows][H][W][8]
  const bf16_t* wgt;   // [N][9][8]
  bf16_t* out;         // [rows*H*W][N]
  int rows, H, W, N;
  int R, nimg;         // a unit is nimg images x R rows; nimg * R * W = 256
  int units, upw;
  const float* bias;
  int relu;
  const void* zero;
  bf16_t* pool;        // may be null: [rows*(H/2)*(W/2)][N], the 2 x 2 max pooling of `out`
  uint8_t* pool_code;  // with pool: one byte per pooled element (see pool_code_of)
  int raw3;            // src is [rows][H][W][3]: a pixel is three 2-byte loads, channels 3-7 are zero
  int lw, lr;          // W = 1 << lw, R = 1 << lr
  uint32_t by_patch, by_pw, by_upi;   // reciprocal_below of PR PW, PW and H / R
};

// The copies of the other layers' weights ride in front of the units (CAST): they were 5 us as a launch of their own, most of it
// its start and end, and nothing reads them before the next launch (32-64-128 net on 32 x 32 images: 128 rows 88.3 -> 83.1 us,
// 1024 rows 209 -> 203 us; 11 M parameters: the same).  The layer's own weights then come from the parameters,
// and absent pieces are zeroed in registers: the zero page is cleared by this launch.
struct Conv1Casts {
  const float* w;      // this layer's weights [N][9][3]
  int blocks;          // workgroups that copy
  const float* params;
  bf16_t* shadow;
  uint32_t* zero_page;
  CastTable tab;
};
struct NoCasts {};

// The sums of a batch norm behind the layer (STAT): one record of every workgroup, whose units are all of one worker's images, in place of a
// launch that reads the output back.  In double, from the pieces that the lanes store.
// Step of the ResNet-18 shape in us, that launch / these sums: two workers, 64 images 1075 / 1071; four, 128 images 1334 / 1330; eight, 2048 images 10520 /
// 10501; two, 2048 images 10345 / 10328 (the launch took 7.8 us with 128 images and 53 with 2048).
struct Conv1Sums {
  double* partial;     // [workgroup][N][2]
  int K;
  // worker k has the workgroups gfirst[k] .. and the images ifirst[k] ..
  int32_t gfirst[OMNI_MAX_WORKERS + 1], ifirst[OMNI_MAX_WORKERS + 1];
};
struct NoSums {};

// Eight channels of a tap, of which three are real.  (Cleared by a mask: with a choice the compiler makes the loads conditional.)
__device__ __forceinline__ u32x4 weights3(const float* w, bool in) {
  const uint32_t mask = in ? ~0u : 0u;
  return u32x4{pack_bf16(w[0], w[1]) & mask, pack_bf16(w[2], 0.f) & mask, 0u, 0u};
}

template <int NBLK, bool CAST, bool STAT>   // NBLK: 32-channel blocks of output channels, 1 or 2
__global__ __launch_bounds__(kThreads, 2) void conv1_fwd_kernel(Conv1Params p, std::conditional_t<CAST, Conv1Casts, NoCasts> casts,
                                                                std::conditional_t<STAT, Conv1Sums, NoSums> sums) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smemF[];
  int block = (int)blockIdx.x;
  if constexpr (CAST) {
    if (block < casts.blocks) {
      cast_weights_body(casts.tab, casts.params, casts.shadow, casts.zero_page, block, reinterpret_cast<bf16_t*>(smemF));
      return;
    }
    block -= casts.blocks;
  }
  constexpr int NT = 32 * NBLK;
  constexpr int kPitch = NT + 8;   // bf16 elements per staged output row
  const int W = p.W, H = p.H, R = p.R;
  const int PW = W + 2, PR = R + 2;
  const int npatch = p.nimg * PR * PW;
  u32x4* sP = reinterpret_cast<u32x4*>(smemF);                                  // [npatch] pieces of 8 channels
  bf16_t* so = reinterpret_cast<bf16_t*>(smemF + (size_t)((npatch + 3) & ~3) * 16);   // [256][kPitch]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 31, h = lane >> 5;
  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);

  // ---- weights: B fragment of k-step ks = taps 2ks (lanes 0-31) and 2ks+1 (lanes 32-63) of channel j
  bf16x8 wf[NBLK][5];
#pragma unroll
  for (int b = 0; b < NBLK; ++b)
#pragma unroll
    for (int ks = 0; ks < 5; ++ks) {
      const int tap = 2 * ks + h, co = 32 * b + j;
      const bool in = tap < 9 && co < p.N;
      if constexpr (CAST) wf[b][ks] = as_bf16x8(weights3(casts.w + (in ? (co * 9 + tap) * 3 : 0), in));
      else wf[b][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(in ? p.wgt + ((size_t)co * 9 + tap) * 8 : zp));
    }
  float bj[NBLK];
#pragma unroll
  for (int b = 0; b < NBLK; ++b) bj[b] = (p.bias && 32 * b + j < p.N) ? p.bias[32 * b + j] : 0.f;

  // ---- patch staging: piece x = tid + 256 t is patch position x (two per thread)
  int prel[2], pil[2], ppr[2];
  bool pcol[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int x = min(tid + t * kThreads, npatch - 1);
    const int il = (int)__umulhi((uint32_t)x, p.by_patch), rem = x - il * (PR * PW);
    const int pr = (int)__umulhi((uint32_t)rem, p.by_pw), pc = rem - pr * PW;
    pil[t] = il; ppr[t] = pr;
    pcol[t] = tid + t * kThreads < npatch && pc >= 1 && pc <= W;
    prel[t] = ((il * H + pr - 1) * W + pc - 1) * (p.raw3 ? 3 : 8);
  }
  // ---- fragment addresses: positions wave*64 + a*32 + j, tap offset by lane half
  int pbase[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int pos = wave * 64 + a * 32 + j;
    const int rr = pos >> p.lw, w = pos & (W - 1);
    const int il = rr >> p.lr, r = rr & (R - 1);
    pbase[a] = (il * PR + r) * PW + w;
  }
  int toff[5];
#pragma unroll
  for (int ks = 0; ks < 5; ++ks) {
    const int tap = min(2 * ks + h, 8);   // the tenth "tap" does not exist: its weights are zero, its data are zeroed below
    toff[ks] = (tap / 3) * PW + tap % 3;
  }

  auto unit_geom = [&](int unit, int& n0, int& r0, int& nvalid) {
    if (p.nimg == 1) {
      const int upi = H >> p.lr;
      const int img = quotient(unit, p.by_upi, upi);
      n0 = img; r0 = (unit - img * upi) * R; nvalid = 1;
    } else {
      n0 = unit * p.nimg; r0 = 0; nvalid = min(p.nimg, p.rows - n0);
    }
  };
  u32x4 rp[2];
  auto load_patch = [&](int unit) {
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const long ubase = ((long)n0 * H + r0) * W * (p.raw3 ? 3 : 8);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = r0 + ppr[t] - 1;
      const bool in = pcol[t] && pil[t] < nvalid && row >= 0 && row < H;
      const bf16_t* q = in ? p.src + (ubase + prel[t]) : CAST ? p.src : zp;
      if (p.raw3) rp[t] = u32x4{(uint32_t)q[0] | ((uint32_t)q[1] << 16), (uint32_t)q[2], 0u, 0u};
      else rp[t] = *reinterpret_cast<const u32x4*>(q);
      if (CAST && !in) rp[t] = u32x4{0u, 0u, 0u, 0u};
    }
  };

  int ubeg = block * p.upw, uend = min(p.units, ubeg + p.upw);
  if constexpr (STAT) {
    const int g = sums.gfirst[lane], i = sums.ifirst[lane];   // (65 entries, all lanes at once)
    const int k = __popcll(__ballot(lane < sums.K && g <= block)) - 1, upi = H >> p.lr;
    const int after = k + 1 < sums.K ? __builtin_amdgcn_readlane(i, k + 1) : p.rows;
    ubeg = __builtin_amdgcn_readlane(i, k) * upi + (block - __builtin_amdgcn_readlane(g, k)) * p.upw;
    uend = min(after * upi, ubeg + p.upw);
  }
  double t[2][8] = {};   // STAT: this lane's sums of eight channels
  load_patch(min(ubeg, p.units - 1));
  for (int unit = ubeg; unit < uend; ++unit) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      if (tid + t * kThreads < npatch) sP[tid + t * kThreads] = rp[t];
    __syncthreads();
    load_patch(min(unit + 1, uend - 1));
    __builtin_amdgcn_sched_barrier(0);

    v16f acc[2][NBLK];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 5; ++ks) {
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        u32x4 q = sP[pbase[a] + toff[ks]];
        if (ks == 4 && h == 1) q = u32x4{0u, 0u, 0u, 0u};
        const bf16x8 fa = as_bf16x8(q);
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, wf[b][ks], acc[a][b], 0, 0, 0);
      }
    }
    // bias, ReLU, round to bf16, stage so that rows leave as 16-byte pieces
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int il = wave * 64 + a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
          float val = acc[a][b][v] + bj[b];
          if (p.relu) val = val > 0.f ? val : 0.f;
          so[il * kPitch + 32 * b + j] = f32_to_bf16(val);
        }
    __syncthreads();
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const long out_base = ((long)n0 * H + r0) * W;
    const int npos = nvalid * R * W;
    constexpr int kPieces = NT / 8;
#pragma unroll
    for (int it = 0; it < kUnitD * kPieces / kThreads; ++it) {
      const int c = tid + kThreads * it;
      const int il = c / kPieces, jl = (c % kPieces) * 8;
      if (il < npos && jl < p.N) {   // N is a multiple of 8
        const u32x4 piece = *reinterpret_cast<const u32x4*>(so + il * kPitch + jl);
        *reinterpret_cast<u32x4*>(p.out + (size_t)(out_base + il) * p.N + jl) = piece;
        if constexpr (STAT) bn_sums_add(t, piece);
      }
    }
    if (!STAT && p.pool) {
      // 2 x 2 max pooling of the unit from the staged rows (a unit is whole rows of whole images: its
      // pooled positions are a contiguous run of the pooled tensor)
      const int Wh = W >> 1, Rh = R >> 1;
      const long pool_base = ((long)n0 * (H >> 1) + (r0 >> 1)) * Wh;
      const int npool = nvalid * Rh * Wh;
#pragma unroll
      for (int it = 0; it < ((kUnitD / 4) * kPieces + kThreads - 1) / kThreads; ++it) {
        const int c = tid + kThreads * it;
        const int q = c / kPieces, jl = (c % kPieces) * 8;
        if (q >= npool || jl >= p.N) continue;
        const int pw = q & (Wh - 1), ir = q >> (p.lw - 1);   // (an image's rows follow the image's before, halved as they are)
        const bf16_t* s0 = so + (2 * ir * W + 2 * pw) * kPitch + jl;
        float a[8], b[8], cc[8], d[8], m[8];
        Piece<bf16_t>::load(s0, a);
        Piece<bf16_t>::load(s0 + kPitch, b);
        Piece<bf16_t>::load(s0 + W * kPitch, cc);
        Piece<bf16_t>::load(s0 + (W + 1) * kPitch, d);
        u32x2 code = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          code[e >> 2] |= pool_code_of(a[e], b[e], cc[e], d[e], p.relu != 0, m[e]) << (8 * (e & 3));
        Piece<bf16_t>::store(p.pool + (size_t)(pool_base + q) * p.N + jl, m);
        *reinterpret_cast<u32x2*>(p.pool_code + (size_t)(pool_base + q) * p.N + jl) = code;
      }
    }
    // (the next iteration's patch store touches sP only; `so` is rewritten after the next barrier)
  }
  if constexpr (STAT) {
    // the position lanes' sums of a channel, eight at a time, then the parts: a fixed order
    constexpr int kPieces = NT / 8, kLanes = kThreads / kPieces, kParts = kThreads / NT;
    double (*const rows)[kPieces][9] = reinterpret_cast<double (*)[kPieces][9]>(so);   // [kLanes]
    double (*const part_sum)[NT] = reinterpret_cast<double (*)[NT]>(so + sizeof(double) / sizeof(bf16_t) * kLanes * kPieces * 9);
    static_assert((kLanes * kPieces * 9 + kParts * NT) * sizeof(double) <= (size_t)kUnitD * kPitch * sizeof(bf16_t), "they take the staged output's place");
    static_assert(kLanes / kParts == 8, "eight lanes to a part");
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 8; ++e) rows[tid / kPieces][tid % kPieces][e] = t[which][e];
      __syncthreads();
      const int c = tid % NT, part = tid / NT;
      double sum = 0.0;
#pragma unroll
      for (int r = 0; r < 8; ++r) sum += rows[part * 8 + r][c >> 3][c & 7];
      part_sum[part][c] = sum;
      __syncthreads();
      if (tid < p.N) {
        sum = part_sum[0][tid];
#pragma unroll
        for (int q = 1; q < kParts; ++q) sum += part_sum[q][tid];
        sums.partial[((size_t)block * p.N + tid) * 2 + which] = sum;
      }
    }
  }
}

}  // namespace

template <int TN, int MODE>
static void launch_gemm2(hipStream_t st, const ConvParams& p, int tiles) {
  constexpr int BN = 64 * TN;
  constexpr size_t kBytes =
      (size_t)2 * (BM + BN) * (BK2 + 8) * sizeof(bf16_t) + (MODE != GEN ? 0 : kMaxPieces * sizeof(int));
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&conv_gemm2_kernel<TN, MODE>), kBytes);
  hipLaunchKernelGGL((conv_gemm2_kernel<TN, MODE>), dim3(tiles), dim3(kThreads), kBytes, st, p);
}

// 3x3 / pad 1 / stride 1 (forward, or dgrad of such a layer) with channels a multiple of 32 and a
// map whose rows tile into units of 256 positions: kernel D.  Returns false if the shape does not qualify.
static bool conv3_gemm(hipStream_t st, const bf16_t* src, const bf16_t* wgt, bf16_t* out, int M, int N,
                       const ConvGeom& g, const float* bias, const bf16_t* mask, bool relu, bool accumulate,
                       bf16_t* pool, uint8_t* pool_code, bool* pooled, const bf16_t* addend) {
  const int H = g.Hs, W = g.Ws;
  if (g.raw3 || g.ks != 3 || g.stride != 1 || g.pad != 1 || g.Hp != H || g.Wp != W) return false;
  if (g.Cs % 32 != 0 || N % 8 != 0 || (long)g.rows * H * W != M) return false;
  if ((long)M * g.Cs >= (1L << 31)) return false;   // 32-bit element offsets in the kernel
  if (W < 4 || W > kUnitD || kUnitD % W != 0) return false;
  const int R = std::min(H, kUnitD / W);
  if (H % R != 0 || kUnitD % (R * W) != 0) return false;
  const int nimg = kUnitD / (R * W);
  if (nimg > 1 && R != H) return false;
  const int npatch = nimg * (R + 2) * (W + 2);
  // channels of the reduction staged at a time: 64 where the patch of a unit then fits the registers
  // that carry it to LDS (on 4 x 4 maps a unit is 16 images and their halos are most of the patch)
  const int kc = (g.Cs % 64 == 0 && npatch * 8 <= kMaxPatchPieces * kThreads) ? 64 : 32;
  const int oc = kc / 8;
  if (npatch * oc > kMaxPatchPieces * kThreads) return false;
  Conv3Params p{};
  p.src = src; p.wgt = wgt; p.out = out; p.rows = g.rows; p.H = H; p.W = W; p.Cs = g.Cs; p.N = N;
  p.R = R; p.nimg = nimg; p.flip = g.transposed ? 1 : 0; p.zero = g.zero;
  p.bias = bias; p.mask = mask; p.relu = relu ? 1 : 0; p.accumulate = accumulate ? 1 : 0;
  // the pooled copy is written from the same staged tile when a unit holds whole 2 x 2 windows
  p.pool = (pool && pool_code && !mask && !accumulate && !g.transposed && H % 2 == 0 && W % 2 == 0 && R % 2 == 0)
               ? pool : nullptr;
  p.pool_code = pool_code;
  p.addend = addend;
  *pooled = p.pool != nullptr;
  const int nb = N <= 32 ? 1 : 2;                 // a 32-channel tile for layers with at most 32 output channels
  const int tn = 32 * nb;
  const size_t stage = ((size_t)npatch + 2 * tn) * (kc + 8) * sizeof(bf16_t);
  const size_t outt = (size_t)kUnitD * (tn + 4) * sizeof(float);
  const size_t lds = std::max(stage, outt);
  if (lds > 80 * 1024) return false;
  const int big = npatch * oc > 11 * kThreads ? 1 : 0;
  const int units = nimg == 1 ? g.rows * (H / R) : (g.rows + nimg - 1) / nimg;
  const int tiles_n = (N + tn - 1) / tn;
  // several units per workgroup once there are enough workgroups to fill the chip a few times over
  int upw = 1;
  while (upw < 4 && (long)units * tiles_n / (upw * 2) >= 2048) upw *= 2;
  p.units = units; p.upw = upw;
  const dim3 grid(((units + upw - 1) / upw) * tiles_n);
  const bool w8 = W == 8 && R % 8 == 0;
#define OMNI_CONV3(NP_, NB_, KC_, W8_)                                                                \
  {                                                                                                   \
    static LdsLimit limit;                                                                            \
    limit.raise(reinterpret_cast<const void*>(&conv3_gemm_kernel<NP_, NB_, KC_, W8_>), 80 * 1024);    \
    hipLaunchKernelGGL((conv3_gemm_kernel<NP_, NB_, KC_, W8_>), grid, dim3(kThreads), lds, st, p);    \
  }
#define OMNI_CONV3_W8(NP_, NB_, KC_) { if (w8) OMNI_CONV3(NP_, NB_, KC_, true) else OMNI_CONV3(NP_, NB_, KC_, false) }
#define OMNI_CONV3_KC(NP_, NB_) { if (kc == 64) OMNI_CONV3_W8(NP_, NB_, 64) else OMNI_CONV3_W8(NP_, NB_, 32) }
  if (nb == 1) { if (big) OMNI_CONV3_KC(13, 1) else OMNI_CONV3_KC(11, 1) }
  else
  { if (big) OMNI_CONV3_KC(13, 2) else OMNI_CONV3_KC(11, 2) }
#undef OMNI_CONV3_KC
#undef OMNI_CONV3_W8
#undef OMNI_CONV3
  return true;
}

// First layer forward (8 stored channels, 3x3 / pad 1 / stride 1, at most 64 outputs): kernel F.
static bool conv1_fwd_shape(int N, const ConvGeom& g, long M) {
  const int H = g.Hs, W = g.Ws;
  if (g.transposed || g.Cs != 8 || g.ks != 3 || g.stride != 1 || g.pad != 1) return false;
  if (g.Hp != H || g.Wp != W || N % 8 != 0 || N > 64 || (long)g.rows * H * W != M) return false;
  if (W < 8 || W > kUnitD || kUnitD % W != 0) return false;
  const int R = std::min(H, kUnitD / W);
  if (H % R != 0 || kUnitD % (R * W) != 0) return false;
  const int nimg = kUnitD / (R * W);
  if (nimg > 1 && R != H) return false;
  return nimg * (R + 2) * (W + 2) <= 2 * kThreads;
}

static bool conv1_fwd(hipStream_t st, const bf16_t* src, const bf16_t* wgt, bf16_t* out, int M, int N,
                      const ConvGeom& g, const float* bias, const bf16_t* mask, bool relu, bool accumulate,
                      bf16_t* pool, uint8_t* pool_code, bool* pooled, BnStatRequest* stats, const Conv1Casts* casts = nullptr) {
  const int H = g.Hs, W = g.Ws;
  if (mask || accumulate || !conv1_fwd_shape(N, g, M)) return false;
  const int R = std::min(H, kUnitD / W);
  const int nimg = kUnitD / (R * W);
  const int npatch = nimg * (R + 2) * (W + 2);
  Conv1Params p{};
  p.raw3 = g.raw3;
  p.src = src; p.wgt = wgt; p.out = out; p.rows = g.rows; p.H = H; p.W = W; p.N = N; p.R = R; p.nimg = nimg;
  p.bias = bias; p.relu = relu ? 1 : 0; p.zero = g.zero;
  p.pool = (pool && pool_code && H % 2 == 0 && W % 2 == 0 && R % 2 == 0) ? pool : nullptr;
  p.pool_code = pool_code;
  *pooled = p.pool != nullptr;
  p.units = nimg == 1 ? g.rows * (H / R) : (g.rows + nimg - 1) / nimg;
  p.lw = __builtin_ctz(W); p.lr = __builtin_ctz(R);   // (both divide 256)
  p.by_patch = reciprocal_below((R + 2) * (W + 2), 2 * kThreads);
  p.by_pw = reciprocal_below(W + 2, 2 * kThreads);
  p.by_upi = reciprocal_below(H / R, p.units);
  p.upw = 1;
  while (p.upw < 8 && p.units / (p.upw * 2) >= 1024) p.upw *= 2;
  const int nblk = N > 32 ? 2 : 1;
  const size_t lds = (size_t)((npatch + 3) & ~3) * 16 + (size_t)kUnitD * (32 * nblk + 8) * sizeof(bf16_t);
  static_assert(kUnitD * 40 >= kCastTile * kCastStride, "a copied tile fits the staged output");
  int groups = (p.units + p.upw - 1) / p.upw;
  Conv1Sums sums{};
  if (stats && stats->partial && stats->seg && !stats->x && stats->seg->off[stats->seg->K] == g.rows && !bias && !relu && !p.pool && nimg == 1) {
    const Segments& seg = *stats->seg;
    const int upi = H / R;
    auto groups_of = [&](int k, int u) { return ((long)(seg.off[k + 1] - seg.off[k]) * upi + u - 1) / u; };
    auto groups_at = [&](int u) {
      long n = 0;
      for (int k = 0; k < seg.K; ++k) n += groups_of(k, u);
      return n;
    };
    // more units to a workgroup where there is no room for the records, but no fewer than two workgroups per compute unit (one worker, 600
    // images, 150 workgroups: step 4131 -> 4160 us; 2048 images, 256: 10352 -> 10501)
    int u = p.upw;
    while (groups_at(u) > (long)seg.K * kBnMaxSplits && u < 64) u *= 2;
    if (groups_at(u) <= (long)seg.K * kBnMaxSplits && (u == p.upw || groups_at(u) >= 512)) {
      p.upw = u;
      sums.partial = stats->partial;
      sums.K = seg.K;
      for (int k = 0; k <= seg.K; ++k) {
        sums.ifirst[k] = seg.off[k];
        if (k < seg.K) sums.gfirst[k + 1] = sums.gfirst[k] + (int)groups_of(k, u);
        stats->table.first[k] = sums.gfirst[k];
      }
      groups = sums.gfirst[seg.K];
      stats->done = true;
    }
  }
  const dim3 grid(groups + (casts ? casts->blocks : 0)), block(kThreads);
#define OMNI_CONV1_(NBLK_, CAST_, ARG_)                                                                                                \
  {                                                                                                                                    \
    if (sums.partial) hipLaunchKernelGGL((conv1_fwd_kernel<NBLK_, CAST_, true>), grid, block, lds, st, p, ARG_, sums);                 \
    else hipLaunchKernelGGL((conv1_fwd_kernel<NBLK_, CAST_, false>), grid, block, lds, st, p, ARG_, NoSums{});                         \
  }
#define OMNI_CONV1(NBLK_) { if (casts) OMNI_CONV1_(NBLK_, true, *casts) else OMNI_CONV1_(NBLK_, false, NoCasts{}) }
  if (nblk == 2) OMNI_CONV1(2) else OMNI_CONV1(1)
#undef OMNI_CONV1
#undef OMNI_CONV1_
  return true;
}

// (Three channels, as images have: every lane fetches its weights a row apart, and more of them cost more than the copies' launch:
// 370 images of 32 x 32 x 8 to 64 channels 65.4 us against 23.3 and 4.9, 423 of 32 x 32 x 8 to 32 36.9 against 15.6 and 5.5.)
bool conv_first_layer_takes_casts(int Cout, int cin_real, const ConvGeom& g, long M) {
  return cin_real == 3 && conv1_fwd_shape(Cout, g, M);
}

bool conv_first_layer_and_casts(hipStream_t st, const bf16_t* src, const float* params, size_t w_off, bf16_t* shadow,
                                const CastEntry* entries, int n, uint32_t* zero_page, bf16_t* out, int M, int N,
                                const ConvGeom& g, const float* bias, bool relu, bf16_t* pool, uint8_t* pool_code, BnStatRequest* stats) {
  Conv1Casts c{};
  c.w = params + w_off; c.params = params; c.shadow = shadow; c.zero_page = zero_page;
  c.blocks = cast_table(c.tab, entries, n);
  bool pooled = false;
  conv1_fwd(st, src, nullptr, out, M, N, g, bias, nullptr, relu, false, pool, pool_code, &pooled, stats, &c);
  return pooled;
}

bool conv_first_layer_raw_supported(int Cout, int cin_real, const ConvGeom& g, long M) {
  return cin_real == 3 && conv1_fwd_shape(Cout, g, M) && conv_wgrad_pooled_supported(Cout, cin_real, g);
}

bool conv_gemm_bf16(hipStream_t st, const bf16_t* src, const bf16_t* wgt, bf16_t* out, int M, int N,
                    const ConvGeom& g, const float* bias, const bf16_t* mask, bool relu, bool accumulate,
                    bf16_t* pool_out, uint8_t* pool_code, const bf16_t* addend, BnStatRequest* stats,
                    UnpoolRequest* unpool) {
  bool pooled = false;
  if (g.frag == 1)
    return conv_frag_bf16(st, src, wgt, out, N, g, bias, mask, relu, accumulate, pool_out, pool_code, addend, stats, unpool);
  if (g.frag == 3) {
    conv_gather_bf16(st, src, wgt, out, N, g, bias, relu, stats);
    return false;
  }
  // 3x3 / stride 1 / pad 1: the wide-tile kernel where the shape and the amount of work allow it, else the 256-position one
  if (conv3_wide_bf16(st, src, wgt, out, M, N, g, bias, mask, relu, accumulate, addend, pool_out, pool_code, stats, unpool))
    return pool_out && pool_code;
  if (conv3_gemm(st, src, wgt, out, M, N, g, bias, mask, relu, accumulate, pool_out, pool_code, &pooled, addend))
    return pooled;
  if (!addend && conv1_fwd(st, src, wgt, out, M, N, g, bias, mask, relu, accumulate, pool_out, pool_code, &pooled, stats))
    return pooled;
  if (g.raw3) return false;   // (callers ask conv_first_layer_raw_supported first: nothing else reads a 3-channel source)
  ConvParams p{};
  p.src = src; p.wgt = wgt; p.out = out; p.M = M; p.N = N; p.g = g;
  p.bias = bias; p.mask = mask; p.relu = relu ? 1 : 0; p.accumulate = accumulate ? 1 : 0;
  p.addend = addend;
  int tiles_m = (M + BM - 1) / BM;
  const bool chan_ok = g.Cs % BK2 == 0 && g.ks <= 3;
  const bool fast = chan_ok && (!g.transposed || g.stride == 1);
  // dgrad of a stride-2 convolution: the gathered tensor is the half-resolution output gradient
  const bool phased = chan_ok && g.transposed && g.stride == 2 && g.Hp % 2 == 0 && g.Wp % 2 == 0 &&
                      g.Hs == g.Hp / 2 && g.Ws == g.Wp / 2 && (long)g.rows * g.Hp * g.Wp == M;
  if (phased) {
    const long cls = (long)g.rows * (g.Hp / 2) * (g.Wp / 2);
    tiles_m = 4 * (int)((cls + BM - 1) / BM);   // every parity class is padded to whole tiles
  }
  const int mode = phased ? PHASED : fast ? FASTM : GEN;
  const int tiles = tiles_m * (N > 64 ? (N + 127) / 128 : (N + 63) / 64);
#define OMNI_GEMM2(TN)                                           \
  {                                                              \
    if (mode == PHASED) launch_gemm2<TN, PHASED>(st, p, tiles);  \
    else if (mode == FASTM) launch_gemm2<TN, FASTM>(st, p, tiles); \
    else launch_gemm2<TN, GEN>(st, p, tiles);                    \
  }
  if (N > 64) OMNI_GEMM2(2) else OMNI_GEMM2(1)
#undef OMNI_GEMM2
  return false;
}

}  // namespace omni
