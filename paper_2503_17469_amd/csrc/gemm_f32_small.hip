// fp32 products of fully connected layers that are too small, or too oddly shaped, for 64 x 64 LDS tiles
// (v_mfma_f32_16x16x4_f32).
//
// The contractions are those of gemm_f32.hip (the gradient line of Algorithm 1, procedure Train):
//   forward   Y  = X W^T + bias, optional ReLU
//   dgrad     dX = dY W, optional ReLU mask, optional accumulate
//   wgrad     G_k = dY_k^T X_k for every worker, all layers in one launch, with the losses of the head and, where
//             the step applies it, the SGD update of the very parameters a workgroup has just finished
//
// What bounds them is latency: a few MFLOP per layer, so a product costs its launch, the first loads, a chain of
// steps and the drain.  Therefore
//   * a wavefront fetches its own operands, several chunks ahead, in whole 128-byte lines, and turns them into the
//     instruction's layout through LDS of its own (weight gradients need no turning): no barrier in the main loop;
//   * the output is cut into 16 x 16 or 32 x 32 tiles, so that a few hundred rows already give hundreds of tiles, and
//     the reduction of a tile is split over the four wavefronts of its workgroup and added up in wavefront order
//     through LDS at the end (a split over workgroups needs a second pass through memory and a device-wide release);
//   * rows may start at any multiple of 4 bytes (16-byte loads need no more), and a piece that would run past the end of
//     a row is moved back to end there, so odd widths take the same instructions as even ones.
// All sums have a fixed order: results repeat bit for bit.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"
#include "head_device.h"
#include "kernels.h"
#include "quotient.h"
#include "update_device.h"
#include "xcd_tiles.h"

namespace omni {

namespace {

template <int N> struct Vec;
template <> struct Vec<2> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Vec<4> { typedef v4f_a4 type; };

template <int N>
__device__ inline void load_n(const float* p, float (&v)[N]) {
  if constexpr (N == 1) {
    v[0] = *p;
  } else {
    const typename Vec<N>::type t = *reinterpret_cast<const typename Vec<N>::type*>(p);
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = t[e];
  }
}
template <int N>
__device__ inline void store_n(float* p, const float (&v)[N]) {
  if constexpr (N == 1) {
    *p = v[0];
  } else {
    typename Vec<N>::type t;
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = v[e];
    *reinterpret_cast<typename Vec<N>::type*>(p) = t;
  }
}

constexpr int kChunk = 32;   // reduction elements of a forward / dgrad step
constexpr long kSmallMaxTiles64 = 256;   // products with fewer 64 x 64 tiles come here

struct SmallGemm {
  const float* A;      // [M][K], reduction index contiguous
  const float* B;      // forward: [N][K]; dgrad: [K][N]
  float* C;            // [M][N]
  int M, N, K;
  const float* bias;   // forward, may be null
  const float* mask;   // dgrad, [M][N], may be null
  int relu, accumulate;
  XcdTiles tiles;
};

// A k-contiguous operand of a chunk, 16 WB rows of 128 bytes, arrives with 8 lanes per row (whole lines per group of
// consecutive lanes: with one lane per row, the layout the instruction wants, the vector cache takes one access per
// lane and delivers 16 bytes per clock; measured, 4 times slower) and turns into the instruction's layout through a
// wavefront-private LDS block with 36-float rows (conflict-free both ways; LDS operations of a wavefront complete in
// order, so no barrier).
constexpr int kRowFloats = 36;
template <int WB> struct SmallLine { v4f v[2 * WB]; };      // as loaded: rows lane / 8 + 8 i, elements 4 (lane % 8) ..
template <int WB> struct SmallFrag { v4f v[WB][2]; };       // as multiplied: element 16 s + 4 g + q of row r of block i
template <int WB> struct SmallCols { float v[2][4][WB]; };  // dgrad's B: columns WB r .. of reduction row 16 s + 4 g + q

// (addresses are a uniform base plus a lane offset that never changes: no vector instruction per load)
template <int WB>
__device__ __forceinline__ void line_load(SmallLine<WB>& l, const float* base, const uint32_t (&off)[2 * WB]) {
#pragma unroll
  for (int i = 0; i < 2 * WB; ++i) l.v[i] = *reinterpret_cast<const v4f_a4*>(base + off[i]);
}
template <int WB>
__device__ __forceinline__ void line_store(const SmallLine<WB>& l, float* lds, int lane) {
#pragma unroll
  for (int i = 0; i < 2 * WB; ++i)
    *reinterpret_cast<v4f*>(lds + ((lane >> 3) + 8 * i) * kRowFloats + (lane & 7) * 4) = l.v[i];
}
template <int WB>
__device__ __forceinline__ void frag_load(SmallFrag<WB>& f, const float* lds, int r, int g) {
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      f.v[i][s] = *reinterpret_cast<const v4f*>(lds + (16 * i + r) * kRowFloats + 16 * s + 4 * g);
}
template <int WB>
__device__ __forceinline__ void cols_load(SmallCols<WB>& c, const float* base, uint32_t off, int N) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) load_n<WB>(base + (size_t)(16 * s + q) * N + off, c.v[s][q]);
}
// reduction elements below `lo` count zero (the last chunk of a row is moved back to end at K: what the chunk before
// it covers is not counted again), in both operands: 0 * infinity is no zero
template <int WB>
__device__ __forceinline__ void frag_clear_below(SmallFrag<WB>& f, int lo, int g) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < WB; ++i) f.v[i][s][q] = 16 * s + 4 * g + q < lo ? 0.f : f.v[i][s][q];
}

template <int WB>
__device__ __forceinline__ void cols_clear_below(SmallCols<WB>& c, int lo, int g) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < WB; ++j) c.v[s][q][j] = 16 * s + 4 * g + q < lo ? 0.f : c.v[s][q][j];
}

template <bool DGRAD, int WB, int NW>
constexpr int small_gemm_floats() { return NW * (DGRAD ? 1 : 2) * 16 * WB * kRowFloats; }

template <bool DGRAD, int WB, int NW>
__device__ __forceinline__ void small_gemm_body(const SmallGemm& p, int block, float* lds) {
  constexpr int T = 16 * WB, D = 2;                        // D chunks on their way from memory
  constexpr int kWave = (DGRAD ? 1 : 2) * T * kRowFloats;  // floats of a wavefront's LDS block (at least its partial tile)
  static_assert(kWave >= T * T, "the partial tile reuses the staging block");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  int tile_m, tile_n;
  if (!xcd_tile(p.tiles, block, tile_m, tile_n)) return;
  const int row0 = tile_m * T, col0 = tile_n * T;
  const int M = p.M, N = p.N, K = p.K;
  float* la = lds + wave * kWave;
  float* lb = la + T * kRowFloats;

  // rows and columns past the end shadow the last ones; their results are not stored
  const float* a0 = p.A + (size_t)row0 * K;
  const float* b0 = DGRAD ? p.B : p.B + (size_t)col0 * K;
  uint32_t aoff[2 * WB], boff[2 * WB];
#pragma unroll
  for (int i = 0; i < 2 * WB; ++i) {
    const int lr = (lane >> 3) + 8 * i, lk = (lane & 7) * 4;
    aoff[i] = (uint32_t)min(lr, M - 1 - row0) * (uint32_t)K + lk;
    boff[i] = (uint32_t)min(lr, N - 1 - col0) * (uint32_t)K + lk;
  }
  const uint32_t coff = (uint32_t)(4 * g) * (uint32_t)N + (uint32_t)min(col0 + WB * r, N - WB);   // dgrad

  // Every D chunks are summed by themselves and then added: short chains.  (One chain over a whole reduction had up to 1.8
  // times the error against float64 of the two chains of gemm_f32.hip.)  One block: two accumulators in turn, so that
  // consecutive instructions do not depend on each other.
  constexpr int kChains = WB == 1 ? 2 : 1;
  const v4f kZero = {0.f, 0.f, 0.f, 0.f};
  v4f sum[kChains][WB][WB], acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j) acc[i][j] = kZero;
  auto mma = [&](const SmallFrag<WB>& a, const SmallFrag<WB>& b, const SmallCols<WB>& c, bool first) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
          for (int j = 0; j < WB; ++j) {
            v4f& t = sum[q % kChains][i][j];
            t = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[i][s][q], DGRAD ? c.v[s][q][j] : b.v[j][s][q],
                                                     first && s == 0 && q < kChains ? kZero : t, 0, 0, 0);
          }
  };
  auto settle = [&]() {
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
      for (int j = 0; j < WB; ++j) acc[i][j] += WB == 1 ? sum[0][i][j] + sum[kChains - 1][i][j] : sum[0][i][j];
  };

  // Forward: the bias travels beside the last products, all results of a thread are in one column.  (The mask of an input
  // gradient fetched there as well: launches with several workgroups per compute unit took 0.3 us longer.)
  static_assert(64 * NW % T == 0, "one column per thread");
  float bias = 0.f;
  auto fetch_bias = [&]() {
    if (!DGRAD && p.bias) bias = p.bias[min(col0 + tid % T, N - 1)];
  };

  const int nc = (K + kChunk - 1) / kChunk;
  const int cb = wave * nc / NW, ce = (wave + 1) * nc / NW;
  if (K < kChunk || ce <= cb) fetch_bias();
  if (K >= kChunk) {
    if (ce > cb) {
      // (a chunk past this wavefront's last one is that one again, unused: loads are never conditional)
      auto start = [&](int ch) { return min(min(ch, ce - 1) * kChunk, K - kChunk); };
      SmallLine<WB> ga[D], gb[D];
      SmallCols<WB> gc[D];
      SmallFrag<WB> fa, fb;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        line_load<WB>(ga[d], a0 + start(cb + d), aoff);
        if constexpr (DGRAD) cols_load<WB>(gc[d], b0 + (size_t)start(cb + d) * N, coff, N);
        else line_load<WB>(gb[d], b0 + start(cb + d), boff);
      }
      auto stage = [&](int d, int ch) {    // chunk ch from its registers through LDS, then refill them
        line_store<WB>(ga[d], la, lane);
        line_load<WB>(ga[d], a0 + start(ch + D), aoff);
        if constexpr (!DGRAD) {
          line_store<WB>(gb[d], lb, lane);
          line_load<WB>(gb[d], b0 + start(ch + D), boff);
        }
        frag_load<WB>(fa, la, r, g);
        if constexpr (!DGRAD) frag_load<WB>(fb, lb, r, g);
        const int lo = ch * kChunk - start(ch);
        if (lo > 0) {
          frag_clear_below<WB>(fa, lo, g);
          if constexpr (DGRAD) cols_clear_below<WB>(gc[d], lo, g);
          else frag_clear_below<WB>(fb, lo, g);
        }
      };
      int ch = cb;
      for (; ch + D <= ce; ch += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          stage(d, ch + d);
          mma(fa, fb, gc[d], d == 0);
          if constexpr (DGRAD) cols_load<WB>(gc[d], b0 + (size_t)start(ch + d + D) * N, coff, N);
          __builtin_amdgcn_sched_barrier(0);   // the loads stay in this order, so that a wait is for the oldest only
        }
        settle();
      }
      fetch_bias();
      for (int d = 0; ch + d < ce; ++d) {   // (D = 2: at most one)
        stage(0, ch + d);
        mma(fa, fb, gc[0], true);
        settle();
      }
    }
  } else if (ce > cb) {
    // fewer reduction elements than a chunk: element by element
    SmallFrag<WB> fa, fb;
    SmallCols<WB> fc;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 16 * s + 4 * g + q;
        const bool in = k < K;
        const int ko = in ? k : 0;   // (absent: element 0 of the row, counted zero)
#pragma unroll
        for (int i = 0; i < WB; ++i) {
          const float t = p.A[(size_t)min(row0 + 16 * i + r, M - 1) * K + ko];
          fa.v[i][s][q] = in ? t : 0.f;
          if constexpr (!DGRAD) {
            const float u = p.B[(size_t)min(col0 + 16 * i + r, N - 1) * K + ko];
            fb.v[i][s][q] = in ? u : 0.f;
          }
        }
        if constexpr (DGRAD) {
          load_n<WB>(p.B + (size_t)ko * N + min(col0 + WB * r, N - WB), fc.v[s][q]);
#pragma unroll
          for (int j = 0; j < WB; ++j) fc.v[s][q][j] = in ? fc.v[s][q][j] : 0.f;
        }
      }
    mma(fa, fb, fc, true);
    settle();
  }

  // accumulator register v of lane (r, g): row 4 g + v of its block, column r
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        la[(16 * i + 4 * g + v) * T + (DGRAD ? WB * r + j : 16 * j + r)] = acc[i][j][v];
      }
  __syncthreads();
#pragma unroll
  for (int e0 = 0; e0 < T * T; e0 += 64 * NW) {
    const int e = e0 + tid;
    if (T * T < 64 * NW && e >= T * T) break;
    const int row = row0 + e / T, col = col0 + e % T;
    if (row >= M || col >= N) continue;
    // (dgrad: a group of WB columns that was moved back holds column `col` at another place)
    const int grp = col0 + e % T / WB * WB;
    const int at = DGRAD && WB > 1 ? e + (grp - min(grp, N - WB)) : e;
    float y = lds[at];
#pragma unroll
    for (int w = 1; w < NW; ++w) y += lds[w * kWave + at];
    const size_t idx = (size_t)row * N + col;
    if (DGRAD) {
      if (p.mask) y = p.mask[idx] > 0.f ? y : 0.f;
      if (p.accumulate) y += p.C[idx];
    } else {
      if (p.bias) y += bias;
      if (p.relu) y = fmaxf(y, 0.f);
    }
    p.C[idx] = y;
  }
}

template <bool DGRAD, int WB, int NW>
__global__ __launch_bounds__(64 * NW, 3) void small_gemm_kernel(SmallGemm p) {
  __shared__ __attribute__((aligned(16))) float lds[small_gemm_floats<DGRAD, WB, NW>()];
  small_gemm_body<DGRAD, WB, NW>(p, (int)blockIdx.x, lds);
}

// An input gradient and, in front of its tiles, the classifier's parameter gradients and losses.
template <int WB>
__global__ __launch_bounds__(256, 3) void small_dgrad_head_kernel(SmallGemm p, HeadRole head, Segments seg) {
  constexpr int kGemm = small_gemm_floats<true, WB, 4>();
  __shared__ __attribute__((aligned(16))) float lds[kGemm > kHeadWgradLdsFloats ? kGemm : kHeadWgradLdsFloats];
  const int b = (int)blockIdx.x;
  if (b < head.blocks) head_wgrad_loss_body<float, 2>(head.p, seg, b, head.gx, lds);
  else small_gemm_body<true, WB, 4>(p, b - head.blocks, lds);
}

// ------------------------------------------------------------------ weight gradients

constexpr int kSmallJobs = 8;
struct SmallWgradJob {
  const float* dy;   // [rows][M]
  const float* x;    // [rows][N]
  float* gw;         // worker 0's [M][N]
  float* gb;         // worker 0's [M], may be null
  float* theta;      // with the update: the layer's weights, bias and their velocities
  float* theta_bias;
  float* vel;
  float* vel_bias;
  int M, N, tiles_n;
  uint32_t by_tiles_n;   // reciprocal_below(tiles_n)
};
struct SmallWgrad {
  int n, tiles;
  int first[kSmallJobs];   // first tile of the jobs
  size_t worker_stride;
  SmallWgradJob job[kSmallJobs];
};
// Many rows for few tiles: the rows are cut into shares, each of one worker (worker k has the shares first[k] .. first[k+1]-1
// of equal length), a workgroup takes one share, and gw and gb point at [share][worker_stride] of scratch.  Many workers for few tiles:
// a share is a worker, and gw and gb point at G (wgrad_workers_apart).
struct SmallShares {
  int32_t first[OMNI_MAX_WORKERS + 1];
};

// A chunk is 16 rows per wavefront: lane (r, g) supplies column r of dy and the WB neighbouring columns WB r .. of x of
// rows 4 s + g.
template <int WB>
struct WgradChunk {
  float a[4], b[4][WB];
};

// A wavefront (NW = 1, four tiles per workgroup) or the four wavefronts of a workgroup (NW = 4) own a 16 x 16 WB tile of
// one layer's weights and walk through all workers' rows, 16 rows each at a time; where a worker's rows end, its tile goes
// out to G[k].  UPD: 0 gradients only, 1 / 2 the SGD / momentum update of the tile's parameters at the end.
// The workgroup behind the last tile computes the losses.  SHARES: see SmallShares (UPD = 0; split_reduce_kernel follows,
// or the update where a share is a worker).
// The vector cache takes a load instruction of any width every 16 cycles, so with WB = 4 (one 4-byte and one 16-byte load
// per four matrix instructions, 128 matrix cycles) it stays out of the way; 16 x 16 and 32 x 32 tiles with 4- and 8-byte
// loads took twice the time.  997-501-243-37 net, 333 rows, 7 workers: 20.2 us with momentum (21.3 with the tables read
// where they are used and the parameters at the end).
template <int WB, int NW, int UPD, bool SHARES>
__global__ __launch_bounds__(256, 2) void small_wgrad_kernel(SmallWgrad p, Segments seg, Lambdas lam, Optim opt,
                                                          HeadLossParams hl, SmallShares sh) {
  static_assert(!SHARES || (NW == 4 && UPD == 0), "shares: four wavefronts, no update");
  constexpr int TN = 16 * WB, D = 4;
  constexpr bool MOM = UPD == 2;
  constexpr int kTileFloats = 16 * TN;
  constexpr int kOwn = (kTileFloats + 255) / 256;          // elements a thread adds up (NW = 4)
  __shared__ __attribute__((aligned(16))) float red[NW == 1 ? 1 : NW][NW == 1 ? kHeadLossLdsFloats : kTileFloats + 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (A line of arguments that nothing has touched takes 640 cycles: the lanes fetch the workers' rows and weights at once.)
  const int off_lane = seg.off[lane], off_last = seg.off[OMNI_MAX_WORKERS];
  const float lam_lane = UPD ? lam.v[lane] : 0.f;
  auto off = [&](int k) { return k < OMNI_MAX_WORKERS ? __builtin_amdgcn_readlane(off_lane, k) : off_last; };
  const int groups = NW == 1 ? (p.tiles + 3) / 4 : SHARES ? p.tiles * sh.first[seg.K] : p.tiles;
  if ((int)blockIdx.x == groups) {
    head_loss_body(hl, seg, &red[0][0]);
    return;
  }
  const int share = SHARES ? (int)blockIdx.x / p.tiles : 0;
  const int tile = NW == 1 ? (int)blockIdx.x * 4 + wave : (int)blockIdx.x - share * p.tiles;
  if (NW == 1 && tile >= p.tiles) return;   // (no barrier below with NW = 1)
  // the rows walked: all workers' one after the other, or a share of one worker's
  int beg0 = 0, end0 = off(1);
  const int nwork = SHARES ? 1 : seg.K;
  if (SHARES) {
    int k = 0;
    while (k + 1 < seg.K && share >= sh.first[k + 1]) ++k;
    const int at = share - sh.first[k], of = sh.first[k + 1] - sh.first[k], bk = off(k + 1) - off(k);
    beg0 = off(k) + (int)((long)bk * at / of);
    end0 = off(k) + (int)((long)bk * (at + 1) / of);
  }
  int ji = 0;
#pragma unroll
  for (int i = 1; i < kSmallJobs; ++i) ji += i < p.n && tile >= p.first[i] ? 1 : 0;
  const SmallWgradJob& J = p.job[ji];
  const int local = tile - p.first[ji];
  const int tile_m = quotient(local, J.by_tiles_n, J.tiles_n);
  const int tile_n = local - tile_m * J.tiles_n;
  const int M = J.M, N = J.N;
  const int r = lane & 15, g = lane >> 4;
  const int i0 = tile_m * 16, is = min(i0 + r, M - 1);                  // column of dy (past the end: the last one, unused)
  const int j_nom = tile_n * TN + WB * r, js = min(j_nom, N - WB);      // first column of x, moved back at the edge
  const bool want_bias = J.gb != nullptr && tile_n == 0;

  // A chunk that would run past the end of its worker's rows is moved back to end there; rows that are not its own are
  // zeroed in both operands (they may be another worker's: 0 * infinity is no zero).  Every address is then a uniform base plus a lane offset that never changes.
  constexpr int kSuper = 16 * NW;
  const int wrow = NW == 1 ? 0 : 16 * wave;
  const int last_row = off(seg.K) - 1;
  uint32_t aoff[4], boff[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t row = (uint32_t)min(4 * s + g, last_row);   // (fewer than 16 rows in all)
    aoff[s] = row * (uint32_t)M + (uint32_t)is;
    boff[s] = row * (uint32_t)N + (uint32_t)js;
  }
  auto start = [&](int k, int end) { return max(min(k + wrow, end - 16), 0); };
  auto load = [&](WgradChunk<WB>& c, int k, int end) {
    const size_t ks = (size_t)start(k, end);
    const float* dyk = J.dy + ks * (size_t)M;
    const float* xk = J.x + ks * (size_t)N;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      c.a[s] = dyk[aoff[s]];
      load_n<WB>(xk + boff[s], c.b[s]);
    }
  };
  // A chunk is summed by itself and added while the next one is multiplied, as above (one chain over a worker's rows had up to 3
  // times the error of the two of gemm_f32.hip).  One block: two accumulators in turn, so that no instruction waits for the last.
  constexpr int kChains = WB == 1 ? 2 : 1;
  v4f sum[2][kChains][WB], acc[WB];   // (chunks in turn)
  float bsum = 0.f, bgsum = 0.f, gsum[WB][4], own[kOwn];
  auto clear = [&]() {
    bsum = 0.f;
#pragma unroll
    for (int j = 0; j < WB; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
  };
  const v4f kZero = {0.f, 0.f, 0.f, 0.f};
  auto settle = [&](int set) {
#pragma unroll
    for (int j = 0; j < WB; ++j) acc[j] += WB == 1 ? sum[set][0][j] + sum[set][kChains - 1][j] : sum[set][0][j];
  };
  auto settled = [&](int set) {     // nothing in it that is still to be added
#pragma unroll
    for (int ch = 0; ch < kChains; ++ch)
#pragma unroll
      for (int j = 0; j < WB; ++j) sum[set][ch][j] = kZero;
  };
  settled(1);
  clear();
#pragma unroll
  for (int j = 0; j < WB; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) gsum[j][v] = 0.f;
#pragma unroll
  for (int e = 0; e < kOwn; ++e) own[e] = 0.f;

  // place of element e of the exchanged tile: column e % TN of row e / TN; of a group of WB columns moved back, the columns
  // that the group before it also holds are left to that one
  auto place = [&](int e, int& row, int& col) {
    const int cn = tile_n * TN + e % TN / WB * WB;
    row = i0 + e / TN;
    col = min(cn, N - WB) + e % WB;
    return row < M && col >= cn;
  };

  // the worker's rows are done: its tile goes out
  auto flush = [&](int w, int set) {       // (the other set has been added already)
    settle(set);
    settled(set);
    const int dst = SHARES ? share : w;
    float* G = J.gw + (size_t)dst * p.worker_stride;
    const float l = UPD ? lane_value(lam_lane, w) : 0.f;
    if (want_bias) {
      bsum += __shfl_xor(bsum, 16, 64);
      bsum += __shfl_xor(bsum, 32, 64);
    }
    if constexpr (NW == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = i0 + 4 * g + v;
        float t[WB];
#pragma unroll
        for (int j = 0; j < WB; ++j) {
          t[j] = acc[j][v];
          if (UPD) gsum[j][v] += l * t[j];
        }
        if (row < M) store_n<WB>(G + (size_t)row * N + js, t);
      }
      if (want_bias) {
        if (g == 0 && i0 + r < M) J.gb[(size_t)dst * p.worker_stride + i0 + r] = bsum;
        if (UPD) bgsum += l * bsum;
      }
    } else {
      __syncthreads();   // the exchange of the worker before has been read
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float t[WB];
#pragma unroll
        for (int j = 0; j < WB; ++j) t[j] = acc[j][v];
        store_n<WB>(&red[wave][(4 * g + v) * TN + WB * r], t);
      }
      if (want_bias && g == 0) red[wave][kTileFloats + r] = bsum;
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kOwn; ++q) {
        const int e = q * 256 + tid;
        float t = red[0][e];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww) t += red[ww][e];
        int row, col;
        if (place(e, row, col)) G[(size_t)row * N + col] = t;
        if (UPD) own[q] += l * t;
      }
      if (want_bias && tid < 16) {
        float t = red[0][kTileFloats + tid];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww) t += red[ww][kTileFloats + tid];
        if (i0 + tid < M) J.gb[(size_t)dst * p.worker_stride + i0 + tid] = t;
        if (UPD) bgsum += l * t;
      }
    }
    clear();
  };

  // stream of chunks: (worker, first row, end of its rows), D of them in flight
  int lw = 0, lk = beg0, lend = end0;       // next chunk to load
  auto advance = [&](int& w, int& k, int& end) {
    k += kSuper;
    if (__builtin_expect(k >= end, 0)) {
      ++w;
      if (w < nwork) { k = off(w); end = off(w + 1); }
    }
  };
  WgradChunk<WB> c[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load(c[d], lk, lend);
    if (lw < nwork) advance(lw, lk, lend);       // (past the last chunk: the last one again, unused)
  }
  // the parameters travel while the gradients are formed (loaded at the end, they were 2500 of a small network's 13500 cycles)
  float th1[NW == 1 && UPD ? 4 : 1][WB], ve1[NW == 1 && UPD ? 4 : 1][WB], th4[kOwn], ve4[kOwn], thb = 0.f, veb = 0.f;
  if constexpr (UPD != 0) {
    if constexpr (NW == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const size_t at = (size_t)min(i0 + 4 * g + v, M - 1) * N + js;
        load_n<WB>(J.theta + at, th1[v]);
        if (MOM) load_n<WB>(J.vel + at, ve1[v]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < kOwn; ++q) {
        int row, col;
        (void)place(q * 256 + tid, row, col);
        const size_t at = (size_t)min(row, M - 1) * N + col;
        th4[q] = J.theta[at];
        ve4[q] = MOM ? J.vel[at] : 0.f;
      }
    }
    if (want_bias) {
      const int bi = min(i0 + (NW == 1 ? r : tid & 15), M - 1);
      thb = J.theta_bias[bi];
      veb = MOM ? J.vel_bias[bi] : 0.f;
    }
  }
  int w = 0, k = beg0, end = end0;
  // (everything that does not happen in every chunk is out of line: a taken branch costs the wavefront an instruction
  // fetch, and a handful of them per chunk cost as much as its matrix instructions)
  for (bool more = true; more;) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (__builtin_expect(k + wrow + 16 > end, 0)) {
        const int ks = start(k, end), lo = k + wrow - ks, hi = end - ks;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bool own = 4 * s + g >= lo && 4 * s + g < hi;
          c[d].a[s] = own ? c[d].a[s] : 0.f;
#pragma unroll
          for (int j = 0; j < WB; ++j) c[d].b[s][j] = own ? c[d].b[s][j] : 0.f;
        }
      }
      if (want_bias) bsum += (c[d].a[0] + c[d].a[1]) + (c[d].a[2] + c[d].a[3]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < WB; ++j) {
          v4f& a = sum[d & 1][s % kChains][j];
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(c[d].a[s], c[d].b[s][j], s < kChains ? kZero : a, 0, 0, 0);
        }
      load(c[d], lk, lend);
      settle((d + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
      k += kSuper;
      if (__builtin_expect(k >= end, 0)) {
        flush(w, d & 1);
        ++w;
        if (w == nwork) { more = false; break; }
        k = off(w);
        end = off(w + 1);
      }
      if (__builtin_expect(lw < nwork, 1)) advance(lw, lk, lend);
    }
  }

  if constexpr (UPD != 0) {
    if constexpr (NW == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = i0 + 4 * g + v;
        if (row >= M) continue;
        float (&th)[WB] = th1[v], (&ve)[WB] = ve1[v];
        const size_t at = (size_t)row * N + js;
#pragma unroll
        for (int j = 0; j < WB; ++j) apply_update<MOM>(th[j], ve[j], gsum[j][v], opt);
        if (js == j_nom) {
          store_n<WB>(J.theta + at, th);
          if (MOM) store_n<WB>(J.vel + at, ve);
        } else {
#pragma unroll
          for (int j = 0; j < WB; ++j)
            if (js + j >= j_nom) {
              J.theta[at + j] = th[j];
              if (MOM) J.vel[at + j] = ve[j];
            }
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < kOwn; ++q) {
        int row, col;
        if (!place(q * 256 + tid, row, col)) continue;
        const size_t at = (size_t)row * N + col;
        apply_update<MOM>(th4[q], ve4[q], own[q], opt);
        J.theta[at] = th4[q];
        if (MOM) J.vel[at] = ve4[q];
      }
    }
    const int bi = i0 + (NW == 1 ? r : tid);
    if (want_bias && (NW == 1 ? g == 0 : tid < 16) && bi < M) {
      apply_update<MOM>(thb, veb, bgsum, opt);
      J.theta_bias[bi] = thb;
      if (MOM) J.vel_bias[bi] = veb;
    }
  }
}

// Second stage of the shares: a worker's are added in order into G[k], and with UPD the update of all parameters follows
// from the registers, in weighted_sgd_kernel's order (the results are the same bit for bit).
template <int UPD>
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ part, float* __restrict__ G,
                                                           size_t stride, long P, int K, SmallShares sh, Lambdas lam,
                                                           Optim opt, float* __restrict__ theta, float* __restrict__ vel) {
  constexpr bool MOM = UPD == 2;
  const long j = (long)blockIdx.x * 256 + threadIdx.x;
  if (j >= P) return;
  float th = UPD ? theta[j] : 0.f, ve = MOM ? vel[j] : 0.f, sum = 0.f;
  for (int k = 0; k < K; ++k) {
    const int s0 = sh.first[k], s1 = sh.first[k + 1];
    float g = 0.f;
    for (int s = s0; s < s1; s += 8) {               // eight loads in flight, added in order
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)min(s + u, s1 - 1) * stride + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) g = s + u < s1 ? g + v[u] : g;
    }
    G[(size_t)k * stride + j] = g;
    if (UPD) sum += lam.v[k] * g;
  }
  if (UPD) {
    apply_update<MOM>(th, ve, sum, opt);
    theta[j] = th;
    if (MOM) vel[j] = ve;
  }
}

}  // namespace

namespace {

inline int tiles_of(int rows, int cols, int t) { return ((rows + t - 1) / t) * ((cols + t - 1) / t); }

template <bool DGRAD>
void small_gemm(hipStream_t st, SmallGemm p, const HeadWgradParams* head, const Segments& seg) {
  // Four wavefronts per tile (with 8 or 16 the reduction is split further, but every one of them waits for its first
  // chunk: no faster anywhere).  32 x 32 tiles need half the operand traffic, 16 x 16 tiles spread a product with few
  // tiles over more compute units: measured, the lines cross near 160 tiles of 32 x 32.
  const int t32 = tiles_of(p.M, p.N, 32);
  const bool wide = p.N >= 2 && p.K >= 256 && t32 >= 160;
  const int T = wide ? 32 : 16;
  p.tiles = xcd_tiles((p.M + T - 1) / T, (p.N + T - 1) / T);
  if (DGRAD && head) {
    const HeadRole role = head_role(head, seg);
    const dim3 grid(p.tiles.grid() + role.blocks);
    if (wide) hipLaunchKernelGGL(small_dgrad_head_kernel<2>, grid, dim3(256), 0, st, p, role, seg);
    else hipLaunchKernelGGL(small_dgrad_head_kernel<1>, grid, dim3(256), 0, st, p, role, seg);
    return;
  }
  if (wide)
    hipLaunchKernelGGL((small_gemm_kernel<DGRAD, 2, 4>), dim3(p.tiles.grid()), dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((small_gemm_kernel<DGRAD, 1, 4>), dim3(p.tiles.grid()), dim3(256), 0, st, p);
}

template <int WB, int NW>
void launch_wgrad(hipStream_t st, const SmallWgrad& p, const Segments& seg, const Lambdas& lam, const Optim& opt,
                  const HeadLossParams& hl, int upd, bool loss, const KernelTimer* timer) {
  const dim3 grid((NW == 1 ? (p.tiles + 3) / 4 : p.tiles) + (loss ? 1 : 0)), block(256);
  const SmallShares none{};
#define OMNI_SMALL_WGRAD(U)                                                                                             \
  if (timer)                                                                                                            \
    hipExtLaunchKernelGGL((small_wgrad_kernel<WB, NW, U, false>), grid, block, 0, st, timer->start, timer->stop, 0, p,  \
                          seg, lam, opt, hl, none);                                                                     \
  else                                                                                                                  \
    hipLaunchKernelGGL((small_wgrad_kernel<WB, NW, U, false>), grid, block, 0, st, p, seg, lam, opt, hl, none)
  if (upd == 0) { OMNI_SMALL_WGRAD(0); }
  else if (upd == 1) { OMNI_SMALL_WGRAD(1); }
  else { OMNI_SMALL_WGRAD(2); }
#undef OMNI_SMALL_WGRAD
}

// Shares of a weight gradient with `tiles` tiles: as many as give the chip four workgroups per compute unit, at least 64 rows
// each and one per worker, within `scratch_rows` in all.  A compute unit needs about 6.5 ns per row of a tile, which only the
// compute units without a tile can take off it, and the second launch costs about 5 us: measured with 1024 and 4096 rows, the
// line lies near 850 rows times the idle part of the chip (64-128-10 net, 4096 rows: step 42 -> 26 us; 256-256-10, 1024 rows:
// 23 -> 26).
long shares_wanted(long tiles, long rows) {
  if (tiles < 1 || rows * (256 - tiles) < 850 * 256) return 0;
  return std::min<long>(std::min<long>(1024 / tiles, rows / 64), 64);
}
bool wgrad_shares(long tiles, const Segments& seg, size_t scratch_rows, SmallShares& sh) {
  const long rows = seg.off[seg.K];
  for (long want = shares_wanted(tiles, rows); want >= 2; --want) {
    sh.first[0] = 0;
    for (int k = 0; k < seg.K; ++k)
      sh.first[k + 1] = sh.first[k] + (int)std::max<long>(1, want * (seg.off[k + 1] - seg.off[k]) / rows);
    if ((size_t)sh.first[seg.K] <= scratch_rows) return sh.first[seg.K] >= 2;
  }
  return false;
}

// Whether every worker's rows are one share that goes straight to G, and the update is a launch of its own behind it: the walk through
// the workers, 1.4 us each with the exchange at its end, against that launch (4 us).  Step in us, together / apart:
//    4 tiles   8 workers,  64 rows 19.5 / 18.8   16, 600 31.2 / 21.3   32, 600 52.9 / 27.4
//   43 tiles   8 workers,  64 rows 20.6 / 19.4   16, 600 33.8 / 23.4   32, 600 55.5 / 32.5
//   64 tiles   8 workers,  64 rows 21.2 / 22.6    8, 333 25.4 / 23.3   12,  39 31.5 / 32.7   16, 128 34.4 / 30.3   32, 600 56.9 / 50.5
//  125 tiles   8 workers, 333 rows 37.4 / 37.8   16, 600 48.7 / 51.0   32, 600 70.6 / 75.8
// (four workers, 24 tiles: 16.2 / 16.1)
bool wgrad_workers_apart(long tiles, const Segments& seg) {
  return seg.K >= 8 && (tiles <= 44 || (tiles <= 64 && (seg.K >= 16 || seg.off[seg.K] >= 256)));
}

// 16 x 64 tiles of the jobs; narrow: some layer's rows are shorter than a vector, which takes 16 x 16 tiles and no shares
long wgrad_tiles(const LinearWgradJob* jobs, int n, bool& narrow) {
  long tiles = 0;
  narrow = false;
  for (int i = 0; i < n; ++i) {
    tiles += (long)((jobs[i].cout + 15) / 16) * ((jobs[i].cin + 63) / 64);
    narrow = narrow || jobs[i].cin < 4;
  }
  return tiles;
}

}  // namespace

bool linear_f32_small(int rows, int cols, int kred) {
  const long tiles64 = (long)tiles_of(rows, cols, 64);
  return kred < 32 || cols < 4 || tiles64 < kSmallMaxTiles64;
}

void linear_fwd_f32_small(hipStream_t st, const float* x, const float* w, const float* bias, float* y, int rows,
                          int cin, int cout, bool relu) {
  small_gemm<false>(st, SmallGemm{x, w, y, rows, cout, cin, bias, nullptr, relu ? 1 : 0, 0, {}}, nullptr, Segments{});
}

void linear_dgrad_f32_small(hipStream_t st, const float* dy, const float* w, const float* mask, float* dx, int rows,
                            int cin, int cout, bool accumulate, const HeadWgradParams* head, const Segments& seg) {
  small_gemm<true>(st, SmallGemm{dy, w, dx, rows, cin, cout, nullptr, mask, 0, accumulate ? 1 : 0, {}}, head, seg);
}

size_t linear_wgrad_f32_share_rows(const LinearWgradJob* jobs, int n, int K_max, int B_max) {
  bool narrow;
  const long want = shares_wanted(wgrad_tiles(jobs, n, narrow), B_max);
  return narrow || n > kSmallJobs || want < 2 ? 0 : (size_t)(want + K_max - 1);
}

bool linear_wgrad_f32_small(hipStream_t st, const LinearWgradJob* jobs, int n, size_t worker_stride, const Segments& seg,
                            const HeadLossParams* loss, const SgdArgs* sgd, const KernelTimer* timer,
                            const WgradScratch& scratch) {
  bool narrow;
  const long tiles = wgrad_tiles(jobs, n, narrow);
  // Enough tiles for the chip's 1024 SIMDs, or few rows: one wavefront walks all rows of a tile and needs no exchange.
  // Otherwise the rows are dealt to the four wavefronts of a workgroup.
  const int nw = tiles >= 512 || seg.off[seg.K] <= 64 ? 1 : 4;
  const int TN = narrow ? 16 : 64;
  const int upd = sgd ? (sgd->velocity ? 2 : 1) : 0;
  const Lambdas lam = lambdas_of(seg);
  const Optim opt = sgd ? Optim{sgd->lr, sgd->momentum, sgd->weight_decay} : Optim{0.f, 0.f, 0.f};
  const bool one = n <= kSmallJobs;
  SmallShares sh{};
  const bool shares = scratch.part && !narrow && one && wgrad_shares(tiles, seg, scratch.rows, sh);
  const bool apart = !shares && !narrow && one && wgrad_workers_apart(tiles, seg);
  if (shares || apart) {
    if (apart)
      for (int k = 0; k <= seg.K; ++k) sh.first[k] = k;
    SmallWgrad p{};
    p.n = n;
    p.worker_stride = worker_stride;
    for (int i = 0; i < n; ++i) {
      const LinearWgradJob& j = jobs[i];
      SmallWgradJob& q = p.job[i];
      q.dy = j.dy; q.x = j.x; q.M = j.cout; q.N = j.cin;
      q.gw = apart ? j.gw : scratch.part + j.w_off;
      q.gb = apart || !j.gb ? j.gb : scratch.part + j.b_off;
      q.tiles_n = (j.cin + TN - 1) / TN;
      p.first[i] = p.tiles;
      p.tiles += (j.cout + 15) / 16 * q.tiles_n;
      q.by_tiles_n = reciprocal_below(q.tiles_n, p.tiles - p.first[i]);
    }
    if (timer) (void)hipEventRecord(timer->start, st);
    hipLaunchKernelGGL((small_wgrad_kernel<4, 4, 0, true>), dim3(p.tiles * sh.first[seg.K] + (loss ? 1 : 0)), dim3(256), 0, st,
                       p, seg, lam, opt, loss ? *loss : HeadLossParams{}, sh);
    if (apart) {
      if (timer) (void)hipEventRecord(timer->stop, st);
      return false;
    }
    const dim3 grid((unsigned)((scratch.params + 255) / 256));
#define OMNI_REDUCE(U)                                                                                                   \
  hipLaunchKernelGGL(split_reduce_kernel<U>, grid, dim3(256), 0, st, scratch.part, scratch.G, worker_stride,             \
                     (long)scratch.params, seg.K, sh, lam, opt, sgd ? sgd->params : nullptr, sgd ? sgd->velocity : nullptr)
    if (upd == 0) OMNI_REDUCE(0);
    else if (upd == 1) OMNI_REDUCE(1);
    else OMNI_REDUCE(2);
#undef OMNI_REDUCE
    if (timer) (void)hipEventRecord(timer->stop, st);
    return sgd != nullptr;
  }
  if (timer && !one) (void)hipEventRecord(timer->start, st);
  for (int base = 0; base < n; base += kSmallJobs) {
    SmallWgrad p{};
    p.n = std::min(n - base, kSmallJobs);
    p.worker_stride = worker_stride;
    for (int i = 0; i < p.n; ++i) {
      const LinearWgradJob& j = jobs[base + i];
      SmallWgradJob& q = p.job[i];
      q.dy = j.dy; q.x = j.x; q.gw = j.gw; q.gb = j.gb; q.M = j.cout; q.N = j.cin;
      if (sgd) {
        q.theta = sgd->params + j.w_off; q.theta_bias = sgd->params + j.b_off;
        if (sgd->velocity) { q.vel = sgd->velocity + j.w_off; q.vel_bias = sgd->velocity + j.b_off; }
      }
      q.tiles_n = (j.cin + TN - 1) / TN;
      p.first[i] = p.tiles;
      p.tiles += (j.cout + 15) / 16 * q.tiles_n;
      q.by_tiles_n = reciprocal_below(q.tiles_n, p.tiles - p.first[i]);
    }
    const bool last = base + kSmallJobs >= n;
    const HeadLossParams hl = loss ? *loss : HeadLossParams{};
    const bool with_loss = loss && last;
    const KernelTimer* tm = one ? timer : nullptr;
    if (narrow) launch_wgrad<1, 4>(st, p, seg, lam, opt, hl, upd, with_loss, tm);
    else if (nw == 1) launch_wgrad<4, 1>(st, p, seg, lam, opt, hl, upd, with_loss, tm);
    else launch_wgrad<4, 4>(st, p, seg, lam, opt, hl, upd, with_loss, tm);
  }
  if (timer && !one) (void)hipEventRecord(timer->stop, st);
  return sgd != nullptr;
}

}  // namespace omni
