// fp32 matrix products on the CDNA4 matrix cores (v_mfma_f32_32x32x2_f32).
//
// These are the dense contractions inside the per-worker gradient of
// Algorithm 1 (procedure Train, gradient line) for fully connected layers:
//   forward   Y  = X W^T + bias            (rows of all workers in one launch)
//   dgrad     dX = dY W                     (rows of all workers in one launch)
//   wgrad     G_k = dY_k^T X_k              (one output per worker, reduction
//                                            over that worker's rows only)
//
// One kernel template serves all three.  It computes C[i][j] = sum_kk A(i,kk) *
// B(j,kk) where each operand is either "k-contiguous" (element (r,kk) at
// base[r*ld + kk]) or "row-contiguous" (element (r,kk) at base[kk*ld + r]).
// A workgroup is 4 wavefronts in a 2x2 grid over a 64x64 output tile; each
// wavefront owns one 32x32 accumulator block.  Operand slabs of BK reduction
// steps are staged through LDS with register prefetch of the next slab
// (double-buffered LDS, one barrier per slab).
//
// Products with too few tiles to fill the chip are those of gemm_f32_direct.hip and gemm_f32_small.hip, the largest those of
// gemm_f32_split.hip (all are asked first).
//
// wgrad gives every workgroup one output tile position and lets it walk through
// ALL workers' row ranges one after the other, flushing the accumulator into
// worker k's gradient when k's rows end.  Every workgroup then does the same
// amount of work however ragged the b_k are, and, holding all workers' gradients
// of its tile in turn, it can apply the SGD update of the tile's parameters at
// the end.  The weight gradients of all layers share one launch
// (linear_wgrad_f32_batch): their workgroups follow each other in one grid.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"
#include "head_device.h"
#include "kernels.h"
#include "update_device.h"

namespace omni {

typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

constexpr int kThreads = 256;
constexpr int kTile = 64;
// Weight gradients come here with this many 64 x 64 tiles in the launch (one per compute unit), whatever the rows; fewer
// go to gemm_f32_small.hip (its time against this kernel's, with the update: 136 tiles, 1000 rows 34.5 / 37.0 us; 164 tiles,
// 333 rows 19.6 / 24.1, 2000 rows 61.5 / 66.1; 256 tiles, 64 rows 12.5 / 14.4, 333 rows 26.1 / 24.1; 1024 tiles, 32 rows
// 22.3 / 19.2, 480 rows 71.1 / 51.1).
constexpr long kTiledWgradTiles = 256;

// Staging of one operand slab: R rows x BK reduction steps.
template <int R, int BK, bool MC>
struct Slab {
  static constexpr int kChunks = R * BK / 4;
  static constexpr int kPerThread = kChunks / kThreads;
  static_assert(kChunks % kThreads == 0 && kPerThread >= 1, "slab must divide over the workgroup");
  // k-contiguous slabs sit in LDS as [row][BK+4] (16-byte reads along kk, rows
  // land 4 banks apart); row-contiguous slabs as [kk][R+8].
  static constexpr int kStride = MC ? (R + 8) : (BK + 4);
  static constexpr int kFloats = MC ? BK * (R + 8) : R * (BK + 4);

  // Loads never branch, so that the compiler keeps them in flight across the whole MFMA section of the
  // current slab.  Requires at least BK reduction steps and at least 4 rows in a row-contiguous operand; rows may start at
  // any multiple of 4 bytes (16-byte loads need no more).  A row-contiguous piece that would run past the last
  // row is moved back to end there: its place in the tile then holds other rows than its index says (piece_start).
  // Everything that does not change from slab to slab is worked out once per
  // thread (`Pre`): the per-slab address is one 64-bit add per piece.  The vector
  // ALU shares issue slots with the matrix pipe, so every instruction saved here
  // is matrix time gained.
  struct Pre {
    long cpart[kPerThread];   // element offset of the piece for slab start 0
  };
  __device__ static inline Pre prepare(int ld, int row0, int rows, int tid) {
    Pre pre;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int c = tid + kThreads * i;
      if (!MC) {
        const int r = row0 + c / (BK / 4), kc = (c % (BK / 4)) * 4;
        pre.cpart[i] = r < rows ? (long)r * ld + kc : (long)kc;      // absent row: row 0 stands in
      } else {
        const int kk = c / (R / 4), r = row0 + (c % (R / 4)) * 4;
        pre.cpart[i] = (long)kk * ld + max(min(r, rows - 4), 0);
      }
    }
    return pre;
  }

  // A slab whose BK reduction steps all lie inside the
  // range is loaded as it is.  A slab that would run past the end of its range is moved
  // back so that it ENDS at the end of the range (start ks = max(kend - BK, 0): the caller
  // guarantees at least BK reduction steps in the operand, so this stays in bounds); the
  // steps of the slab outside [k0, kend) are zeroed in LDS afterwards (zero_outside), which
  // happens once per range.  Rows outside the operand are not zeroed at all: they only
  // feed outputs that are never stored.  The loop over full slabs then has no validity
  // bits, no selects and one address add per piece.
  __device__ static inline void load_fast(v4f (&reg)[kPerThread], const float* __restrict__ base, int ld, int ks,
                                          const Pre& pre) {
    const float* sbase = base + (MC ? (long)ks * ld : (long)ks);
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) reg[i] = *reinterpret_cast<const v4f_a4*>(sbase + pre.cpart[i]);
  }
  __device__ static inline void store_fast(const v4f (&reg)[kPerThread], float* lds, int tid, int i) {
    const int c = tid + kThreads * i;
    if (!MC) {
      const int r = c / (BK / 4), kc = (c % (BK / 4)) * 4;
      *reinterpret_cast<v4f*>(lds + r * kStride + kc) = reg[i];
    } else {
      const int kk = c / (R / 4), rc = (c % (R / 4)) * 4;
      *reinterpret_cast<v4f*>(lds + kk * kStride + rc) = reg[i];
    }
  }
  // zero the reduction steps of a staged slab outside [lo, hi)
  __device__ static inline void zero_outside(float* lds, int lo, int hi, int tid) {
    for (int idx = tid; idx < R * BK; idx += kThreads) {
      const int kk = MC ? idx / R : idx % BK;
      const int r = MC ? idx % R : idx / BK;
      if (kk < lo || kk >= hi) lds[MC ? kk * kStride + r : r * kStride + kk] = 0.f;
    }
  }

  // First operand row of the four-row piece that tile index i belongs to (row-contiguous operands, see above).
  __device__ static inline int piece_start(int row0, int i, int rows) { return min(row0 + (i & ~3), rows - 4); }

  // Operand registers for the 4 MFMA steps covering kk = ks*8 .. ks*8+7 of the
  // slab, for the 32-row block starting at `row`.  Lane l supplies row l%32 and
  // reduction index ks*8 + (l/32)*4 + q in step q; both operands use the same
  // map, which is all the instruction needs.
  __device__ static inline v4f frag(const float* lds, int row, int ks, int lane) {
    const int r = row + (lane & 31), kb = ks * 8 + (lane >> 5) * 4;
    if (!MC) {
      return *reinterpret_cast<const v4f*>(lds + r * kStride + kb);
    } else {
      v4f v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = lds[(kb + q) * kStride + r];
      return v;
    }
  }
};

enum { MODE_FWD = 0, MODE_DGRAD = 1, MODE_WGRAD = 2 };

// LDS of one workgroup, in floats: two stages of both slabs and, for WGRAD, the bias-gradient partial sums.
template <int BK, bool A_MC, bool B_MC, int MODE>
constexpr int gemm_lds_floats() {
  return 2 * (Slab<kTile, BK, A_MC>::kFloats + Slab<kTile, BK, B_MC>::kFloats) + (MODE == MODE_WGRAD ? 4 * kTile : 0);
}

struct GemmParams {
  const float* A;
  const float* B;
  float* C;
  int M, N;  // rows of A / rows of B = rows / cols of C
  int lda, ldb, ldc;
  int kred;            // reduction length (FWD / DGRAD)
  const float* bias;   // FWD: added per output column, may be null
  const float* mask;   // DGRAD: [M][ldc]; the value passes where mask > 0, may be null
  int relu;            // FWD
  int accumulate;      // DGRAD: C += result
  int xcd_remap;       // FWD / DGRAD: 1 if the workgroups are re-ordered per XCD
  size_t c_worker_stride;  // WGRAD: floats between consecutive workers' outputs
  float* bias_grad;        // WGRAD: per worker column sums of A (at + worker*c_worker_stride), may be null
  float* theta;            // WGRAD with the update: this layer's weights and bias (and velocities), null without
  float* theta_bias;
  float* velocity;
  float* velocity_bias;
};

// (The second launch bound caps the kernel at 256 registers: the compiler then issues the MFMAs on
// ordinary vector registers.  With accumulation registers it copied all 32 accumulator registers in
// and out around the MFMAs of every step, 64 extra vector instructions per 16 MFMAs, because the
// per-worker flush inside the loop reads and zeroes them.)
// The whole workgroup program; bx is the workgroup's place among nbx workgroups.
// UPD (WGRAD): 1 / 2 if the workgroups, having walked through ALL workers, also apply the SGD / momentum update to
// the parameters of their tile (lam, opt).
template <int BK, bool A_MC, bool B_MC, int MODE, int UPD>
__device__ __forceinline__ void gemm_f32_body(const GemmParams& p, const Segments& seg, const int bx, const int nbx, float* lds,
                                              const Lambdas* lam = nullptr, const Optim* opt = nullptr) {
  using SA = Slab<kTile, BK, A_MC>;
  using SB = Slab<kTile, BK, B_MC>;
  constexpr int kStage = SA::kFloats + SB::kFloats;
  // WGRAD: the four wavefronts' bias-gradient partial sums
  float (*bred)[kTile] = reinterpret_cast<float (*)[kTile]>(lds + 2 * kStage);
  constexpr int kFlushStride = kTile + 4;          // WGRAD: row stride of the output tile staged for the flush
  static_assert(kTile * kFlushStride <= kStage, "the staged output tile must fit one LDS stage");
  auto sA = [&](int stage) { return lds + stage * kStage; };
  auto sB = [&](int stage) { return lds + stage * kStage + SA::kFloats; };

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_n = (p.N + kTile - 1) / kTile;
  const int tiles_m = (p.M + kTile - 1) / kTile;
  int tile = bx;
  // Forward / dgrad workgroups are dealt to the 8 XCDs round-robin by index; re-ordered so that each XCD owns a
  // contiguous run of tiles, whose columns of B its own L2 then holds.
  if (MODE != MODE_WGRAD && p.xcd_remap) tile = (bx & 7) * (nbx >> 3) + (bx >> 3);
  // tile_n major: consecutive tiles share the same rows of B
  const int tile_n = (MODE == MODE_WGRAD) ? tile % tiles_n : tile / tiles_m;
  const int tile_m = (MODE == MODE_WGRAD) ? tile / tiles_n : tile % tiles_m;
  const int row0 = tile_m * kTile, col0 = tile_n * kTile;
  const int wrow = (wave >> 1) * 32, wcol = (wave & 1) * 32;

  // The reduction is a stream of slabs over one or more consecutive ranges
  // ("workers"); the accumulator is flushed whenever a range ends.  A slab is
  // (range index w, start k0, end of its range kend); w == nrange marks the end.
  const int nrange = (MODE == MODE_WGRAD) ? seg.K : 1;
  int w0 = 0, k00, kend0;
  if (MODE == MODE_WGRAD) {
    k00 = seg.off[0];
    kend0 = seg.off[1];
  } else {
    k00 = 0;
    kend0 = p.kred;
  }
#define OMNI_NEXT_SLAB(W, K0, KEND, NW, NK0, NKEND)       \
  int NW = W, NK0 = K0 + BK, NKEND = KEND;                \
  if (NK0 >= KEND) {                                      \
    NW = W + 1;                                           \
    if (MODE == MODE_WGRAD && NW < nrange) {              \
      NK0 = seg.off[NW];                                  \
      NKEND = seg.off[NW + 1];                            \
    }                                                     \
  }

  // A slab's sum (acc) and the range's (acc2), to which the slab's is added when it is complete: chains of BK products and one
  // of slabs.  Against float64 the error is a third of that of two chains over a reduction of 3072, half over 1000.
  v16f acc, acc2;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = acc2[v] = 0.f;
  // WGRAD with the update: sum_k lambda_k G[k] of the 16-byte pieces this thread stores, in the order of the update
  // kernel, so that the gradient rows are never fetched again
  v4f gsum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) gsum[q] = v4f{0.f, 0.f, 0.f, 0.f};
  float bgsum = 0.f;
  const bool want_bias_grad = (MODE == MODE_WGRAD) && p.bias_grad != nullptr && tile_n == 0;
  float bsum = 0.f;

  // Accumulator layout of the 32x32 block: register v of lane l holds
  // row 8*(v/4) + 4*(l/32) + v%4, column l%32.
  const int j = col0 + wcol + (lane & 31);
  const int ibase = row0 + wrow + 4 * (lane >> 5);

  // Two register sets hold the slabs one and two steps ahead of the one being
  // multiplied, so every global load has two MFMA sections to arrive in.  WGRAD has the registers for one set only
  // (four wavefronts per SIMD: 128); a load has one section, and the other wavefronts', to arrive in.
  constexpr bool kOneSet = MODE == MODE_WGRAD;
  const typename SA::Pre preA = SA::prepare(p.lda, row0, p.M, tid);
  const typename SB::Pre preB = SB::prepare(p.ldb, col0, p.N, tid);
  v4f ra0[SA::kPerThread], rb0[SB::kPerThread], ra1[SA::kPerThread], rb1[SB::kPerThread];
  OMNI_NEXT_SLAB(w0, k00, kend0, w1, k01, kend1)
  // start of the slab as it is fetched (see Slab::load_fast)
#define OMNI_KSTART(K0, KEND) ((K0) + BK <= (KEND) ? (K0) : max((KEND) - BK, 0))
  // Prefetches past the end of the stream are still issued (they re-read the
  // first slab and are discarded): a load that is issued on one path only would force
  // every later wait to assume it is not there and drain the whole queue.
  if (w1 >= nrange) { k01 = 0; kend1 = 0; }
  SA::load_fast(ra0, p.A, p.lda, OMNI_KSTART(k00, kend0), preA);
  SB::load_fast(rb0, p.B, p.ldb, OMNI_KSTART(k00, kend0), preB);
  if (!kOneSet) {
    SA::load_fast(ra1, p.A, p.lda, OMNI_KSTART(k01, kend1), preA);
    SB::load_fast(rb1, p.B, p.ldb, OMNI_KSTART(k01, kend1), preB);
  }
#pragma unroll
  for (int i = 0; i < SA::kPerThread; ++i) SA::store_fast(ra0, sA(0), tid, i);
#pragma unroll
  for (int i = 0; i < SB::kPerThread; ++i) SB::store_fast(rb0, sB(0), tid, i);
  if (k00 + BK > kend0) {
    const int ks = OMNI_KSTART(k00, kend0);
    __syncthreads();
    SA::zero_outside(sA(0), k00 - ks, kend0 - ks, tid);
    SB::zero_outside(sB(0), k00 - ks, kend0 - ks, tid);
  }
  __syncthreads();

  // One pipeline step: multiply slab 0 (already in LDS stage CUR, a constant of each of the two
  // copies of the step, so that every LDS address is an immediate offset), fetch the
  // slab two ahead into the free register set (LA/LB), then move the slab one
  // ahead from its register set (NA/NB) into the other LDS stage.
#define OMNI_STEP(CUR, LA, LB, NA, NB)                                                               \
  {                                                                                                     \
    int w2 = nrange, k02 = 0, kend2 = 0;                                                                \
    if (w1 < nrange) {                                                                                  \
      OMNI_NEXT_SLAB(w1, k01, kend1, tw, tk0, tkend)                                                    \
      w2 = tw; k02 = tk0; kend2 = tkend;                                                                \
    }                                                                                                   \
    if (w2 >= nrange) { k02 = 0; kend2 = 0; }                                                           \
    {                                                                                                   \
      const int ks2 = kOneSet ? OMNI_KSTART(k01, kend1) : OMNI_KSTART(k02, kend2);                      \
      SA::load_fast(LA, p.A, p.lda, ks2, preA);                                                         \
      SB::load_fast(LB, p.B, p.ldb, ks2, preB);                                                         \
    }                                                                                                   \
    __builtin_amdgcn_sched_barrier(0); /* keep the fetches ahead of the MFMA section */                 \
    /* The slab one step ahead has been in flight for a whole step: its pieces go to the other LDS */  \
    /* stage in between the MFMA groups of this slab, and the operand fragments of the next group   */  \
    /* are fetched before the current group is issued, so that the matrix pipe is not left waiting. */  \
    {                                                                                                   \
      v4f fa[2], fb[2];                                                                                 \
      fa[0] = SA::frag(sA(CUR), wrow, 0, lane);                                                         \
      fb[0] = SB::frag(sB(CUR), wcol, 0, lane);                                                         \
      _Pragma("unroll") for (int ks = 0; ks < BK / 8; ++ks) {                                           \
        if (ks + 1 < BK / 8) {                                                                          \
          fa[(ks + 1) & 1] = SA::frag(sA(CUR), wrow, ks + 1, lane);                                     \
          fb[(ks + 1) & 1] = SB::frag(sB(CUR), wcol, ks + 1, lane);                                     \
        }                                                                                               \
        _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                                 \
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[ks & 1][q], fb[ks & 1][q], acc, 0, 0, 0);       \
        }                                                                                               \
        if (kOneSet) {                                                                                  \
        } else if (ks < SA::kPerThread) SA::store_fast(NA, sA(1 - CUR), tid, ks);                       \
        else if (ks - SA::kPerThread < SB::kPerThread) SB::store_fast(NB, sB(1 - CUR), tid, ks - SA::kPerThread); \
        __builtin_amdgcn_sched_barrier(0);                                                              \
      }                                                                                                 \
    }                                                                                                   \
    if (kOneSet) {                                                                                      \
      _Pragma("unroll") for (int i = 0; i < SA::kPerThread; ++i) SA::store_fast(LA, sA(1 - CUR), tid, i); \
      _Pragma("unroll") for (int i = 0; i < SB::kPerThread; ++i) SB::store_fast(LB, sB(1 - CUR), tid, i); \
    }                                                                                                   \
    _Pragma("unroll") for (int v = 0; v < 16; ++v) { acc2[v] += acc[v]; acc[v] = 0.f; }                 \
    if (w1 < nrange && k01 + BK > kend1) {                                                              \
      /* the slab just staged runs past the end of its range: it was fetched moved back; clear the */  \
      /* reduction steps that are not its own (once per range; all its pieces must have landed)     */  \
      const int ks1 = OMNI_KSTART(k01, kend1);                                                          \
      __syncthreads();                                                                                  \
      SA::zero_outside(sA(1 - CUR), k01 - ks1, kend1 - ks1, tid);                                       \
      SB::zero_outside(sB(1 - CUR), k01 - ks1, kend1 - ks1, tid);                                       \
    }                                                                                                   \
    if (want_bias_grad) {                                                                               \
      /* A is the output-gradient slab [kk][row]: its column sums are the bias gradient.  Each */       \
      /* wavefront adds a quarter of the slab's reduction steps; the quarters meet at the flush. */     \
      _Pragma("unroll") for (int kk = 0; kk < BK / 4; ++kk)                                             \
        bsum += sA(CUR)[(wave * (BK / 4) + kk) * SA::kStride + lane];                                   \
    }                                                                                                   \
    if (MODE == MODE_WGRAD && w1 != w0) {                                                               \
      /* this worker's rows are done: its tile goes out (stores only; the prefetch stays in flight) */ \
      float* C = p.C + (size_t)w0 * p.c_worker_stride;                                                  \
      /* through the LDS stage that was just multiplied, so that every thread writes 16-byte pieces */   \
      /* of whole 256-byte rows (scattered 4-byte stores, 16 per lane, cost 3 us per launch).  A piece */ \
      /* moved back at the edge of the matrix writes a few elements a second time, with the same values. */ \
      float* tile = sA(CUR);                                                                            \
      __syncthreads(); /* every wavefront is done reading this stage */                                 \
      _Pragma("unroll") for (int v = 0; v < 16; ++v)                                                    \
        tile[(wrow + 4 * (lane >> 5) + 8 * (v / 4) + (v % 4)) * kFlushStride + wcol + (lane & 31)] = acc2[v]; \
      if (want_bias_grad) bred[wave][lane] = bsum;                                                      \
      __syncthreads();                                                                                  \
      _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                                   \
        const int idx = tid + kThreads * q, r = idx >> 4, c4 = (idx & 15) * 4;                          \
        const v4f t = *reinterpret_cast<const v4f*>(tile + r * kFlushStride + c4);                      \
        *reinterpret_cast<v4f_a4*>(C + (size_t)(SA::piece_start(row0, r, p.M) + (r & 3)) * p.ldc +      \
                                   SB::piece_start(col0, c4, p.N)) = t;                                 \
        if (UPD) gsum[q] += lam->v[w0] * t;                                                             \
      }                                                                                                 \
      if (want_bias_grad && tid < kTile) {                                                              \
        const float t = ((bred[0][tid] + bred[1][tid]) + bred[2][tid]) + bred[3][tid];                  \
        p.bias_grad[(size_t)w0 * p.c_worker_stride + SA::piece_start(row0, tid, p.M) + (tid & 3)] = t;  \
        if (UPD) bgsum += lam->v[w0] * t;                                                               \
      }                                                                                                 \
      bsum = 0.f;                                                                                       \
      _Pragma("unroll") for (int v = 0; v < 16; ++v) acc2[v] = 0.f;                                     \
    }                                                                                                   \
    if (w1 >= nrange) break;                                                                            \
    __syncthreads();                                                                                    \
    w0 = w1; k00 = k01; kend0 = kend1;                                                                  \
    w1 = w2; k01 = k02; kend1 = kend2;                                                                  \
  }
  for (;;) {
    if (kOneSet) {
      OMNI_STEP(0, ra0, rb0, ra0, rb0)
      OMNI_STEP(1, ra0, rb0, ra0, rb0)
    } else {
      OMNI_STEP(0, ra0, rb0, ra1, rb1)
      OMNI_STEP(1, ra1, rb1, ra0, rb0)
    }
  }
#undef OMNI_STEP
#undef OMNI_NEXT_SLAB
#undef OMNI_KSTART

  if (MODE == MODE_WGRAD && UPD != 0) {
    constexpr bool MOM = UPD == 2;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = tid + kThreads * q, r = idx >> 4, c4 = (idx & 15) * 4;
      const int rs = SA::piece_start(row0, r, p.M), cs = SB::piece_start(col0, c4, p.N);
      const size_t e0 = (size_t)(rs + (r & 3)) * p.ldc + cs;
      v4f th = *reinterpret_cast<const v4f_a4*>(p.theta + e0), vel = {0.f, 0.f, 0.f, 0.f};
      if (MOM) vel = *reinterpret_cast<const v4f_a4*>(p.velocity + e0);
      apply_update<MOM>(th, vel, gsum[q], *opt);
      if (rs + (r & 3) < row0 + (r & ~3)) continue;      // this row belongs to the piece before it
      if (cs == col0 + c4) {
        *reinterpret_cast<v4f_a4*>(p.theta + e0) = th;
        if (MOM) *reinterpret_cast<v4f_a4*>(p.velocity + e0) = vel;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (cs + e >= col0 + c4) {
            p.theta[e0 + e] = th[e];
            if (MOM) p.velocity[e0 + e] = vel[e];
          }
      }
    }
    if (want_bias_grad && tid < kTile) {
      const int i = SA::piece_start(row0, tid, p.M) + (tid & 3);
      if (i >= row0 + (tid & ~3)) {
        float th = p.theta_bias[i], vel = MOM ? p.velocity_bias[i] : 0.f;
        apply_update<MOM>(th, vel, bgsum, *opt);
        p.theta_bias[i] = th;
        if (MOM) p.velocity_bias[i] = vel;
      }
    }
  }
  if (MODE != MODE_WGRAD) {
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = acc2[v];
    // dgrad: the column that sits at this lane's place in the tile; of a piece moved back, the columns that an
    // earlier piece also holds are left to that one
    const int jt = wcol + (lane & 31);
    const int jc = B_MC ? SB::piece_start(col0, jt, p.N) + (jt & 3) : j;
    const bool jok = B_MC ? jc >= col0 + (jt & ~3) : j < p.N;
    if (jok) {
      float bj = 0.f;
      if (MODE == MODE_FWD && p.bias) bj = p.bias[j];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = ibase + 8 * (v / 4) + (v % 4);
        if (i >= p.M) continue;
        float val = acc[v];
        const size_t idx = (size_t)i * p.ldc + jc;
        if (MODE == MODE_FWD) {
          val += bj;
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

template <int BK, bool A_MC, bool B_MC, int MODE>
__global__ __launch_bounds__(kThreads, 2) void gemm_f32_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(16))) float lds[gemm_lds_floats<BK, A_MC, B_MC, MODE>()];
  gemm_f32_body<BK, A_MC, B_MC, MODE, 0>(p, Segments{}, (int)blockIdx.x, (int)gridDim.x, lds);
}

// An input gradient and, in front of its tiles, the classifier's parameter gradients and losses: its workgroups wait for
// memory most of the time and run beside the product's.
__global__ __launch_bounds__(kThreads, 4) void gemm_f32_dgrad_head_kernel(GemmParams p, int tiles, HeadRole head,
                                                                          Segments seg) {
  constexpr int kGemm = gemm_lds_floats<32, false, true, MODE_DGRAD>();
  __shared__ __attribute__((aligned(16))) float lds[kGemm > kHeadWgradLdsFloats ? kGemm : kHeadWgradLdsFloats];
  const int b = (int)blockIdx.x;
  if (b < head.blocks)
    head_wgrad_loss_body<float, 1>(head.p, seg, b, head.gx, lds);
  else
    gemm_f32_body<32, false, true, MODE_DGRAD, 0>(p, seg, b - head.blocks, tiles, lds);
}

// Weight gradients of several layers in ONE launch: the workgroups of the problems follow each other
// along x (problem i owns start[i] .. start[i+1]-1, one per tile).  A launch
// has a start-up and a drain during which the matrix pipes idle; run together, one problem's
// workgroups start while another's finish.  With the update, the workgroups behind the last tile update the
// classifier's parameters, whose gradients an earlier launch has left in G.
// Four workgroups per compute unit: 1024 tiles (the 3072-1024-1024 net) are then resident at once; with three, the
// last quarter of them ran by itself, one wavefront per SIMD (15 per cent slower at 480 rows).
constexpr int kMaxBatch = 8;
struct WgradBatch {
  int n;
  int start[kMaxBatch + 1];
  size_t worker_stride;
  long head_n;                 // classifier: parameters, where they start, and worker 0's gradients of them
  float* head_theta;
  float* head_velocity;
  const float* head_grad;
  GemmParams prob[kMaxBatch];
};

template <int BK, int UPD>
__global__ __launch_bounds__(kThreads, 4) void gemm_f32_wgrad_batch_kernel(WgradBatch b, Segments seg, Lambdas lam,
                                                                           Optim opt) {
  __shared__ __attribute__((aligned(16))) float lds[gemm_lds_floats<BK, true, true, MODE_WGRAD>()];
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
  const GemmParams& p = b.prob[pi];
  const int local = (int)blockIdx.x - b.start[pi];
  const int tiles = ((p.M + kTile - 1) / kTile) * ((p.N + kTile - 1) / kTile);
  gemm_f32_body<BK, true, true, MODE_WGRAD, UPD>(p, seg, local, tiles, lds, &lam, &opt);
}

template <bool A_MC, bool B_MC, int MODE>
void launch(hipStream_t st, GemmParams& p) {
  const int tiles = ((p.M + kTile - 1) / kTile) * ((p.N + kTile - 1) / kTile);
  p.xcd_remap = tiles % 8 == 0 ? 1 : 0;
  hipLaunchKernelGGL((gemm_f32_kernel<32, A_MC, B_MC, MODE>), dim3(tiles), dim3(kThreads), 0, st, p);
}

int gemm_tiles(int rows, int cols) { return ((rows + kTile - 1) / kTile) * ((cols + kTile - 1) / kTile); }

}  // namespace

void linear_fwd_f32(hipStream_t st, const float* x, const float* w, const float* bias, float* y,
                    int rows, int cin, int cout, bool relu) {
  if (linear_f32_split(rows, cout, cin)) {
    linear_fwd_f32_split(st, x, w, bias, y, rows, cin, cout, relu);
    return;
  }
  if (linear_fwd_f32_direct(st, x, w, bias, y, rows, cin, cout, relu)) return;
  if (linear_f32_small(rows, cout, cin)) {
    linear_fwd_f32_small(st, x, w, bias, y, rows, cin, cout, relu);
    return;
  }
  GemmParams p{};
  p.A = x; p.B = w; p.C = y; p.M = rows; p.N = cout; p.lda = cin; p.ldb = cin; p.ldc = cout;
  p.kred = cin; p.bias = bias; p.relu = relu ? 1 : 0;
  launch<false, false, MODE_FWD>(st, p);
}

void linear_dgrad_f32(hipStream_t st, const float* dy, const float* w, const float* mask, float* dx,
                      int rows, int cin, int cout, bool accumulate, const HeadWgradParams* head, const Segments& seg) {
  if (linear_f32_split(rows, cin, cout)) {
    if (head) head_wgrad_loss(st, false, *head, seg);
    linear_dgrad_f32_split(st, dy, w, mask, dx, rows, cin, cout, accumulate);
    return;
  }
  if (linear_dgrad_f32_direct(st, dy, w, mask, dx, rows, cin, cout, accumulate, head, seg)) return;
  if (linear_f32_small(rows, cin, cout)) {
    linear_dgrad_f32_small(st, dy, w, mask, dx, rows, cin, cout, accumulate, head, seg);
    return;
  }
  GemmParams p{};
  p.A = dy; p.B = w; p.C = dx; p.M = rows; p.N = cin; p.lda = cout; p.ldb = cin; p.ldc = cin;
  p.kred = cout; p.mask = mask; p.accumulate = accumulate ? 1 : 0;
  if (!head) {
    launch<false, true, MODE_DGRAD>(st, p);
    return;
  }
  const int tiles = gemm_tiles(p.M, p.N);
  p.xcd_remap = tiles % 8 == 0 ? 1 : 0;
  const HeadRole role = head_role(head, seg);
  hipLaunchKernelGGL(gemm_f32_dgrad_head_kernel, dim3(tiles + role.blocks), dim3(kThreads), 0, st, p, tiles, role, seg);
}

bool linear_wgrad_f32_tiled(const LinearWgradJob* jobs, int n, int rows) {
  long tiles64 = 0;
  bool tileable = rows >= 32;
  for (int i = 0; i < n; ++i) {
    tiles64 += gemm_tiles(jobs[i].cout, jobs[i].cin);
    tileable = tileable && jobs[i].cout >= 4 && jobs[i].cin >= 4;
  }
  return tileable && tiles64 >= kTiledWgradTiles;
}

void linear_wgrad_f32_batch(hipStream_t st, const LinearWgradJob* jobs, int n, size_t worker_stride,
                            const Segments& seg, const LinearWgradJob* head, const SgdArgs* sgd,
                            const KernelTimer* timer) {
  if (linear_wgrad_f32_split_shape(jobs, n, seg)) {
    linear_wgrad_f32_split(st, jobs, n, worker_stride, seg, head, sgd, timer);
    return;
  }
  const int upd = sgd ? (sgd->velocity ? 2 : 1) : 0;
  const Lambdas lam = lambdas_of(seg);
  const Optim opt = sgd ? Optim{sgd->lr, sgd->momentum, sgd->weight_decay} : Optim{0.f, 0.f, 0.f};
  const bool one = n <= kMaxBatch;
  if (timer && !one) (void)hipEventRecord(timer->start, st);
  for (int base = 0; base < n; base += kMaxBatch) {
    WgradBatch b{};
    b.n = std::min(n - base, kMaxBatch);
    b.worker_stride = worker_stride;
    for (int i = 0; i < b.n; ++i) {
      const LinearWgradJob& j = jobs[base + i];
      GemmParams& p = b.prob[i];
      p.A = j.dy; p.B = j.x; p.C = j.gw; p.M = j.cout; p.N = j.cin; p.lda = j.cout; p.ldb = j.cin; p.ldc = j.cin;
      p.c_worker_stride = worker_stride; p.bias_grad = j.gb;
      if (sgd) {
        p.theta = sgd->params + j.w_off; p.theta_bias = sgd->params + j.b_off;
        if (sgd->velocity) { p.velocity = sgd->velocity + j.w_off; p.velocity_bias = sgd->velocity + j.b_off; }
      }
      b.start[i + 1] = b.start[i] + gemm_tiles(p.M, p.N);
    }
    if (sgd && head && base + kMaxBatch >= n) {
      b.head_n = (long)head->cout * head->cin + (head->gb ? head->cout : 0);   // (the bias follows the weight)
      b.head_theta = sgd->params + head->w_off;
      if (sgd->velocity) b.head_velocity = sgd->velocity + head->w_off;
      b.head_grad = head->gw;
    }
    const dim3 grid(b.start[b.n] + (unsigned)((b.head_n + kThreads - 1) / kThreads)), block(kThreads);
#define OMNI_WGRAD(U)                                                                                              \
  if (timer && one)                                                                                                \
    hipExtLaunchKernelGGL((gemm_f32_wgrad_batch_kernel<32, U>), grid, block, 0, st, timer->start, timer->stop, 0,  \
                          b, seg, lam, opt);                                                                       \
  else                                                                                                             \
    hipLaunchKernelGGL((gemm_f32_wgrad_batch_kernel<32, U>), grid, block, 0, st, b, seg, lam, opt)
    if (upd == 0) { OMNI_WGRAD(0); }
    else if (upd == 1) { OMNI_WGRAD(1); }
    else { OMNI_WGRAD(2); }
#undef OMNI_WGRAD
  }
  if (timer && !one) (void)hipEventRecord(timer->stop, st);
}

}  // namespace omni
