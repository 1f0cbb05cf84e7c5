// Weight gradients of the bf16 convolutions: wgrad of conv_bf16.hip's list,
//
//   G_k[co][u][v][ci] = sum over worker k's rows and all positions of dY[m][co] * X[n, h*s+u-p, w*s+v-p, ci].
//
// Five forms, by shape: kernel B (any), the ring form (3x3 / stride 1 / pad 1 on maps 4, 8, 16 and 32 wide,
// conv3_wgrad_ring_device.h), kernel C (the same on wider maps), the transposing-read form (3x3 / stride 2,
// conv3_wgrad_tr_device.h) and kernel G (3 input channels).  A layer's output is small and its reduction (positions)
// long, so each worker's positions are cut into chunks, one workgroup per (tile, chunk); a worker with several chunks
// gets its partial tiles added by a second kernel in chunk order (bit-reproducible, no atomics).
//
// Weight gradients feed nothing but the update, so they need not run one by one: a launch takes the layers collected since
// the last (conv_wgrad_batch), and so does the second stage's.  At small batches a layer's launch lasts 20 us, of which
// much is start-up and drain, and every fork to a side stream costs the host about 12 us in event calls and the main
// stream 3 us: the three-layer net at 128 images was bound by exactly that (17 launches and 14 event calls, 154 us of
// host work per step).  Layers that share a launch also share the chip, so each is cut into fewer chunks, and
// fewer partial tiles travel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "bf16.h"
#include "common.h"
#include "conv3_wgrad_ring_device.h"
#include "conv3_wgrad_tr_device.h"
#include "conv_device.h"
#include "head_device.h"
#include "kernels.h"
#include "lds_barrier_device.h"
#include "lds_limit.h"
#include "quotient.h"
#include "update_device.h"
#include "wgrad_chunk.h"

namespace omni {

namespace {

constexpr int BK = 32;

// ------------------------------------------------------------------ kernel B
struct WgradParams {
  const bf16_t* dy;    // [positions][Cout]
  const bf16_t* src;   // layer input [rows][Hs][Ws][Cs]
  float* gw;           // worker w: gw + w*worker_stride, [Cout][taps][cin_real]
  float* gb;           // worker w: gb + w*worker_stride, [Cout]; may be null
  size_t worker_stride;
  int Cout, cin_real;
  ConvGeom g;          // Hp, Wp: output positions; gather as in the forward pass
  int chunk;           // positions per workgroup (multiple of BK)
  float* partial;      // [(tile * total_chunks + chunk index)][TM*TN*16][256] (+ bias tail)
};

template <int TM, int TN>
__device__ __forceinline__ void wgrad_general_body(const WgradParams& p, const Segments& seg, const Chunk& ck, int tile,
                                                   unsigned char* smem) {
  constexpr int BM = 64 * TM, BN = 64 * TN;   // output tile: BM output channels x BN reduction columns
  // 80-byte rows: a fragment is one aligned 16-byte read, and the 16 consecutive rows that sixteen
  // lanes read spread evenly over the 64 read banks.  Rows 8 apart would land in the same banks, and
  // the channel pieces that the lanes of one transposing write cover are 8 rows apart: every group of
  // 16 rows is moved by another 32 bytes, so that the pieces of a write spread over the four quarters
  // of the 32 write banks while no fragment read is disturbed.  (72-byte rows with 8-byte fragment
  // reads measured 70 % of their LDS cycles as bank conflicts.)
  constexpr int kRow = BK + 8;
  auto roff = [](int row) { return row * kRow + (row >> 4) * 16; };
  constexpr int kA = BM * kRow + BM, kB = BN * kRow + BN;
  constexpr int kTileFloats = TM * TN * 16 * kThreads;
  bf16_t* const lds = reinterpret_cast<bf16_t*>(smem);
  int* const tab = reinterpret_cast<int*>(smem + 2 * (kA + kB) * sizeof(bf16_t));   // [kMaxPieces]
  auto sA = [&](int s) { return lds + s * (kA + kB); };
  auto sB = [&](int s) { return lds + s * (kA + kB) + kA; };

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ConvGeom g = p.g;
  const int N = g.K;
  const int tiles_n = (N + BN - 1) / BN;
  const int tile_m = tile / tiles_n, tile_n = tile % tiles_n;
  const int row0 = tile_m * BM, col0 = tile_n * BN;
  const int wrow = (wave >> 1) * 32 * TM, wcol = (wave & 1) * 32 * TN;
  const int wk = ck.wk, chunk_idx = ck.idx, nchunks = ck.n;
  const int hw = g.Hp * g.Wp;
  const int mbeg = seg.off[wk] * hw + chunk_idx * p.chunk;
  const int mend = min(seg.off[wk + 1] * hw, mbeg + p.chunk);

  build_tap_table(tab, g, tid);
  __syncthreads();

  // Staging tasks.  The first BM threads: (BM/8) output-channel pieces x 8
  // groups of 4 positions of dY.  The next BN threads: (BN/8) reduction pieces x
  // 8 groups of the gathered input.
  const bool is_a = tid < BM;
  const int t2 = is_a ? tid : tid - BM;
  const int npiece = is_a ? BM / 8 : BN / 8;
  // consecutive lanes: 8 pieces (128 contiguous bytes of one position), then 2 position groups, then
  // the second 8 pieces if there are 16, then the remaining position groups
  const int piece = npiece == 8 ? (t2 & 7) : ((t2 & 7) | ((t2 >> 1) & 8));
  const int mg = npiece == 8 ? (t2 >> 3) : (((t2 >> 3) & 1) | ((t2 >> 4) & 6));
  const bool task = tid < BM + BN;   // (mg < 8 follows)
  int bu = 0, bv = 0, bci = 0;
  bool piece_ok;
  if (is_a) {
    piece_ok = row0 + piece * 8 < p.Cout;
  } else {
    const int q = (col0 >> 3) + piece;
    piece_ok = q * 8 < g.K;
    const int t = tab[piece_ok ? q : 0];
    bu = t & 15; bv = (t >> 4) & 15; bci = t >> 8;
  }

  v16f acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
  const bool want_bias = p.gb != nullptr && tile_n == 0;
  float bsum = 0.f;

  u32x4 r[4];
  // Loads never branch and their base pointer is chosen once (a guarded load, or a pointer
  // re-selected per load, makes the compiler wait for every load before issuing the next):
  // an absent piece is read from a page of zeros.
  const bf16_t* const base = is_a ? p.dy : p.src;
  const bf16_t* const zp = static_cast<const bf16_t*>(g.zero);
  auto load_slab = [&](int m0) {
    const int mfirst = m0 + mg * 4;
    int n = 0, h = 0, w = 0;
    decode_pos(g, min(mfirst, max(mend - 1, 0)), n, h, w);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = mfirst + q;
      const long oa = (long)m * p.Cout + row0 + piece * 8;
      const long ob = gather_offset(g, n, h, w, bu, bv, bci);
      const long o = is_a ? oa : ob;
      const bool in = task && piece_ok && m < mend && o >= 0;
      if (++w == g.Wp) { w = 0; if (++h == g.Hp) { h = 0; ++n; } }
      r[q] = *reinterpret_cast<const u32x4*>(in ? base + o : zp);
    }
  };
  auto store_slab = [&](int s) {
    if (!task) return;
    const u32x4* c = r;
    bf16_t* dst = (is_a ? sA(s) : sB(s)) + roff(piece * 8) + mg * 4;
    // word d of piece q holds channels 2d (low half) and 2d+1 (high half) of position q
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      u32x2 lo, hi;
      lo[0] = (c[0][d] & 0xFFFFu) | (c[1][d] << 16);
      lo[1] = (c[2][d] & 0xFFFFu) | (c[3][d] << 16);
      hi[0] = (c[0][d] >> 16) | (c[1][d] & 0xFFFF0000u);
      hi[1] = (c[2][d] >> 16) | (c[3][d] & 0xFFFF0000u);
      *reinterpret_cast<u32x2*>(dst + (2 * d) * kRow) = lo;
      *reinterpret_cast<u32x2*>(dst + (2 * d + 1) * kRow) = hi;
    }
  };
  auto frag = [&](const bf16_t* base, int row, int ko) {
    return as_bf16x8(*reinterpret_cast<const u32x4*>(base + roff(row) + ko));
  };

  const int nslab = (mend - mbeg + BK - 1) / BK;
  load_slab(mbeg);
  store_slab(0);
  __syncthreads();
  for (int s = 0; s < nslab; ++s) {
    const int cur = s & 1;
    load_slab(s + 1 < nslab ? mbeg + (s + 1) * BK : mend);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 fa[TM], fb[TN];
      const int ko = ks * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int a = 0; a < TM; ++a) fa[a] = frag(sA(cur), wrow + a * 32 + (lane & 31), ko);
#pragma unroll
      for (int b = 0; b < TN; ++b) fb[b] = frag(sB(cur), wcol + b * 32 + (lane & 31), ko);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    if (want_bias && tid < BM) {
      // rows of the dY slab are output channels: their sums over positions are the bias gradient
      const u32x4* rowp = reinterpret_cast<const u32x4*>(sA(cur) + roff(tid));
#pragma unroll
      for (int d = 0; d < BK / 8; ++d) {
        const u32x4 q = rowp[d];
#pragma unroll
        for (int e = 0; e < 4; ++e) bsum += bf16_lo(q[e]) + bf16_hi(q[e]);
      }
    }
    if (s + 1 < nslab) {
      store_slab(cur ^ 1);
      __syncthreads();
    }
  }

  // ---- a worker cut into several chunks: park the partial tile, a second kernel adds them up
  if (nchunks > 1) {
    float* mine = p.partial + ((size_t)tile * ck.total + ck.row) * (kTileFloats + BM);
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) mine[((a * TN + b) * 16 + v) * kThreads + tid] = acc[a][b][v];
    if (tid < BM) mine[kTileFloats + tid] = bsum;
    return;
  }

  const int taps = g.ks * g.ks;
  float* gw = p.gw + (size_t)wk * p.worker_stride;
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int kcol = col0 + wcol + b * 32 + (lane & 31);
    if (kcol >= g.K) continue;
    const int tap = kcol / g.Cs, ci = kcol - tap * g.Cs;
    if (ci >= p.cin_real) continue;   // padding channels of the first layer
    const int colreal = tap * p.cin_real + ci;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int co = row0 + wrow + a * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4);
        if (co < p.Cout) gw[(size_t)co * (taps * p.cin_real) + colreal] = acc[a][b][v];
      }
  }
  if (want_bias && tid < BM && row0 + tid < p.Cout) p.gb[(size_t)wk * p.worker_stride + row0 + tid] = bsum;
}

// Second stage of a chunked wgrad: one workgroup per (tile, worker, one of TM*TN*16 register slots).
// Each thread owns the same (output channel, reduction column) as the thread of
// the first stage that held this slot, and adds the worker's chunks in chunk
// order (fixed order: results repeat bit for bit).
template <int TM, int TN>
__device__ __forceinline__ void wgrad_general_reduce(const WgradParams& p, const Chunk& ck, int tile, int slot, float* lds) {
  constexpr int BM = 64 * TM, BN = 64 * TN;
  constexpr int kTileFloats = TM * TN * 16 * kThreads;
  const int wk = ck.wk, nchunks = ck.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ConvGeom g = p.g;
  const int tiles_n = (g.K + BN - 1) / BN;
  const int tile_m = tile / tiles_n, tile_n = tile % tiles_n;
  const int row0 = tile_m * BM, col0 = tile_n * BN;
  const int wrow = (wave >> 1) * 32 * TM, wcol = (wave & 1) * 32 * TN;
  const float* all = p.partial + ((size_t)tile * ck.total + ck.row) * (kTileFloats + BM);
  const size_t stride = kTileFloats + BM;

  // Each wavefront adds a quarter of the chunks (16-byte loads, 8 in flight), then
  // the four quarter sums are added in wavefront order.
  float (*red)[kThreads] = reinterpret_cast<float (*)[kThreads]>(lds);   // [4]
  {
    const float* src = all + (size_t)slot * kThreads + lane * 4;
    const int cbeg = wave * nchunks / 4, cend = (wave + 1) * nchunks / 4;
    v4f acc4 = {0.f, 0.f, 0.f, 0.f};
    int c = cbeg;
    for (; c + 8 <= cend; c += 8) {
      v4f t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = *reinterpret_cast<const v4f*>(src + (size_t)(c + u) * stride);
#pragma unroll
      for (int u = 0; u < 8; ++u) acc4 += t[u];
    }
    for (; c < cend; ++c) acc4 += *reinterpret_cast<const v4f*>(src + (size_t)c * stride);
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][lane * 4 + e] = acc4[e];
  }
  __syncthreads();
  const float s0 = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  const int a = slot / (TN * 16), b = (slot / 16) % TN, v = slot % 16;
  const int kcol = col0 + wcol + b * 32 + (lane & 31);
  const int co = row0 + wrow + a * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4);
  const int taps = g.ks * g.ks;
  if (kcol < g.K && co < p.Cout) {
    const int tap = kcol / g.Cs, ci = kcol - tap * g.Cs;
    if (ci < p.cin_real)
      p.gw[(size_t)wk * p.worker_stride + (size_t)co * (taps * p.cin_real) + tap * p.cin_real + ci] = s0;
  }
  if (slot == 0 && p.gb != nullptr && tile_n == 0 && tid < BM && row0 + tid < p.Cout) {
    float bs = 0.f;                      // eight loads in flight, additions in chunk order
    const float* bsrc = all + kTileFloats + tid;
    int c = 0;
    for (; c + 8 <= nchunks; c += 8) {
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = bsrc[(size_t)(c + u) * stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) bs += t[u];
    }
    for (; c < nchunks; ++c) bs += bsrc[(size_t)c * stride];
    p.gb[(size_t)wk * p.worker_stride + row0 + tid] = bs;
  }
}


// ------------------------------------------------------------------ kernel C
// Weight gradient of 3x3, stride-1, pad-1 convolutions on maps that the ring form does not take: 64 and 128 wide (narrower ones where
// units of a great many rows have no reciprocal).
// Kernel B treats the nine filter taps as nine independent column blocks: the
// input is fetched and transposed nine times and dY once per column tile, and at
// 64 channels that memory traffic, not the matrix pipe, sets the pace.  Here a
// workgroup owns 64 output channels x 64 input channels x ALL nine taps and walks
// through units of 128 output positions (a strip of rows of one image, or a few
// whole small images):
//   * dY^T [64 co][128 positions] and the input patch X^T [64 ci][rows+2][W+16]
//     (with its zero halo) are transposed into LDS ONCE per unit;
//   * the B operand of tap (u, v) is the patch shifted by (u-1) rows and (v-1)
//     columns: the row shift is an address offset; the column shift of one
//     element is made in registers from the aligned 16-byte read and its two
//     neighbour words (v_alignbit), so one LDS read serves three taps;
//   * each wavefront holds 32 co x 32 ci x 9 taps = nine accumulator blocks.
// Units never straddle workers; a worker's units are cut into chunks, one
// workgroup per (tile, chunk), partial tiles are added by a second kernel in
// chunk order (bit-reproducible, no atomics).
constexpr int kSA = 2 * kUnit + 16;                 // bytes between channels of dY^T
// Channel rows 8 apart are a multiple of 32 words apart: the eight channel octets that sixteen lanes
// of one transposing write cover would all land in the same banks (measured: 87 % of the LDS cycles
// of the staging writes were bank conflicts).  Every group of eight rows is therefore moved by
// another 16 bytes, which makes the writes conflict-free.  The price is on the other side: the 16
// consecutive rows that sixteen lanes of a 16-byte fragment read cover now overlap in one bank group
// (measured: fragment reads conflict-free before, 63 % conflict cycles after), still far fewer
// conflict cycles in all (5.6e7 -> 1.5e7 per launch on 64-channel 32 x 32 maps together with the
// lane swaps below).  A skew per sixteen rows leaves the reads alone but brings the write conflicts
// back (2.4e7 in all).
constexpr int kSkewPad = 128;   // room for the skew of 64 rows (7 x 16 bytes), kept a multiple of 128
__device__ inline int row_skew(int row) { return (row >> 3) * 16; }
// four positions x eight channels (c[q] = the 16-byte piece of position q) -> eight
// channel rows of four positions each
__device__ inline void transpose_store(const u32x4 c[4], unsigned char* dst, int row_bytes) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    u32x2 lo, hi;
    lo[0] = (c[0][d] & 0xFFFFu) | (c[1][d] << 16);
    lo[1] = (c[2][d] & 0xFFFFu) | (c[3][d] << 16);
    hi[0] = (c[0][d] >> 16) | (c[1][d] & 0xFFFF0000u);
    hi[1] = (c[2][d] >> 16) | (c[3][d] & 0xFFFF0000u);
    *reinterpret_cast<u32x2*>(dst + (2 * d) * row_bytes) = lo;
    *reinterpret_cast<u32x2*>(dst + (2 * d + 1) * row_bytes) = hi;
  }
}

// The three taps of one filter row: q holds the window's 8 columns (two per word), pl the word
// before it (its upper half is the column to the left), pn the word after (lower half: to the right).
__device__ inline void wgrad3_taps(v16f (&acc)[9], int du, const bf16x8 fa, const u32x4 q, uint32_t pl, uint32_t pn) {
  const uint32_t m01 = __builtin_amdgcn_alignbit(q[1], q[0], 16);
  const uint32_t m12 = __builtin_amdgcn_alignbit(q[2], q[1], 16);
  const uint32_t m23 = __builtin_amdgcn_alignbit(q[3], q[2], 16);
  const u32x4 left = {__builtin_amdgcn_alignbit(q[0], pl, 16), m01, m12, m23};
  const u32x4 right = {m01, m12, m23, __builtin_amdgcn_alignbit(pn, q[3], 16)};
  acc[du * 3 + 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, as_bf16x8(left), acc[du * 3 + 0], 0, 0, 0);
  acc[du * 3 + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, as_bf16x8(q), acc[du * 3 + 1], 0, 0, 0);
  acc[du * 3 + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, as_bf16x8(right), acc[du * 3 + 2], 0, 0, 0);
}

__device__ __forceinline__ void wgrad3_body(const Wgrad3Params& p, const Chunk& ck, int tile, unsigned char* smem3) {
  constexpr int KSTEPS = kUnit / 16;   // reduction steps per unit
  unsigned char* sA = smem3;                 // dY^T: 64 rows of kSA bytes
  unsigned char* sX = smem3 + 64 * kSA + kSkewPad;   // X^T: 64 rows of p.SX bytes (both arrays: + the skew)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 31, h = lane >> 5;
  const int tiles_ci = (p.Cin + 63) / 64, tile_co = tile / tiles_ci;
  const int co0 = tile_co * 64, ci0 = (tile - tile_co * tiles_ci) * 64;
  const int wco = (wave >> 1) * 32, wci = (wave & 1) * 32;
  const int H = p.H, W = p.W, R = p.R;
  const int wk = ck.wk, chunk_idx = ck.idx, nchunks = ck.n;
  const int bk = ck.end - ck.beg;
  const int upi = p.nimg == 1 ? H / R : 1;   // units per image when a unit is part of one image
  const int units_k = p.nimg == 1 ? bk * upi : (bk + p.nimg - 1) >> p.nimg_log;
  const int ubeg = chunk_idx * p.upc, uend = min(units_k, ubeg + p.upc);

  // ---- staging tasks (the same for every unit, relative to the unit's first image and row)
  // dY: 8 channel octets x 32 groups of 4 positions
  auto over_r = [&](int rows) { return (int)(((uint32_t)rows * p.by_r) >> 16); };
  const int a_oct = tid & 7;
  int a_rel, a_il;
  {
    const int p0 = 4 * (tid >> 3), rr = p0 / W, w = p0 - rr * W;
    a_il = over_r(rr);
    a_rel = (a_il * H + (rr - a_il * R)) * W + w;
  }
  const bool a_chan_ok = co0 + 8 * a_oct < p.Cout;
  unsigned char* a_dst = sA + (8 * a_oct) * kSA + row_skew(8 * a_oct) + 8 * (tid >> 3);
  // X: channel octets x (W/4 groups of 4 columns) x patch rows: at most two tasks a thread, three on 128-wide maps (a row of one
  // image and its neighbours) and for one row of 64
  const int wq = W >> 2;
  const int ntasks = p.prows * wq * 8;
  struct Task {
    int rel, il, rr, dst;
    bool here;
  };
  auto task_at = [&](int x) {
    const bool in = x < ntasks;
    const int oct = in ? x & 7 : 0, g = in ? x >> 3 : 0;
    const int pr = g / wq, wg = g - pr * wq;
    const int il = (int)(((uint32_t)pr * p.by_patch) >> 16), rr = pr - il * (R + 2);   // input row = first row + rr - 1
    return Task{((il * H + rr - 1) * W + 4 * wg) * p.Cin + 8 * oct, il, rr, (8 * oct) * p.SX + row_skew(8 * oct) + (pr * p.Wp + 4 * wg + 8) * 2,
                in && ci0 + 8 * oct < p.Cin};   // false: no such piece, or a channel octet past the end
  };
  const Task task[2] = {task_at(tid), task_at(tid + kThreads)};

  u32x4 ra[4], rx[2][4];
  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);
  // first image and row of unit u; units are loaded one after the other
  int img_at, row_at;
  {
    const int img = quotient(ubeg, p.by_upi, upi);
    img_at = ck.beg + (p.nimg == 1 ? img : ubeg << p.nimg_log);
    row_at = p.nimg == 1 ? (ubeg - img * upi) * R : 0;
  }
  // Loads never branch (a guarded load makes the compiler wait for each group before the
  // next): an absent piece is read from a page of zeros.
  auto images = [&]() { return p.nimg == 1 ? 1 : min(p.nimg, ck.end - img_at); };
  auto load_task = [&](const Task& t, u32x4 (&to)[4]) {
    const int row = row_at + t.rr - 1;
    const bool in = t.here && t.il < images() && row >= 0 && row < H;
    const bf16_t* src = in ? p.src + (((long)img_at * H + row_at) * W * p.Cin + t.rel + ci0) : zp;
    const int st = in ? p.Cin : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) to[q] = *reinterpret_cast<const u32x4*>(src + q * st);
  };
  auto load_unit = [&]() {
    const int nvalid = images();
    const long base_pos = ((long)img_at * H + row_at) * W;
    {
      const bool in = a_chan_ok && a_il < nvalid;
      const bf16_t* src = in ? p.dy + ((base_pos + a_rel) * p.Cout + co0 + 8 * a_oct) : zp;
      const int st = in ? p.Cout : 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) ra[q] = *reinterpret_cast<const u32x4*>(src + q * st);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) load_task(task[t], rx[t]);
  };
  auto next_unit = [&]() {
    row_at += R;
    if (row_at >= H) {
      row_at = 0;
      img_at += p.nimg;
    }
  };
  auto store_unit = [&]() {
    if (a_chan_ok) transpose_store(ra, a_dst, kSA);
#pragma unroll
    for (int t = 0; t < 2; ++t)
      if (task[t].here) transpose_store(rx[t], sX + task[t].dst, p.SX);   // (else no such patch piece, or channels that stay zero)
    // the third task, whose pieces no registers are left for while the unit before is multiplied.  (128 images of 64 channels on 128x128,
    // whole step: 3.13 ms, 3.15 with registers for it, of which eleven spill, and 4.10 in kernel B.)
    if (ntasks > 2 * kThreads) {
      const Task third = task_at(tid + 2 * kThreads);
      load_task(third, rx[0]);
      if (third.here) transpose_store(rx[0], sX + third.dst, p.SX);
    }
  };
  load_unit();   // (every chunk has a unit)

  // The halo columns of the patch are never written again: they stay zero.  So do the rows of
  // channels past the end of the tensor (their staging tasks are skipped altogether).
  for (int i = tid * 16; i < 64 * kSA + 64 * p.SX + 2 * kSkewPad; i += kThreads * 16)
    *reinterpret_cast<u32x4*>(smem3 + i) = u32x4{0u, 0u, 0u, 0u};

  // ---- fragment addresses: k-step ks covers positions 16 ks .. 16 ks + 15, this lane the 8 at 16 ks + 8 h
  int offB[KSTEPS];
#pragma unroll
  for (int i = 0; i < KSTEPS; ++i) {
    const int pos = (2 * i + h) * 8, rr = pos / W, w0 = pos - rr * W;
    const int il = over_r(rr);
    offB[i] = ((il * (R + 2) + (rr - il * R)) * p.Wp + w0 + 8) * 2;
  }
  const unsigned char* a_frag = sA + (wco + j) * kSA + row_skew(wco + j) + h * 16;
  const unsigned char* x_frag = sX + (wci + j) * p.SX + row_skew(wci + j);
  const int row_shift = p.Wp * 2;

  v16f acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
  const bool want_bias = p.gb != nullptr && ci0 == 0;
  float bsum = 0.f;

  for (int u = ubeg; u < uend; ++u) {
    __syncthreads();   // the previous unit's fragments have been read (and, first time, the zero fill is done)
    store_unit();
    __syncthreads();
    if (u + 1 < uend) next_unit();
    load_unit();   // always issued: in flight during the MFMAs below
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const bf16x8 fa = as_bf16x8(*reinterpret_cast<const u32x4*>(a_frag + ks * 32));
#pragma unroll
      for (int du = 0; du < 3; ++du) {
        const unsigned char* xb = x_frag + offB[ks] + du * row_shift;
        wgrad3_taps(acc, du, fa, *reinterpret_cast<const u32x4*>(xb), *reinterpret_cast<const uint32_t*>(xb - 4),
                    *reinterpret_cast<const uint32_t*>(xb + 16));
      }
    }
    if (want_bias) {
      // rows of dY^T are output channels: their sums over positions are the bias gradient; every
      // wavefront adds a quarter of the unit's positions (one wavefront walking all 128 was a serial
      // chain of a thousand cycles per unit that the other three waited for at the next barrier)
      const uint32_t* rowp = reinterpret_cast<const uint32_t*>(sA + lane * kSA + row_skew(lane)) + wave * (kUnit / 8);
#pragma unroll
      for (int d = 0; d < kUnit / 8; ++d) bsum += bf16_lo(rowp[d]) + bf16_hi(rowp[d]);
    }
  }
  if (want_bias) {
    // the four quarters meet, in wavefront order
    __syncthreads();
    float* quarter = reinterpret_cast<float*>(sA);
    quarter[tid] = bsum;
    __syncthreads();
    if (tid < 64) bsum = ((quarter[tid] + quarter[64 + tid]) + quarter[128 + tid]) + quarter[192 + tid];
  }
  const int ci = ci0 + wci + j;
  const bool holds = ci < p.cin_real;
  if (nchunks > 1) {
    float* mine = p.partial + ((size_t)tile * ck.total + ck.row) * kTile3Stride;
    if (holds) park3(mine, acc, wave, lane);             // (the second stage reads the same lanes only)
    if (tid < 64) mine[kTile3Floats + tid] = bsum;
    return;
  }
  float* gw = p.gw + (size_t)wk * p.worker_stride;
  if (holds) {
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int co = co0 + wco + 8 * (v / 4) + 4 * h + (v % 4);
        if (co < p.Cout) gw[((size_t)co * 9 + t) * p.cin_real + ci] = acc[t][v];
      }
  }
  if (want_bias && tid < 64 && co0 + tid < p.Cout) p.gb[(size_t)wk * p.worker_stride + co0 + tid] = bsum;
}

// ---- the order in which a worker's chunks are added, in the second stage and in the one with the update alike (their results are
// the same bits): four quarters of the chunks, each in chunk order, one after the other; the bias gradients in one chain.
__device__ inline int quarter_chunks(int n) { return (n + 3) >> 2; }
template <typename V>
__device__ inline V add_quarters(V a, V b, V c, V d) { return ((a + b) + c) + d; }
// The sum of n values `stride` floats apart, eight loads in flight.
template <typename V = float>
__device__ inline V chain_of(const float* src, int n, size_t stride) {
  V s = {};
  for (int c = 0; c < n; c += 8) {
    V t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = *reinterpret_cast<const V*>(src + (size_t)min(c + u, n - 1) * stride);
#pragma unroll
    for (int u = 0; u < 8; ++u) s = c + u < n ? s + t[u] : s;
  }
  return s;
}

// Kernel C's and the ring form's element of a tile: register v of one tap and quadrant, as lane `lane` held it.
struct Place3 {
  int co0, ci0, wci, co, ci;
  size_t at;      // in the weight
  bool in;
};
__device__ __forceinline__ Place3 wgrad3_place(const Wgrad3Params& p, int tile, int quad, int tap, int v, int lane) {
  const int tiles_ci = (p.Cin + 63) / 64, row = tile / tiles_ci;
  const int co0 = row * 64, ci0 = (tile - row * tiles_ci) * 64, wci = (quad & 1) * 32;
  const int co = co0 + (quad >> 1) * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4), ci = ci0 + wci + (lane & 31);
  return Place3{co0, ci0, wci, co, ci, ((size_t)co * 9 + tap) * p.cin_real + ci, co < p.Cout && ci < p.cin_real};
}

// Second stage: one workgroup per (tile, worker, 9 taps x 4 register quarters x 4 tile quadrants); it
// owns the (output channel, input channel) pairs one wavefront of the first stage held; each of its
// four wavefronts adds a quarter of the worker's chunks (eight 16-byte loads in flight), the quarters meet in LDS.
__device__ __forceinline__ void wgrad3_reduce(const Wgrad3Params& p, const Chunk& ck, int tile, int z, float* lds) {
  v4f (*part)[64] = reinterpret_cast<v4f (*)[64]>(lds);   // [4]
  const int wk = ck.wk, nchunks = ck.n;
  const int quad = z & 3, vq = (z >> 2) & 3, tap = z >> 4;
  const int tid = threadIdx.x, lane = tid & 63, sub = tid >> 6;
  const float* all = p.partial + ((size_t)tile * ck.total + ck.row) * kTile3Stride;
  const int per = quarter_chunks(nchunks);
  const int c0 = min(sub * per, nchunks), c1 = min(c0 + per, nchunks);
  const Place3 first = wgrad3_place(p, tile, quad, tap, 4 * vq, lane);
  v4f s = {0.f, 0.f, 0.f, 0.f};
  if (first.ci < p.cin_real)
    s = chain_of<v4f>(all + (size_t)c0 * kTile3Stride + partial3_at(tap, vq, quad, lane), c1 - c0, kTile3Stride);
  part[sub][lane] = s;
  __syncthreads();
  if (sub == 0) {
    const v4f tot = add_quarters(part[0][lane], part[1][lane], part[2][lane], part[3][lane]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const Place3 pl = wgrad3_place(p, tile, quad, tap, 4 * vq + e, lane);
      if (pl.in) p.gw[(size_t)wk * p.worker_stride + pl.at] = tot[e];
    }
  }
  const int co = first.co0 + tid;
  if (z == 0 && p.gb != nullptr && first.ci0 == 0 && tid < 64 && co < p.Cout)
    p.gb[(size_t)wk * p.worker_stride + co] = chain_of(all + kTile3Floats + tid, nchunks, kTile3Stride);
}


// ---------------------------------------------------------------------------------------------
// Kernel G: weight gradient of the first layer -- 3 input channels stored as 8, 3x3 / stride 1 /
// pad 1, maps 32 wide, at most 64 output channels.
//
//   G_k[co][u][v][ci] = sum over the positions of worker k of dY[pos][co] * X[pos + (u-1, v-1)][ci]
//
// As a matrix product the output is tiny (Cout x 27) and the reduction (all positions) is
// everything, so the layer is bound by reading dY and X once: what kernel C spends on a 64 x 64
// channel tile that is 15/16 empty, and on parking and re-reading such tiles, is avoided by giving
// the product its own shape: rows = output channels (32 per block), columns = (tap, channel) pairs and, behind
// them, a column of ones (its product is the bias gradient): 28 of 32 for three channels, 37 of 64 for four;
// reduction = positions, 16 per v_mfma_f32_32x32x16_bf16.  dY is staged as it arrives ([pos][channel], 16-byte pieces) and
// transposed by the LDS read (tr_pair).  X is staged as planes, one per channel and horizontal tap, each
// shifted by its tap: the eight positions of an operand are then one aligned 16-byte read for every tap, and the
// shifting costs nine 2-byte writes per pixel once instead of eight 2-byte reads per operand and lane, which bound this
// kernel: 2048 images, 32 channels, pooled, with the classifier's gradients (17 us of it) in the same launch 60 -> 40 us, 64
// channels not pooled 97 -> 76 us (3.7 TB/s).  A workgroup walks units of 4 image rows (128 positions) of one
// worker; its four wavefronts split the positions of a unit and keep whole accumulators, which are
// added through LDS at the end.  Chunks of one worker are added by a second small kernel in chunk
// order (fixed summation order; no atomics).
struct Wgrad1Params {
  const bf16_t* dy;     // [rows][H][32][Cout]
  const bf16_t* src;    // [rows][H][32][8]
  float* gw;            // worker k at gw + k * worker_stride, layout [Cout][3][3][cin_real]
  float* gb;            // may be null
  size_t worker_stride;
  int Cout, cin_real, H;
  int upc;              // units per chunk
  float* partial;       // [chunk][MB * NB * 16 * 64] accumulator images
  // POOLED kernels: dy is not read; it is rebuilt from the gradient of the 2 x 2 max pooling that
  // follows the layer and the pooling's codes (one byte per pooled element: which input took it)
  const bf16_t* dpool;  // [rows][H/2][16][Cout]
  const uint8_t* code;  // [rows][H/2][16][Cout]
  int raw3;             // src is [rows][H][32][3]: a pixel is three 2-byte loads
  uint32_t by_ppp, by_cin, by_upi;   // reciprocal_below of Cout / 8, cin_real and H / 4
};
constexpr int kG_W = 32, kG_R = 4, kG_Unit = kG_W * kG_R;        // 128 positions
constexpr int kG_PatchRows = kG_R + 2;
// Bytes of a plane [patch row][32]: 32 more than the data, so that the planes' reads spread over the banks.
constexpr int kG_Plane = kG_PatchRows * kG_W * 2 + 32;

// Where channel octet oct of a position lies in the staged dY strip.  Every other pair of 128-byte rows has its halves
// swapped: the four rows of a transposing read then fill the 64 banks once, as 64-byte rows do by themselves.
template <int MB>
__device__ inline int wgrad1_y_offset(int pos, int oct) {
  return MB == 2 ? pos * 128 + ((oct * 16) ^ ((pos & 2) << 5)) : pos * 64 + oct * 16;
}
__host__ __device__ inline int wgrad1_col_blocks(int cin_real) { return cin_real * 9 + 1 > 32 ? 2 : 1; }
__host__ __device__ constexpr int wgrad1_stage_bytes(int mb, int cin_real) { return kG_Unit * 64 * mb + 3 * cin_real * kG_Plane; }

// Where the value of accumulator register v of lane `lane` in block (mb, nb) goes in G, null where it is none's (gw, gb: the worker's)
__device__ inline float* wgrad1_place(const Wgrad1Params& p, float* gw, float* gb, int mb, int nb, int v, int lane) {
  const int co = mb * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4), col = nb * 32 + (lane & 31), cols = 9 * p.cin_real;
  if (co >= p.Cout) return nullptr;
  return col < cols ? gw + (size_t)co * cols + col : col == cols && gb != nullptr ? gb + co : nullptr;
}

// POOLED: the layer's output gradient was never written.  Every position takes the gradient of its
// pooling window where the window's code names it and zero elsewhere: 16 + 8 bytes of pooled data
// per two positions instead of 16 bytes of a full-resolution tensor each that a pooling-backward pass would
// have had to write first.
template <int MB, int NB, bool POOLED>
__device__ __forceinline__ void wgrad1_body(const Wgrad1Params& p, const Segments& seg, const Chunk& ck,
                                            unsigned char* smemg) {
  constexpr int SY = 64 * MB;                              // bytes per position of the staged dY strip
  const int cin = p.cin_real;
  const int stage_bytes = wgrad1_stage_bytes(MB, cin);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  const int wk = ck.wk, chunk_idx = ck.idx, nchunks = ck.n;
  const int upi = p.H / kG_R;                              // units per image
  const int units = (ck.end - ck.beg) * upi;
  const int ubeg = chunk_idx * p.upc, uend = min(units, ubeg + p.upc);

  // zero both stages once (halo columns of the planes and absent channels of dY are never written again)
  for (int i = tid * 16; i < 2 * stage_bytes; i += kThreads * 16) *reinterpret_cast<u32x4*>(smemg + i) = u32x4{0, 0, 0, 0};
  __syncthreads();

  // staging tasks of this thread: dY pieces (16 bytes = 8 channels of one position; POOLED: of a pooled position, for
  // the two positions of one row of its window), one pixel of the patch
  const int ppp = p.Cout / 8;                              // pieces per position
  constexpr int kY = POOLED ? MB : 2 * MB;                 // Cout <= 32 MB
  const int ny = (POOLED ? kG_Unit / 2 : kG_Unit) * ppp;
  // two units are on their way at a time (one ahead, a trip of the loop lasted a memory round trip: 1.9 us of 0.5)
  u32x4 ry[2][kY];
  u32x2 rk[2][kY];                                          // POOLED: the codes that go with ry
  // a thread's pieces are the same in every unit: where each comes from (relative to the unit) and goes
  int ysrc[kY], ydst[kY];
  uint32_t yslot[kY];                                       // POOLED: place in the window of the first of the two positions
#pragma unroll
  for (int i = 0; i < kY; ++i) {
    const int q = min(tid + kThreads * i, ny - 1);         // surplus slots re-read the last piece
    const int at = ppp == 1 ? q : quotient(q, p.by_ppp, ppp), oct = q - at * ppp;
    if (POOLED) {                                           // at = row of the unit, window along it
      const int row = at >> 4, pc = at & 15;
      ydst[i] = wgrad1_y_offset<MB>(row * kG_W + 2 * pc, oct);
      ysrc[i] = ((row >> 1) * (kG_W / 2) + pc) * p.Cout + oct * 8;
      yslot[i] = (uint32_t)(row & 1) * 2;
    } else {
      ydst[i] = wgrad1_y_offset<MB>(at, oct);
      ysrc[i] = q * 8;
      yslot[i] = 0;
    }
  }
  const bool has_x = tid < kG_PatchRows * kG_W;
  const int xr = tid / kG_W, xc = tid % kG_W;              // patch row 0..5 (image row strip*4 - 1 + xr), column
  uint32_t rx[2][2];                                        // up to four channels of the pixel
  constexpr int kPlaneEnd = kG_PatchRows * kG_W;
  const int xat[3] = {xc < kG_W - 1 ? xr * kG_W + xc + 1 : kPlaneEnd, xr * kG_W + xc, xc > 0 ? xr * kG_W + xc - 1 : kPlaneEnd};
  // the unit that is fetched next: its image and first row
  int fu = ubeg, fimg, frow;
  {
    const int at = quotient(ubeg, p.by_upi, upi);
    fimg = __builtin_amdgcn_readfirstlane(ck.beg + at);
    frow = __builtin_amdgcn_readfirstlane((ubeg - at * upi) * kG_R);
  }
  auto fetch = [&](int s) {
    const int img = fimg, row0 = frow;
    if (fu < uend - 1) {                                    // (past the last unit: that one again)
      ++fu;
      frow += kG_R;
      if (frow == p.H) {
        frow = 0;
        ++fimg;
      }
    }
    if constexpr (POOLED) {
      const size_t ubase = ((size_t)(img * (p.H >> 1) + (row0 >> 1)) * (kG_W / 2)) * p.Cout;
#pragma unroll
      for (int i = 0; i < kY; ++i) {
        ry[s][i] = *reinterpret_cast<const u32x4*>(p.dpool + ubase + ysrc[i]);
        rk[s][i] = *reinterpret_cast<const u32x2*>(p.code + ubase + ysrc[i]);
      }
    } else {
      const bf16_t* ybase = p.dy + ((size_t)(img * p.H + row0) * kG_W) * p.Cout;
#pragma unroll
      for (int i = 0; i < kY; ++i) ry[s][i] = *reinterpret_cast<const u32x4*>(ybase + ysrc[i]);
    }
    const int grow = row0 - 1 + xr;
    const bool in = has_x && grow >= 0 && grow < p.H;
    const bf16_t* xp = p.src + ((size_t)(img * p.H + (in ? grow : 0)) * kG_W + xc) * (p.raw3 ? 3 : 8);
    if (!has_x) xp = p.src;
    if (p.raw3) {
      rx[s][0] = (uint32_t)xp[0] | ((uint32_t)xp[1] << 16);
      rx[s][1] = xp[2];
    } else {
      const u32x2 t = *reinterpret_cast<const u32x2*>(xp);
      rx[s][0] = t[0];
      rx[s][1] = t[1];
    }
    if (!in) rx[s][0] = rx[s][1] = 0u;
  };
  auto stash = [&](int s) {
    unsigned char* sY = smemg + s * stage_bytes;
    unsigned char* sX = sY + kG_Unit * SY;
#pragma unroll
    for (int i = 0; i < kY; ++i) {
      if (tid + kThreads * i >= ny) continue;
      unsigned char* d = sY + ydst[i];
      if constexpr (POOLED) {
        // keep a channel's gradient where its code names this position's place in the window
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const uint32_t slot = yslot[i] + half;
          u32x4 w;
#pragma unroll
          for (int d2 = 0; d2 < 4; ++d2) {
            const uint32_t kk = rk[s][i][d2 >> 1] >> (16 * (d2 & 1));
            const uint32_t lo = (kk & 0xFFu) == slot ? 0x0000FFFFu : 0u;
            const uint32_t hi = ((kk >> 8) & 0xFFu) == slot ? 0xFFFF0000u : 0u;
            w[d2] = ry[s][i][d2] & (lo | hi);
          }
          *reinterpret_cast<u32x4*>(d + half * SY) = w;
        }
      } else {
        *reinterpret_cast<u32x4*>(d) = ry[s][i];
      }
    }
    if (has_x) {
      // plane v * cin + ci holds X[row][column + v - 1][ci]
      // (a tap whose column lies outside goes to the plane's end, which nothing reads: no branches)
      bf16_t* d = reinterpret_cast<bf16_t*>(sX);
#pragma unroll
      for (int ci = 0; ci < 4; ++ci) {
        if (ci >= cin) break;
        const bf16_t val = (bf16_t)(rx[s][ci >> 1] >> (16 * (ci & 1)));
        d[ci * (kG_Plane / 2) + xat[0]] = val;
        d[(cin + ci) * (kG_Plane / 2) + xat[1]] = val;
        d[(2 * cin + ci) * (kG_Plane / 2) + xat[2]] = val;
      }
    }
  };

  // fragment addressing.  A: see wgrad_tr_body (conv3_wgrad_tr_device.h); rows = output channels of block mb.  B: lane
  // supplies column lane % 32 of block nb at positions 8 * (lane / 32) .. + 7 of the sixteen.
  const int kg = lane >> 5, jl = lane & 31;
  const int g = lane >> 4, sl = lane & 15;
  const int abase = (8 * (g >> 1) + (sl >> 2)) * SY + (16 * (g & 1) + 4 * (sl & 3)) * 2, aswap = MB == 2 ? (sl & 8) << 3 : 0;
  int bbase[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int col = nb * 32 + jl;
    const int tap = col < 9 * cin ? (cin == 1 ? col : quotient(col, p.by_cin, cin)) : 0;
    const int ci = col < 9 * cin ? col - tap * cin : 0;   // (absent columns are not stored)
    bbase[nb] = (tap % 3 * cin + ci) * kG_Plane + (tap / 3 * kG_W + 8 * kg) * 2;
  }
  const int ones_nb = 9 * cin / 32;
  const bool ones = jl == 9 * cin % 32;

  v16f acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  // one unit from stage S; the next one's pieces (set 1 - S) go to the other stage, those of the one after it set out
  auto unit = [&](auto which) {
    constexpr int S = decltype(which)::value;
    fetch(S);
    const unsigned char* sY = smemg + S * stage_bytes;
    const unsigned char* sX = sY + kG_Unit * SY;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kb = wave + 4 * h;                          // 16 positions: image row kb/2, columns (kb%2)*16 ...
      const unsigned char* ya = sY + kb * 16 * SY + abase;
      const unsigned char* xb = sX + ((kb >> 1) * kG_W + (kb & 1) * 16) * 2;
      bf16x8 fa[MB], fb[NB];
#pragma unroll
      for (int a = 0; a < MB; ++a) fa[a] = tr_pair(ya + ((a * 64) ^ aswap), ya + ((a * 64) ^ aswap) + 4 * SY);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        u32x4 w = *reinterpret_cast<const u32x4*>(xb + bbase[b]);
        if (b == ones_nb && ones) w = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
        fb[b] = as_bf16x8(w);
      }
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    stash(S ^ 1);                                           // (past the last unit: never read)
    lds_barrier();                                          // (the loads of the unit after it stay under way: with no branches in
                                                            // stash() and no division in fetch() a step of 128 images 82.1 -> 81.5 us)
  };
  if (ubeg < uend) {
    fetch(0);
    fetch(1);
    stash(0);
    lds_barrier();
    for (int u = ubeg; u < uend; u += 2) {
      unit(std::integral_constant<int, 0>{});
      if (u + 1 < uend) unit(std::integral_constant<int, 1>{});
    }
  }

  // add the four wavefronts' accumulators (wavefront order) and write the chunk's result
  float* red = reinterpret_cast<float*>(smemg);            // [4][MB*NB*16][64] floats = 64 KB at most
  constexpr int kImg = MB * NB * 16 * 64;
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[wave * kImg + ((a * NB + b) * 16 + v) * 64 + lane] = acc[a][b][v];
  __syncthreads();
  float* gw = p.gw + (size_t)wk * p.worker_stride;
  float* gb = p.gb ? p.gb + (size_t)wk * p.worker_stride : nullptr;
  for (int e = tid; e < kImg; e += kThreads) {
    const float val = ((red[e] + red[kImg + e]) + red[2 * kImg + e]) + red[3 * kImg + e];
    if (nchunks > 1) {
      p.partial[(size_t)ck.row * kImg + e] = val;
    } else {
      const int blk = e / (16 * 64), v = (e / 64) % 16, l = e % 64;
      float* const to = wgrad1_place(p, gw, gb, blk / NB, blk % NB, v, l);
      if (to) *to = val;
    }
  }
}

// One workgroup per worker and 64 of the MB * NB * 1024 accumulator elements; each of the four wavefronts adds a
// quarter of the worker's chunks (eight loads in flight), the quarters meet in LDS.
__device__ __forceinline__ void wgrad1_reduce(const Wgrad1Params& p, const Chunk& ck, int z, float* lds) {
  const int NB = wgrad1_col_blocks(p.cin_real);
  const int kImg = (p.Cout > 32 ? 2 : 1) * NB * 16 * 64;
  float (*part)[64] = reinterpret_cast<float (*)[64]>(lds);   // [4]
  const int wk = ck.wk, nchunks = ck.n;
  const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int e = z * 64 + lane;
  const int per = quarter_chunks(nchunks);
  const int c0 = min(sub * per, nchunks), c1 = min(c0 + per, nchunks);
  part[sub][lane] = chain_of(p.partial + (size_t)(ck.row + c0) * kImg + e, c1 - c0, kImg);
  __syncthreads();
  if (sub != 0) return;
  const float s = add_quarters(part[0][lane], part[1][lane], part[2][lane], part[3][lane]);
  float* gw = p.gw + (size_t)wk * p.worker_stride;
  float* gb = p.gb ? p.gb + (size_t)wk * p.worker_stride : nullptr;
  const int blk = e / (16 * 64), v = (e / 64) % 16, l = e % 64;
  float* const to = wgrad1_place(p, gw, gb, blk / NB, blk % NB, v, l);
  if (to) *to = s;
}

// ------------------------------------------------------------------ launches of several layers
enum WgradKind {
  kGeneral11, kGeneral12, kGeneral21, kGeneral22, kPatch4, kPatch8, kPatch16, kPatch32, kPatchAny, kPatch8Narrow, kPatch16Narrow,
  kPatch32Narrow, kStride2, kFirst
};

struct BatchJob {
  int kind;
  int tiles;             // workgroups of the first stage: tiles x chunks, of the second: tiles x workers x slots
  int slots;
  uint32_t by_tiles, by_workers;   // reciprocal_below
  int32_t chunk[OMNI_MAX_WORKERS + 1];   // first chunk of every worker; chunk[K] = all
  union {
    WgradParams general;
    Wgrad3Params patch;
    TrParams stride2;
    Wgrad1Params first;
  };
};
constexpr int kBatchJobs = 6;   // the table travels in the kernel arguments
struct BatchTable {
  int n;
  int first[kBatchJobs];   // the jobs' first_block (second stage: first_reduce), in one line of the arguments
  BatchJob job[kBatchJobs];
};

// (A line of arguments that nothing has touched takes 640 cycles: the lanes fetch chunks and rows of all workers at once, before
// anything that depends on them.)
struct ChunkTable {
  int chunk, off, chunk64, off64;
};
__device__ inline ChunkTable chunk_table(const BatchJob& job, const Segments& seg) {
  static_assert(OMNI_MAX_WORKERS == 64, "one lane per worker");
  const int lane = threadIdx.x & 63;
  return ChunkTable{job.chunk[lane], seg.off[lane], job.chunk[64], seg.off[64]};
}
__device__ inline Chunk chunk_at(const ChunkTable& t, int K, int row) {
  const int wk = __popcll(__ballot((int)(threadIdx.x & 63) < K && t.chunk <= row)) - 1;
  auto chunk = [&](int k) { return k < 64 ? __builtin_amdgcn_readlane(t.chunk, k & 63) : t.chunk64; };
  auto off = [&](int k) { return k < 64 ? __builtin_amdgcn_readlane(t.off, k & 63) : t.off64; };
  const int first = chunk(wk);
  return Chunk{wk, row - first, chunk(wk + 1) - first, row, chunk(K), off(wk), off(wk + 1)};
}
__device__ inline int job_at(const BatchTable& tab, int block) {
  int e = 0;
#pragma unroll
  for (int i = 1; i < kBatchJobs; ++i) e += i < tab.n && block >= tab.first[i] ? 1 : 0;
  return e;
}

__global__ __launch_bounds__(kThreads, 2) void wgrad_batch_kernel(BatchTable tab, Segments seg) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int e = job_at(tab, (int)blockIdx.x);
  const BatchJob& job = tab.job[e];
  const ChunkTable table = chunk_table(job, seg);
  const int local = (int)blockIdx.x - tab.first[e], row = quotient(local, job.by_tiles, job.tiles);
  const int tile = local - row * job.tiles;
  const Chunk ck = chunk_at(table, seg.K, row);
  const Wgrad3Params patch = job.patch;   // (read together; and with a read per use the compiler copies the whole table into scratch)
  switch (job.kind) {
    case kGeneral11: wgrad_general_body<1, 1>(job.general, seg, ck, tile, smem); break;
    case kGeneral12: wgrad_general_body<1, 2>(job.general, seg, ck, tile, smem); break;
    case kGeneral21: wgrad_general_body<2, 1>(job.general, seg, ck, tile, smem); break;
    case kGeneral22: wgrad_general_body<2, 2>(job.general, seg, ck, tile, smem); break;
    case kPatch4: wgrad3_ring_body<4, false, 4>(patch, ck, tile, smem); break;
    case kPatch8: wgrad3_ring_body<8, false, 4>(patch, ck, tile, smem); break;
    case kPatch16: wgrad3_ring_body<16, false, 4>(patch, ck, tile, smem); break;
    case kPatch32: wgrad3_ring_body<32, false, 4>(patch, ck, tile, smem); break;
    case kPatchAny: wgrad3_body(patch, ck, tile, smem); break;
    case kPatch8Narrow: wgrad3_ring_body<8, true, 4>(patch, ck, tile, smem); break;
    case kPatch16Narrow: wgrad3_ring_body<16, true, 4>(patch, ck, tile, smem); break;
    case kPatch32Narrow: wgrad3_ring_body<32, true, 4>(patch, ck, tile, smem); break;
    case kStride2: wgrad_tr_body<2>(job.stride2, seg, ck, tile, smem); break;
    default: break;   // (kFirst has launches of its own)
  }
}

// The same for layers of the ring form alone, with eight wavefronts to a workgroup.  Two share a block of the output and are added in
// LDS: a compute unit is as full as with two workgroups of four, for half the partial tiles in memory.  For launches with nothing
// beside them: these workgroups leave no registers to another kernel's.
__global__ __launch_bounds__(2 * kThreads, 2) void wgrad_ring_kernel(BatchTable tab, Segments seg) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int e = job_at(tab, (int)blockIdx.x);
  const BatchJob& job = tab.job[e];
  const ChunkTable table = chunk_table(job, seg);
  const Wgrad3Params patch = job.patch;   // (all of the arguments on their way together)
  const int local = (int)blockIdx.x - tab.first[e], row = exact_quotient(local, job.by_tiles);
  const int tile = local - row * job.tiles;
  const Chunk ck = chunk_at(table, seg.K, row);
  switch (job.kind) {
    case kPatch4: wgrad3_ring_body<4, false, 8>(patch, ck, tile, smem); break;
    case kPatch8: wgrad3_ring_body<8, false, 8>(patch, ck, tile, smem); break;
    case kPatch16: wgrad3_ring_body<16, false, 8>(patch, ck, tile, smem); break;
    case kPatch32: wgrad3_ring_body<32, false, 8>(patch, ck, tile, smem); break;
    case kPatch8Narrow: wgrad3_ring_body<8, true, 8>(patch, ck, tile, smem); break;
    case kPatch16Narrow: wgrad3_ring_body<16, true, 8>(patch, ck, tile, smem); break;
    case kPatch32Narrow: wgrad3_ring_body<32, true, 8>(patch, ck, tile, smem); break;
    default: break;
  }
}

// The chunks of a layer on the network input and, in front of them, the classifier's parameter gradients and the losses:
// both are short of registers and LDS and long on memory waits, and run four workgroups to a compute unit (in the launch
// above they would be two).
template <int MB, int NB, bool POOLED>
__global__ __launch_bounds__(kThreads, 2) void wgrad_light_kernel(BatchJob job, HeadWgradParams head, int head_x, int head_blocks,
                                                                  Segments seg) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int b = (int)blockIdx.x;
  if (b < head_blocks) {
    head_wgrad_loss_body<bf16_t, 2>(head, seg, b, head_x, reinterpret_cast<float*>(smem));
    return;
  }
  wgrad1_body<MB, NB, POOLED>(job.first, seg, chunk_at(chunk_table(job, seg), seg.K, b - head_blocks), smem);
}

// Second stage of the layers in which some worker has more than one chunk.
__global__ __launch_bounds__(kThreads) void wgrad_reduce_kernel(BatchTable tab, Segments seg) {
  __shared__ __attribute__((aligned(16))) float lds[4 * kThreads];
  const int e = job_at(tab, (int)blockIdx.x);
  const BatchJob& job = tab.job[e];
  const int local = (int)blockIdx.x - tab.first[e];
  const int rest = quotient(local, job.by_tiles, job.tiles), tile = local - rest * job.tiles;
  const int slot = quotient(rest, job.by_workers, seg.K), wk = rest - slot * seg.K;
  const Chunk ck{wk, 0, job.chunk[wk + 1] - job.chunk[wk], job.chunk[wk], job.chunk[seg.K], 0, 0};
  if (ck.n <= 1) return;   // written directly by the first stage
  switch (job.kind) {
    case kGeneral11: wgrad_general_reduce<1, 1>(job.general, ck, tile, slot, lds); break;
    case kGeneral12: wgrad_general_reduce<1, 2>(job.general, ck, tile, slot, lds); break;
    case kGeneral21: wgrad_general_reduce<2, 1>(job.general, ck, tile, slot, lds); break;
    case kGeneral22: wgrad_general_reduce<2, 2>(job.general, ck, tile, slot, lds); break;
    case kStride2: wgrad_tr_reduce(job.stride2, ck, tile, slot); break;
    case kFirst: wgrad1_reduce(job.first, ck, slot, lds); break;
    default: wgrad3_reduce(job.patch, ck, tile, slot, lds); break;
  }
}

// ---- the second stage with the update: all workers' gradients of an element meet in one workgroup, which applies their weighted
// sum (chunks and workers in the order of the two launches it stands for: the same bits).  For steps whose weight gradients are
// one call; kernel C's and the ring form's layers and the first layer's, the parameters of all others follow from G.
struct UpdateTo {
  float* theta;
  float* vel;
  float* G;            // worker 0's gradients of all parameters
  size_t stride;
};
constexpr int kRestRanges = 2 * kBatchJobs + 1;
struct RestTable {     // parameters whose gradients are complete in G already: beg[i] .. end[i] - 1 from workgroup first[i] on
  int n;
  int32_t first[kRestRanges], beg[kRestRanges], end[kRestRanges];
};

template <bool MOM>
__device__ inline void update_one(const UpdateTo& to, size_t at, float th, float ve, float g, const Optim& opt) {
  apply_update<MOM>(th, ve, g, opt);
  to.theta[at] = th;
  if (MOM) to.vel[at] = ve;
}

// The second stage's sum of n values `stride` apart, by one wavefront: the four quarters side by side.
template <typename V = float>
__device__ inline V sum_quarters(const float* src, int n, size_t stride) {
  constexpr int U = 4;                             // sixteen loads in flight
  const int per = quarter_chunks(n);
  V a[4] = {};
  for (int i = 0; i < per; i += U) {
    V t[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) t[u][q] = *reinterpret_cast<const V*>(src + (size_t)min(q * per + i + u, n - 1) * stride);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = i + u < per && q * per + i + u < n ? a[q] + t[u][q] : a[q];
  }
  return add_quarters(a[0], a[1], a[2], a[3]);
}

// Kernel C and the ring form: a workgroup has four registers of one tap and tile quadrant (the pairs one wavefront of the first stage held) or, in the
// last slot, a tile's biases; its NW wavefronts take a worker each, or take turns.  lds: 256 floats per worker.
constexpr int kUpdateSlots3 = 9 * 4 * 4 + 1;
template <bool MOM, int NW>
__device__ __forceinline__ void wgrad3_update(const Wgrad3Params& p, const BatchJob& job, int tile, int z, const Segments& seg,
                                              const Lambdas& lam, const Optim& opt, const UpdateTo& to, float* lds) {
  const bool bias = z == kUpdateSlots3 - 1;
  const int quad = bias ? 0 : z & 3, vq = bias ? 0 : (z >> 2) & 3, tap = bias ? 0 : z >> 4;
  const int tid = threadIdx.x, lane = tid & 63, sub = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = seg.K;
  const Place3 first = wgrad3_place(p, tile, quad, tap, 4 * vq, lane);
  const float* const tiles = p.partial + (size_t)tile * job.chunk[K] * kTile3Stride;
  if (bias) {
    if (p.gb == nullptr || first.ci0 != 0) return;
    const int co = min(first.co0 + lane, p.Cout - 1);
    const bool in = first.co0 + lane < p.Cout;
    const size_t mine = (size_t)(p.gb - to.G) + co;
    const float th = to.theta[mine], ve = MOM ? to.vel[mine] : 0.f;
    for (int wk = sub; wk < K; wk += NW) {
      const int c0 = job.chunk[wk], n = job.chunk[wk + 1] - c0;
      float* const gb = p.gb + (size_t)wk * p.worker_stride + co;
      float s;
      if (n > 1) {
        s = chain_of(tiles + (size_t)c0 * kTile3Stride + kTile3Floats + co - first.co0, n, kTile3Stride);
        if (in) *gb = s;
      } else {
        s = *gb;
      }
      lds[wk * 64 + lane] = s;
    }
    __syncthreads();
    if (sub != 0 || !in) return;
    float g = 0.f;
    for (int k = 0; k < K; ++k) g += lam.v[k] * lds[k * 64 + lane];
    update_one<MOM>(to, mine, th, ve, g, opt);
    return;
  }
  if (first.ci0 + first.wci >= p.cin_real) return; // (nothing there)
  // wavefront sub < 4 applies the update of register 4 vq + sub
  const Place3 own = wgrad3_place(p, tile, quad, tap, 4 * vq + (sub & 3), lane);
  const size_t mine = (size_t)(p.gw - to.G) + (own.in ? own.at : 0);
  const float th = to.theta[mine], ve = MOM ? to.vel[mine] : 0.f;
  v4f* const sums = reinterpret_cast<v4f*>(lds);   // [worker][lane]
  for (int wk = sub; wk < K; wk += NW) {
    const int c0 = job.chunk[wk], n = job.chunk[wk + 1] - c0;
    float* const gw = p.gw + (size_t)wk * p.worker_stride;
    v4f s = {0.f, 0.f, 0.f, 0.f};
    if (n > 1) s = sum_quarters<v4f>(tiles + (size_t)c0 * kTile3Stride + partial3_at(tap, vq, quad, lane), n, kTile3Stride);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const Place3 pl = wgrad3_place(p, tile, quad, tap, 4 * vq + e, lane);
      if (!pl.in) continue;
      if (n > 1) gw[pl.at] = s[e];
      else s[e] = gw[pl.at];                       // (written by the first stage)
    }
    sums[wk * 64 + lane] = s;
  }
  __syncthreads();
  if (sub < 4 && own.in) {
    float g = 0.f;
    for (int k = 0; k < K; ++k) g += lam.v[k] * lds[(k * 64 + lane) * 4 + sub];
    update_one<MOM>(to, mine, th, ve, g, opt);
  }
}

// Kernel G: 64 accumulator elements per workgroup.
template <bool MOM, int NW>
__device__ __forceinline__ void wgrad1_update(const Wgrad1Params& p, const BatchJob& job, int z, const Segments& seg, const Lambdas& lam,
                                              const Optim& opt, const UpdateTo& to, float* lds) {
  const int NB = wgrad1_col_blocks(p.cin_real), MB = p.Cout > 32 ? 2 : 1, kImg = MB * NB * 16 * 64, K = seg.K;
  const int lane = threadIdx.x & 63, sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e = z * 64 + lane, blk = z >> 4, v = z & 15, mb = NB == 2 ? blk >> 1 : blk, nb = NB == 2 ? blk & 1 : 0;
  float* const place = wgrad1_place(p, p.gw, p.gb, mb, nb, v, lane);
  const bool in = place != nullptr;
  float* const g0 = in ? place : p.gw;             // worker 0's
  const size_t at = (size_t)(g0 - to.G);
  const float th = to.theta[at], ve = MOM ? to.vel[at] : 0.f;
  for (int wk = sub; wk < K; wk += NW) {
    const int c0 = job.chunk[wk], n = job.chunk[wk + 1] - c0;
    float s;
    if (n > 1) {
      s = sum_quarters(p.partial + (size_t)c0 * kImg + e, n, kImg);
      if (in) g0[(size_t)wk * p.worker_stride] = s;
    } else {
      s = g0[(size_t)wk * p.worker_stride];
    }
    lds[wk * 64 + lane] = s;
  }
  __syncthreads();
  if (sub == 0 && in) {
    float g = 0.f;
    for (int k = 0; k < K; ++k) g += lam.v[k] * lds[k * 64 + lane];
    update_one<MOM>(to, at, th, ve, g, opt);
  }
}

// Workgroups below rest.first[0]: the table's layers, tiles x slots each; then the rest, an element per thread.  The wavefronts take
// the workers in turn, a round trip to memory each (update_wavefronts).
// Measured, 3-32-64-128: 1024 images, eight workers, 20.3 us with a register per workgroup, 256 bytes a load and twice the partial
// tiles; 17.0 with half the tiles, 13.6 with four registers and eight wavefronts.  128 images, four workers, 10.6 -> 9.7.
template <bool MOM, int NW>
__global__ __launch_bounds__(NW * 64) void wgrad_update_kernel(BatchTable tab, RestTable rest, Segments seg, Lambdas lam, Optim opt,
                                                                UpdateTo to) {
  extern __shared__ __attribute__((aligned(16))) float lds_update[];
  const int b = (int)blockIdx.x;
  if (b >= rest.first[0]) {
    int i = 0;
#pragma unroll
    for (int k = 1; k < kRestRanges; ++k) i += k < rest.n && b >= rest.first[k] ? 1 : 0;
    const int at = rest.beg[i] + (b - rest.first[i]) * NW * 64 + (int)threadIdx.x;
    if (at >= rest.end[i]) return;
    const float th = to.theta[at], ve = MOM ? to.vel[at] : 0.f;
    float g = 0.f;
    for (int k0 = 0; k0 < seg.K; k0 += 8) {        // eight loads in flight
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = to.G[(size_t)min(k0 + u, seg.K - 1) * to.stride + at];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k0 + u < seg.K) g += lam.v[k0 + u] * t[u];
    }
    update_one<MOM>(to, at, th, ve, g, opt);
    return;
  }
  const int e = job_at(tab, b);
  const BatchJob& job = tab.job[e];
  const int local = b - tab.first[e], slot = quotient(local, job.by_tiles, job.tiles), tile = local - slot * job.tiles;
  if (job.kind == kFirst) wgrad1_update<MOM, NW>(job.first, job, slot, seg, lam, opt, to, lds_update);
  else wgrad3_update<MOM, NW>(job.patch, job, tile, slot, seg, lam, opt, to, lds_update);
}

// ------------------------------------------------------------------ planning
// A layer's form, and how its positions may be cut: units per worker, the fewest units a chunk should have, how much
// scratch a (tile, chunk) takes.
struct Plan {
  BatchJob job;
  long units[OMNI_MAX_WORKERS], total_units;
  long min_upc, upc_step;   // units per chunk: at least, and a multiple of
  int alone;                // workgroups aimed at where the layer has a launch to itself
  size_t slot_floats, lds;
  double work;              // microseconds of one workgroup walking all of it, at two workgroups per compute unit (see plan_patch)
  double ring_work;         // ... in a launch of layers of the ring form alone
};

void count_units(Plan& pl, const Segments& seg, int per_image, int images_per_unit) {
  pl.total_units = 0;
  for (int k = 0; k < seg.K; ++k) {
    const long bk = seg.off[k + 1] - seg.off[k];
    pl.units[k] = images_per_unit == 1 ? bk * per_image : (bk + images_per_unit - 1) / images_per_unit;
    pl.total_units += pl.units[k];
  }
}

bool first_layer_shape(int Cout, int cin_real, const ConvGeom& g) {
  const int H = g.Hs, W = g.Ws;
  if (g.ks != 3 || g.stride != 1 || g.pad != 1 || g.transposed || g.Hp != H || g.Wp != W) return false;
  if (g.Cs != 8 || cin_real > 4 || cin_real < 1 || W != kG_W || H % kG_R != 0) return false;
  return Cout % 8 == 0 && Cout >= 8 && Cout <= 64;
}

// The first layer (3 channels stored as 8) on 32-wide maps: kernel G.
bool plan_first(Plan& pl, const ConvWgradJob& j, size_t worker_stride, const Segments& seg) {
  const ConvGeom& g = j.g;
  if (!first_layer_shape(j.Cout, j.cin_real, g)) return false;
  const int mb = j.Cout > 32 ? 2 : 1;
  Wgrad1Params p{};
  p.dy = j.dy; p.src = j.src; p.gw = j.gw; p.gb = j.gb; p.worker_stride = worker_stride;
  p.Cout = j.Cout; p.cin_real = j.cin_real; p.H = g.Hs; p.dpool = j.dpool; p.code = j.pool_code; p.raw3 = g.raw3;
  const int nb = wgrad1_col_blocks(j.cin_real);
  pl.job.kind = kFirst; pl.job.tiles = 1; pl.job.slots = mb * nb * 16; pl.job.first = p;
  count_units(pl, seg, g.Hs / kG_R, 1);
  // about four workgroups per compute unit, at least 4 units each
  const int upi = g.Hs / kG_R;
  pl.job.first.by_ppp = reciprocal_below(j.Cout / 8, kG_Unit * (j.Cout / 8));   // (of a unit's pieces)
  pl.job.first.by_cin = reciprocal_below(j.cin_real, 32 * nb);                   // (of a column)
  pl.job.first.by_upi = reciprocal_below(upi, (uint64_t)seg.off[seg.K] * upi);
  pl.min_upc = 4; pl.upc_step = 1; pl.alone = std::max(64, 1024 - seg.K);
  pl.slot_floats = (size_t)mb * nb * 16 * 64;
  pl.lds = std::max((size_t)2 * wgrad1_stage_bytes(mb, j.cin_real), 4 * pl.slot_floats * sizeof(float));
  return true;
}

// 3x3 / stride 1 / pad 1 and a map whose rows tile into units of 128 positions: the ring form or kernel C.  (Also
// for a first layer with 8 stored channels on maps that are not 32 wide, which kernel G does not
// take: most of the 64-channel tile is then empty.)
bool plan_patch(Plan& pl, const ConvWgradJob& j, size_t worker_stride, const Segments& seg) {
  const ConvGeom& g = j.g;
  const int H = g.Hs, W = g.Ws;
  if (g.ks != 3 || g.stride != 1 || g.pad != 1 || g.transposed || g.Hp != H || g.Wp != W) return false;
  if (j.cin_real > g.Cs || g.Cs % 8 != 0 || j.Cout % 8 != 0) return false;
  const bool w4 = W == 4 && H == 4;
  if (!w4 && (W % 8 != 0 || W > kUnit || kUnit % W != 0)) return false;
  const int R = std::min(H, kUnit / W);
  if (H % R != 0 || kUnit % (R * W) != 0) return false;
  const int nimg = kUnit / (R * W);
  if (nimg > 1 && R != H) return false;
  Wgrad3Params p{};
  p.dy = j.dy; p.src = j.src; p.gw = j.gw; p.gb = j.gb; p.worker_stride = worker_stride;
  p.Cout = j.Cout; p.Cin = g.Cs; p.cin_real = j.cin_real; p.H = H; p.W = W; p.R = R; p.nimg = nimg;
  p.Wp = W + 16; p.prows = nimg * (R + 2);
  // channel stride of X^T in 4-byte words must be 4 mod 8: 16 lanes x 16 bytes then cover all 64 banks
  int words = p.prows * p.Wp / 2;
  words += (4 - words % 8 + 8) % 8;
  p.SX = words * 4;
  p.zero = g.zero;
  while ((1 << p.nimg_log) < nimg) ++p.nimg_log;   // (nimg divides 128)
  auto reciprocal16 = [](int d) { return (uint32_t)(((1 << 16) + d - 1) / d); };   // (exact: rows below 2^9, divisors up to 130)
  p.by_r = reciprocal16(R); p.by_patch = reciprocal16(R + 2);
  p.by_upi = nimg == 1 ? reciprocal_below(H / R, (uint64_t)seg.off[seg.K] * (H / R) + 1) : 0;
  // the form with rings wants whole images of 32 positions (4-wide maps: a step is two images)
  const bool ring = w4 || ((W == 8 || W == 16 || W == 32) && H * W % 32 == 0 && (p.by_upi || nimg > 1 || R == H));
  // at most 32 input channels: half of a 64 x 64 tile would be empty
  const bool narrow = ring && !w4 && g.Cs <= 32;
  pl.lds = ring ? ring_lds_bytes(narrow, 4) : (size_t)64 * kSA + (size_t)64 * p.SX + 2 * kSkewPad;   // + the row skew of both arrays
  if (!ring && pl.lds > 80 * 1024) return false;
  pl.job.kind = !ring ? kPatchAny : w4 ? kPatch4 : W == 8 ? (narrow ? kPatch8Narrow : kPatch8)
              : W == 16 ? (narrow ? kPatch16Narrow : kPatch16) : (narrow ? kPatch32Narrow : kPatch32);
  pl.job.tiles = ((j.Cout + 63) / 64) * ((g.Cs + 63) / 64);
  pl.job.slots = 144; pl.job.patch = p;
  count_units(pl, seg, H / R, nimg);
  // about one workgroup per compute unit (every chunk parks a partial tile of up to 148 KB that the second stage reads
  // back: with 512 chunks that traffic outweighed the extra parallelism, measured -2 % on the three-layer CNN's step).
  // At least four units a chunk (with two, ResNet-18 shape, 20 images: second stages 33 -> 69 us, step 870 -> 925; see plan_batch).
  pl.min_upc = 4; pl.upc_step = 1; pl.alone = 256;
  pl.slot_floats = kTile3Stride;
  // The ring form's units take 2.6 us (narrow: 1.3).  Beside layers of other forms it has the share of a launch that kernel C's 4.5
  // (3.0; 6.0 on 4-wide maps) would give: with its own its chains were up to twice as long, and a gradient's error up to 1.17 times
  // that of kernel C (256 channels on 8x8, 1024 images, eight workers: 5.9e-7 and 5.1e-7).  It costs the step of the ResNet-18 shape 0 to 1.5
  // per cent (256 images 2190 us and 2223, 128, 512, 1024 and 2048 the same).
  pl.work = (w4 ? 6.0 : narrow ? 3.0 : 4.5) * pl.job.tiles * pl.total_units;
  pl.ring_work = (narrow ? 1.3 : 2.6) * pl.job.tiles * pl.total_units;
  return true;
}

// 3x3 / stride 2 / pad 1 without bias: the transposing-read form.  (Its body takes any stride; stride-1 layers have the ring form, which
// reads its operands in the same way from streams that need no patch.)
bool plan_stride2(Plan& pl, const ConvWgradJob& j, size_t worker_stride, const Segments& seg) {
  const ConvGeom& g = j.g;
  const int S = g.stride, Ho = g.Hp, Wo = g.Wp, H = g.Hs, W = g.Ws;
  if (j.gb || g.ks != 3 || g.pad != 1 || g.transposed || g.raw3 || S != 2) return false;
  if (H != S * Ho || W != S * Wo || g.Cs % 8 != 0 || j.Cout % 8 != 0 || j.cin_real > g.Cs) return false;
  // (a reduction step of sixteen positions must lie inside one map row or be made of whole rows of one image)
  if (Wo < 4 || Wo > kTrUnit || (Wo % 16 != 0 && 16 % Wo != 0)) return false;
  const int R = std::min(Ho, kTrUnit / Wo);
  if (Ho % R != 0 || kTrUnit % (R * Wo) != 0 || (R * Wo) % 16 != 0) return false;
  const int nimg = kTrUnit / (R * Wo);
  if ((nimg > 1 && R != Ho) || nimg > 15) return false;
  const int PR = S * (R - 1) + 3, PW = S * (Wo - 1) + 3;
  const int npatch = nimg * PR * PW;
  if (npatch * 4 > kNX * kThreads) return false;
  if ((long)g.rows * H * W * g.Cs >= (1L << 31) || (long)g.rows * Ho * Wo * j.Cout >= (1L << 31)) return false;
  TrParams p{};
  p.dy = j.dy; p.src = j.src; p.gw = j.gw; p.worker_stride = worker_stride;
  p.Cout = j.Cout; p.Cin = g.Cs; p.cin_real = j.cin_real; p.Ho = Ho; p.Wo = Wo; p.H = H; p.W = W;
  p.R = R; p.nimg = nimg; p.PR = PR; p.PW = PW; p.zero = g.zero;
  pl.job.kind = kStride2;
  pl.job.tiles = ((j.Cout + kCo - 1) / kCo) * ((g.Cs + kCi - 1) / kCi);
  pl.job.slots = 36; pl.job.stride2 = p;
  count_units(pl, seg, Ho / R, nimg);
  pl.min_upc = 8; pl.upc_step = 1; pl.alone = 512;   // about two workgroups per compute unit
  pl.slot_floats = kTrTileFloats;
  pl.lds = (size_t)kTrUnit * kTrSA + (size_t)npatch * 80;   // (80 bytes per patch position at stride 2: see the body)
  pl.work = 3.5 * pl.job.tiles * pl.total_units;
  return true;
}

void plan_general(Plan& pl, const ConvWgradJob& j, size_t worker_stride, const Segments& seg) {
  const ConvGeom& g = j.g;
  WgradParams p{};
  p.dy = j.dy; p.src = j.src; p.gw = j.gw; p.gb = j.gb; p.worker_stride = worker_stride;
  p.Cout = j.Cout; p.cin_real = j.cin_real; p.g = g;
  const int tm = j.Cout > 64 ? 2 : 1, tn = g.K > 64 ? 2 : 1;
  pl.job.kind = tm == 1 ? (tn == 1 ? kGeneral11 : kGeneral12) : (tn == 1 ? kGeneral21 : kGeneral22);
  pl.job.tiles = ((j.Cout + 64 * tm - 1) / (64 * tm)) * ((g.K + 64 * tn - 1) / (64 * tn));
  pl.job.slots = tm * tn * 16; pl.job.general = p;
  count_units(pl, seg, g.Hp * g.Wp, 1);   // (a unit is a position, a chunk whole slabs of BK)
  // about two workgroups per compute unit (the reduction is where the parallelism of a small filter bank lies; every
  // extra chunk is a partial tile written and read back), at least 8 slabs each
  pl.min_upc = 8 * BK; pl.upc_step = BK; pl.alone = 512;
  pl.slot_floats = (size_t)tm * tn * 16 * kThreads + 64 * tm;
  pl.lds = (size_t)2 * (64 * tm + 64 * tn) * (BK + 9) * sizeof(bf16_t) + kMaxPieces * sizeof(int);
  pl.work = 1.7 / BK * pl.job.tiles * pl.total_units;
}

// Cuts the layer's positions for about `aim` workgroups within `budget` floats of scratch.
void cut_chunks(Plan& pl, const Segments& seg, long aim, size_t budget) {
  BatchJob& job = pl.job;
  const long want = std::max<long>(1, aim / job.tiles);
  long upc = std::max((pl.total_units + want - 1) / want, pl.min_upc);
  upc = (upc + pl.upc_step - 1) / pl.upc_step * pl.upc_step;
  for (;;) {
    int acc = 0;
    for (int k = 0; k < seg.K; ++k) {
      job.chunk[k] = acc;
      acc += (int)((pl.units[k] + upc - 1) / upc);
    }
    job.chunk[seg.K] = acc;
    // one chunk per worker needs no scratch (every workgroup writes its worker's gradient itself); otherwise the partial
    // tiles must fit, and the workgroups should keep to their share of the chip: a few extra ones would run as
    // a second round
    if (acc <= seg.K) break;
    if ((size_t)job.tiles * acc * pl.slot_floats <= budget &&
        (long)job.tiles * acc <= std::max<long>(aim, 2L * job.tiles * seg.K))
      break;
    upc += std::max(pl.upc_step, upc / 16 / pl.upc_step * pl.upc_step);
  }
  switch (job.kind) {
    case kFirst: job.first.upc = (int)upc; break;
    case kStride2: job.stride2.upc = (int)upc; break;
    case kGeneral11: case kGeneral12: case kGeneral21: case kGeneral22: job.general.chunk = (int)upc; break;
    default: job.patch.upc = (int)upc; break;
  }
}

void set_partial(BatchJob& job, float* partial) {
  switch (job.kind) {
    case kFirst: job.first.partial = partial; break;
    case kStride2: job.stride2.partial = partial; break;
    case kGeneral11: case kGeneral12: case kGeneral21: case kGeneral22: job.general.partial = partial; break;
    default: job.patch.partial = partial; break;
  }
}

// What the layers of one call (at most kBatchJobs) are launched as: a table for the shared first stage, one for the second
// stage, and the layers on the network input, each of which has a first stage of its own.
struct BatchPlan {
  Plan plans[kBatchJobs];
  BatchTable tab, red;
  int light[kBatchJobs], lights;   // places in plans
  int member[kBatchJobs];          // ... of the jobs of tab
  int blocks, rblocks;
  bool ring8;                      // tab in wgrad_ring_kernel
  size_t lds, scratch[kBatchJobs];
};

void plan_batch(BatchPlan& bp, const ConvWgradJob* jobs, int m, size_t worker_stride, const Segments& seg, float* partial,
                size_t floats, int workgroups, bool alone) {
  std::memset(&bp, 0, sizeof(bp));
  bp.ring8 = alone;
  int heavy = 0;
  double work = 0.0;
  for (int i = 0; i < m; ++i) {
    Plan& pl = bp.plans[i];
    if (plan_first(pl, jobs[i], worker_stride, seg)) { bp.light[bp.lights++] = i; continue; }
    if (!plan_patch(pl, jobs[i], worker_stride, seg) && !plan_stride2(pl, jobs[i], worker_stride, seg))
      plan_general(pl, jobs[i], worker_stride, seg);
    bp.ring8 = bp.ring8 && pl.job.kind >= kPatch4 && pl.job.kind <= kPatch32Narrow && pl.job.kind != kPatchAny;
    ++heavy;
  }
  for (int i = 0; i < m; ++i) {
    Plan& pl = bp.plans[i];
    if (pl.job.kind == kFirst) continue;
    // (where eight wavefronts share a chunk, two units: 128 images of 3-32-64-128, step 77.9 us with four, 76.6 with two)
    if (bp.ring8) { pl.work = pl.ring_work; pl.min_upc = 2; }
    work += pl.work;
  }
  // Layers that share the launch share its workgroups in proportion to the time their units take (not
  // to their arithmetic: a 1x1 projection cut for its few multiply-adds walked 100 slabs, 200 us).
  if (bp.ring8) workgroups /= 2;
  // The scratch is shared out in proportion to what that many partial tiles take, in whole 256-byte lines (tiles that began
  // inside a line cost the three-layer net's step 6 per cent).
  const double room = (double)std::min(floats, conv_wgrad_partial_floats());
  long aim[kBatchJobs];
  double wanted = 0.0;
  for (int i = 0; i < m; ++i) {
    const Plan& pl = bp.plans[i];
    aim[i] = pl.job.kind == kFirst || heavy == 1 ? pl.alone : std::max<long>(1, (long)(workgroups * pl.work / work));
    wanted += (double)std::max<long>(aim[i], pl.job.tiles) * pl.slot_floats;
  }
  size_t scratch = 0;
  for (int i = 0; i < m; ++i) {
    Plan& pl = bp.plans[i];
    const bool light = pl.job.kind == kFirst;
    const size_t budget = (size_t)(room * (double)std::max<long>(aim[i], pl.job.tiles) * pl.slot_floats / wanted) / 64 * 64;
    cut_chunks(pl, seg, aim[i], budget);
    set_partial(pl.job, partial + scratch);
    bp.scratch[i] = scratch;
    scratch += budget;
    bool chunked = false;
    for (int k = 0; k < seg.K; ++k) chunked = chunked || pl.job.chunk[k + 1] - pl.job.chunk[k] > 1;
    long rows = pl.job.chunk[seg.K];   // workgroups per tile, in whichever launch has the most
    if (chunked) rows = std::max<long>(rows, std::max<long>((long)seg.K * pl.job.slots, kUpdateSlots3));
    pl.job.by_tiles = reciprocal_below(pl.job.tiles, (uint64_t)pl.job.tiles * rows);
    pl.job.by_workers = reciprocal_below(seg.K, (uint64_t)seg.K * pl.job.slots);
    if (chunked) {
      bp.red.first[bp.red.n] = bp.rblocks;
      bp.rblocks += pl.job.tiles * seg.K * pl.job.slots;
      bp.red.job[bp.red.n++] = pl.job;
    }
    if (light) continue;
    bp.tab.first[bp.tab.n] = bp.blocks;
    bp.blocks += pl.job.tiles * pl.job.chunk[seg.K];
    bp.lds = std::max(bp.lds, bp.ring8 ? ring_lds_bytes(pl.job.kind >= kPatch8Narrow, 8) : pl.lds);
    bp.member[bp.tab.n] = i;
    bp.tab.job[bp.tab.n++] = pl.job;
  }
}

template <int MB, int NB, bool POOLED>
void launch_light(hipStream_t st, const BatchJob& job, const HeadWgradParams* head, size_t lds, const Segments& seg) {
  if (head) lds = std::max(lds, kHeadWgradLdsFloats * sizeof(float));
  // (its most: the channels of a layer on the network input are at most 4; __syncthreads_or takes a little static LDS too)
  constexpr size_t kMost = std::max({(size_t)2 * wgrad1_stage_bytes(MB, 4), (size_t)4 * MB * NB * 16 * 64 * sizeof(float),
                                     kHeadWgradLdsFloats * sizeof(float)});
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&wgrad_light_kernel<MB, NB, POOLED>), kMost);
  const dim3 hg = head ? head_wgrad_grid(*head, seg) : dim3(1, 0, 1);
  const int head_blocks = (int)(hg.x * hg.y);
  hipLaunchKernelGGL((wgrad_light_kernel<MB, NB, POOLED>), dim3(head_blocks + job.chunk[seg.K]), dim3(kThreads), lds, st, job,
                     head ? *head : HeadWgradParams{}, (int)hg.x, head_blocks, seg);
}

}  // namespace

size_t conv_wgrad_partial_floats() { return (size_t)kConvMaxPartialTiles * (2 * 2 * 16 * kThreads + 128); }

bool conv_wgrad_pooled_supported(int Cout, int cin_real, const ConvGeom& g) { return first_layer_shape(Cout, cin_real, g); }

double conv_wgrad_work(const ConvWgradJob& j) {
  return 2.0 * j.g.rows * j.g.Hp * j.g.Wp * j.Cout * j.g.K;
}

namespace {
// Whether the second stage with the update takes longer than one without and a launch for the update (5 us).  With it a wavefront
// adds all chunks of a worker, sixteen loads on their way at a time (with fewer than four workers some wavefronts have none); without, a
// quarter of them, eight: half a microsecond a trip either way, beside the reading of all partial tiles at 4 TB/s.  Step in us with the
// update / without.  One 3-32 layer with pooling, one worker: 64 images 48.6 / 48.1, 128 55.2 / 53.4, 256 68.5 / 62.9, 700 95.3 / 83.9; two
// workers with 20 and 480 91.8 / 80.5.  3-32-64-128, one worker: 128 images 81.1 / 84.2, 256 101.7 / 98.1, 384 123.1 / 115.1, 1024 195.6 / 183.5;
// two with 20 and 480 139.6 / 130.0.  (More workers: eight, one of them with 665 images of 700, 162.0 / 164.3, as all of that worker's
// workgroups of the other second stage lie on one XCD; of a single layer 94.1 / 85.0.)
bool update_too_long(const BatchTable& tab, int K) {
  if (K >= kThreads / 64) return false;
  int most = 0;
  double tiles = 0;
  for (int i = 0; i < tab.n; ++i) {
    const BatchJob& job = tab.job[i];
    for (int k = 0; k < K; ++k) most = std::max(most, job.chunk[k + 1] - job.chunk[k]);
    tiles += (double)job.tiles * job.chunk[K] * (job.kind == kFirst ? job.slots * 64 : kTile3Stride) * sizeof(float) / 4e6;
  }
  return std::max(0.5 * most / 16, tiles) > std::max(0.5 * most / 32, tiles) + 5;
}

// Wavefronts of a workgroup of the second stage with the update.  A compute unit holds sixteen of them (100 registers) however they are
// grouped.  More per workgroup mean fewer turns at the workers, but a barrier at which all wait for the slowest, and registers held
// by those that have no worker left and no part in the update: sixteen only where all of the launch (an element per thread of the other
// parameters included) is resident at once, eight while the workgroups that add chunks are, and the others not many more (13 workers, 887,000
// other parameters: the launch 16.2 us with eight, 13.0 with four).  Step in us with 4 / 8 / 16, by those
// workgroups and by workers (images of each in brackets):
//    145 (3-32-64-128, 16x16)   14 (2) 68.7 / 67.1 / 66.2
//    145 (3-16-96-128, 16x16)   48 (5) 111.3 / 105.0 / 109.9
//    306 (3-32-128-64)          48 (2) 95.2 / 88.7 / 92.3
//    451 (3-32-64-128)           8 (128) 179.7 / 175.9 / 180.9   16 (40) 143.0 / 137.9 / 140.8   64 (8) 147.5 / 139.6 / 142.2
//    725 (3-32-128-64, 16x16)   12 (13) 76.4 / 79.0 / 81.1
//    886 (3-32-128-128)          5 (40) 100.5 / 103.6 / 108.5    16 (8) 88.1 / 91.3 / 94.6       64 (8) 186.2 / 175.6 / 175.0
//   1595 (3-16-128-256, 16x16)   9 (40) 113.4 / 115.8 / 121.8    32 (8) 117.7 / 117.0 / 119.6    64 (8) 163.0 / 151.7 / 152.3
// Of 248 such networks 0.1 per cent slower on average than with the best of the three, 2.4 at most.
int update_wavefronts(int K, int workgroups, long others) {
  if (K <= 4 || (K <= 32 && (workgroups > 512 || workgroups + others / 512 > 900))) return 4;
  return K > 8 && workgroups + (others + 1023) / 1024 <= 256 ? 16 : 8;
}

// The second stage of all layers of a call and the update of all `params` parameters; false, with nothing launched, where some layer
// has another second stage, or the walk in this one is long, or none has any.
bool update_batch(hipStream_t st, const BatchPlan& bp, size_t worker_stride, const Segments& seg, const SgdArgs& sgd, float* G,
                  size_t params) {
  if (bp.red.n == 0 || params > (size_t)INT32_MAX - 1024 || update_too_long(bp.red, seg.K)) return false;
  BatchTable tab = bp.red;
  struct Range { long beg, end; } covered[2 * kBatchJobs];
  int m = 0, blocks = 0;
  for (int i = 0; i < tab.n; ++i) {
    BatchJob& job = tab.job[i];
    const bool first = job.kind == kFirst;
    if (!first && (job.kind < kPatch4 || job.kind > kPatch32Narrow)) return false;
    const float* const gw = first ? job.first.gw : job.patch.gw;
    const float* const gb = first ? job.first.gb : job.patch.gb;
    const int Cout = first ? job.first.Cout : job.patch.Cout, cin = first ? job.first.cin_real : job.patch.cin_real;
    covered[m++] = {gw - G, gw - G + (long)Cout * 9 * cin};
    if (gb) covered[m++] = {gb - G, gb - G + (long)Cout};
    tab.first[i] = blocks;
    blocks += job.tiles * (first ? job.slots : kUpdateSlots3);
  }
  std::sort(covered, covered + m, [](const Range& a, const Range& b) { return a.beg < b.beg; });
  long others = (long)params;
  for (int i = 0; i < m; ++i) others -= covered[i].end - covered[i].beg;
  const int threads = 64 * update_wavefronts(seg.K, blocks, others);
  RestTable rest{};
  rest.first[0] = blocks;
  long at = 0;
  for (int i = 0; i <= m; ++i) {
    const long end = i < m ? covered[i].beg : (long)params;
    if (end > at) {
      rest.first[rest.n] = blocks;
      rest.beg[rest.n] = (int32_t)at;
      rest.end[rest.n++] = (int32_t)end;
      blocks += (int)((end - at + threads - 1) / threads);
    }
    if (i < m) at = covered[i].end;
  }
  const UpdateTo to{sgd.params, sgd.velocity, G, worker_stride};
  const Lambdas lam = lambdas_of(seg);
  const Optim opt{sgd.lr, sgd.momentum, sgd.weight_decay};
  const size_t lds = (size_t)seg.K * 256 * sizeof(float);   // (kernel G: a quarter of it)
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), lds, st, tab, rest, seg, lam, opt, to); };
#define OMNI_UPDATE(NW_) { if (sgd.velocity) launch(wgrad_update_kernel<true, NW_>); else launch(wgrad_update_kernel<false, NW_>); }
  if (threads == 256) OMNI_UPDATE(4) else if (threads == 512) OMNI_UPDATE(8) else OMNI_UPDATE(16)
#undef OMNI_UPDATE
  return true;
}
}  // namespace

// LDS that a workgroup asks for beside the chain of input gradients: more than half of a compute unit's 160 KB, so that one is there at
// a time.  Two take all of its registers (256 a lane), and the chain's next kernel then waits until some of them end: batch norms of
// 8 us took 29 to 45.  Chunks, and with them the sums, stay as they are.  Step of the ResNet-18 shape in us, two / one at a time: one
// worker, 32 images 890 / 890; four, 128 images 1443 / 1382; sixteen, 300 images 2588 / 2522; four, 512 images 3508 / 3448; eight, 2048 images
// 10773 / 10748.  (With 90 KB the chain's convolutions find less room: 1405 with 128 images, 10856 with 2048.)
constexpr size_t kBesideLds = 81 * 1024;

bool conv_wgrad_batch(hipStream_t st, const ConvWgradJob* jobs, int n, size_t worker_stride, const Segments& seg,
                      float* partial, size_t floats, const HeadWgradParams* head, int workgroups, const SgdArgs* sgd, float* G, size_t params,
                      bool alone, bool beside) {
  if (head && n == 0) {
    head_wgrad_loss(st, true, *head, seg);
    return false;
  }
  for (int base = 0; base < n; base += kBatchJobs) {
    BatchPlan bp;
    plan_batch(bp, jobs + base, std::min(n - base, kBatchJobs), worker_stride, seg, partial, floats, workgroups, alone);
    if (bp.blocks > 0 && bp.ring8) {
      static LdsLimit limit;
      limit.raise(reinterpret_cast<const void*>(&wgrad_ring_kernel), std::max(ring_lds_bytes(true, 8), ring_lds_bytes(false, 8)));
      hipLaunchKernelGGL(wgrad_ring_kernel, dim3(bp.blocks), dim3(2 * kThreads), bp.lds, st, bp.tab, seg);
    } else if (bp.blocks > 0) {
      static LdsLimit limit;
      limit.raise(reinterpret_cast<const void*>(&wgrad_batch_kernel), kBesideLds);
      const size_t lds = beside ? std::max(bp.lds, kBesideLds) : bp.lds;
      hipLaunchKernelGGL(wgrad_batch_kernel, dim3(bp.blocks), dim3(kThreads), lds, st, bp.tab, seg);
    }
    const HeadWgradParams* h = base == 0 ? head : nullptr;   // rides with the first of the light launches
    for (int i = 0; i < bp.lights; ++i) {
      const Plan& pl = bp.plans[bp.light[i]];
      const bool pooled = pl.job.first.dpool != nullptr;
      const int nb = wgrad1_col_blocks(pl.job.first.cin_real);
#define OMNI_LIGHT(MB_, NB_)                                                \
  {                                                                         \
    if (pooled) launch_light<MB_, NB_, true>(st, pl.job, h, pl.lds, seg);   \
    else launch_light<MB_, NB_, false>(st, pl.job, h, pl.lds, seg);         \
  }
      if (pl.job.first.Cout > 32) { if (nb == 2) OMNI_LIGHT(2, 2) else OMNI_LIGHT(2, 1) }
      else { if (nb == 2) OMNI_LIGHT(1, 2) else OMNI_LIGHT(1, 1) }
#undef OMNI_LIGHT
      h = nullptr;
    }
    if (h) head_wgrad_loss(st, true, *h, seg);
    if (sgd && n <= kBatchJobs && update_batch(st, bp, worker_stride, seg, *sgd, G, params)) return true;
    if (bp.rblocks > 0) hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(bp.rblocks), dim3(kThreads), 0, st, bp.red, seg);
  }
  return false;
}

void conv_wgrad_describe(const ConvWgradJob* jobs, int n, const Segments& seg, int workgroups, ConvWgradPlanned* out, bool alone) {
  int launch = 0;
  for (int base = 0; base < n; base += kBatchJobs) {
    BatchPlan bp;
    const int m = std::min(n - base, kBatchJobs);
    plan_batch(bp, jobs + base, m, 0, seg, nullptr, conv_wgrad_partial_floats(), workgroups, alone);
    const int shared = launch++;
    for (int i = 0; i < m; ++i) {
      const BatchJob& job = bp.plans[i].job;
      ConvWgradPlanned& o = out[base + i];
      o = ConvWgradPlanned{};
      o.first_layer = job.kind == kFirst;
      o.launch = -1;
      for (int l = 0; l < bp.lights; ++l)
        if (bp.light[l] == i) o.launch = launch + l;
      for (int l = 0; l < bp.tab.n; ++l)
        if (bp.member[l] == i) o.launch = o.launch < 0 && bp.tab.job[l].kind != kFirst ? shared : -2;
      o.workgroups = job.tiles * job.chunk[seg.K];
      for (int k = 0; k < seg.K; ++k) o.reduced = o.reduced || job.chunk[k + 1] - job.chunk[k] > 1;
      o.scratch_begin = bp.scratch[i];
      o.scratch_end = o.scratch_begin + (o.reduced ? (size_t)o.workgroups * bp.plans[i].slot_floats : 0);
    }
    launch += bp.lights;
  }
}

}  // namespace omni
