// Weight gradient of 3x3 / stride-1 / pad-1 convolutions on maps 4 (4x4), 8, 16 and 32 wide, in bf16 with fp32 accumulation, per
// worker (the gradient line of procedure Train, Algorithm 1):
//
//   G_k[co][u][v][ci] = sum over the positions (n, h, w) of worker k of dY[n, h, w, co] * X[n, h + u - 1, w + v - 1, ci]
//
// A workgroup owns 64 output channels x 64 input channels (KS: 32) x all nine taps and walks the positions of X of one chunk of ONE
// worker, 32 (KS: 64) at a time.  With stride 1 a position has the same number in both tensors, so both are streams of
// consecutive rows of channels.  What bounds the walk is the wavefronts' own instructions (one wavefront per SIMD: a matrix instruction
// takes 32 cycles, four vector instructions behind it are free, every further one costs 4) and getting the streams there:
//
//   * both streams run through rings of eight (KS: six) steps in LDS, [position][channel] as in memory, filled by loads that write LDS
//     themselves (no registers, no vector instructions, no LDS writes by the wavefronts), six (four) steps ahead.  A step uses
//     the rows of dY of its neighbours in the ring for the taps below and above; where those lie outside the image, a strip of zeros;
//   * the operands are formed by the transposing read (lds_transpose_device.h).  Which positions a lane half takes is free as long
//     as both operands agree: half h takes the sixteen positions from 16 h on, in two reduction steps.  That is a whole row of a
//     16-wide map, two of an 8-wide, four of a 4-wide one, so that the columns beside a window of X are zeros or
//     registers the lane holds anyway; on 32-wide maps the halves exchange one word;
//   * the three taps of a row are the window shifted by one element.  A window is shifted once and meets its row of dY, the one
//     above and the one below: 16 vector instructions for 18 matrix instructions (with the rows of X walked for every row of dY, 48);
//   * one barrier per step: it says that the next step has arrived and that the step before last has been read, so that operands
//     are read one phase ahead of their use across it.
//
// Before, both operands were transposed on their way into LDS through registers, with two barriers a unit.  One layer of 2048 images
// of the ResNet-18 shape (154.6 GFLOP), alone, four wavefronts: 64 channels on 32x32 199 -> 146 us (1.06 PFLOP/s, matrix pipe 52 %
// busy at the 1.96 GHz the chip has under it), 128 on 16x16 and 256 on 8x8 190 -> 159.  1024 images of 3-32-64-128, both layers:
// 34.1 -> 28.5 us with eight wavefronts (loads of 84 MB at 5.5 TB/s; of 48000 cycles 4000 are arguments and indexes, 5000 the first
// loads, 30000 the walk, 8000 the meeting of the shares).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "bf16.h"
#include "common.h"
#include "conv_device.h"
#include "lds_load_device.h"
#include "lds_transpose_device.h"
#include "quotient.h"
#include "wgrad_chunk.h"

namespace omni {

namespace {

struct Wgrad3Params {
  const bf16_t* dy;    // [rows*H*W][Cout]
  const bf16_t* src;   // [rows][H][W][Cin]
  float* gw;           // worker w: gw + w*worker_stride, [Cout][9][Cin]
  float* gb;           // may be null
  size_t worker_stride;
  int Cout, Cin, H, W;  // Cin: stored channels (a multiple of 8)
  int cin_real;        // channels of the gradient tensor (the first layer stores 3 channels padded to 8)
  int R, nimg;         // a unit is nimg images x R rows; nimg * R * W = 128
  int Wp, prows;       // kernel C on other widths: patch row length W + 16 (data starts at column 8), patch rows nimg * (R + 2)
  int SX;              // ... bytes between channels of X^T
  int upc;             // units per chunk
  int nimg_log;
  uint32_t by_r, by_patch, by_upi;   // 2^16 / R and / (R + 2), rounded up; reciprocal_below(units per image)
  float* partial;      // [(tile * total_chunks + chunk)][kTile3Stride], see partial3_at
  const void* zero;    // page of zeros for absent pieces
};
constexpr int kUnit = 128;
constexpr int kTile3Floats = 9 * 16 * kThreads;    // one partial tile
constexpr int kTile3Stride = kTile3Floats + 64;      // (behind the tile the 64 sums of the bias)
// Where a partial tile has registers 4 vq .. + 3 of a tap's block of the output (quadrant of the tile), as lane `lane` held them: sixteen
// bytes a lane, so that both stages move 1 KB an instruction.
__device__ inline int partial3_at(int tap, int vq, int quad, int lane) { return ((tap * 4 + vq) * 4 + quad) * 256 + lane * 4; }
__device__ inline void park3(float* tile, const v16f (&acc)[9], int quad, int lane) {
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<v4f*>(tile + partial3_at(t, q, quad, lane)) =
          v4f{acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
}

// Wavefronts that share a block of the output (KS: two of a workgroup's four, else one; twice that with eight wavefronts) and take
// 32 positions of a step each; steps in the rings (four wavefronts: two workgroups per compute unit).
constexpr int ring_shares(bool ks, int waves) { return (ks ? 2 : 1) * waves / 4; }
constexpr int ring_steps(bool ks, int waves) { return ks || waves == 8 ? 6 : 8; }
constexpr int ring_x_bytes(bool ks) { return ks ? 64 : 128; }        // per position
constexpr size_t ring_lds_bytes(bool ks, int waves) {
  const size_t rings = (size_t)ring_steps(ks, waves) * 32 * ring_shares(ks, waves) * (128 + ring_x_bytes(ks)) + 16 * 128;
  const size_t merge = ring_shares(ks, waves) > 1 ? (size_t)waves * 18 * 64 * 16 : 0;
  return rings > merge ? rings : merge;
}

// lanes 32-63 receive what lanes 0-31 sent, and the other way round
__device__ inline uint32_t from_partner(uint32_t send, bool upper) {
  const u32x2 sw = __builtin_amdgcn_permlane32_swap(send, send, false, false);
  return upper ? sw[0] : sw[1];
}

typedef short v4s_t __attribute__((ext_vector_type(4)));
// Four rows of one column (two words); the LDS address is a number.
__device__ __forceinline__ u32x2 tr_read(uint32_t at) {
  typedef __attribute__((address_space(3))) v4s_t lds_v4s;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(uintptr_t)at));
}
__device__ __forceinline__ u32x4 tr_window(uint32_t at, int four_rows) {
  const u32x2 a = tr_read(at), b = tr_read(at + four_rows);
  return u32x4{a[0], a[1], b[0], b[1]};
}

// The window of eight columns q, with the word before it (its upper half is the column to the left) or after it.
__device__ __forceinline__ u32x4 shifted_left(u32x4 q, uint32_t before) {
  return u32x4{__builtin_amdgcn_alignbit(q[0], before, 16), __builtin_amdgcn_alignbit(q[1], q[0], 16),
               __builtin_amdgcn_alignbit(q[2], q[1], 16), __builtin_amdgcn_alignbit(q[3], q[2], 16)};
}
__device__ __forceinline__ u32x4 shifted_right(u32x4 q, uint32_t after) {
  return u32x4{__builtin_amdgcn_alignbit(q[1], q[0], 16), __builtin_amdgcn_alignbit(q[2], q[1], 16),
               __builtin_amdgcn_alignbit(q[3], q[2], 16), __builtin_amdgcn_alignbit(after, q[3], 16)};
}
// KS: at most 32 input channels.  NW: wavefronts.  Those that share a block are added at the end.
template <int WM, bool KS, int NW>
__device__ __forceinline__ void wgrad3_ring_body(const Wgrad3Params& p, const Chunk& ck, int tile, unsigned char* smem3) {
  constexpr int XB = ring_x_bytes(KS), SHARES = ring_shares(KS, NW), SP = 32 * SHARES;   // SP: positions of a step
  constexpr int YS = SP * 128, XS = SP * XB;            // bytes of a step
  constexpr int N = ring_steps(KS, NW);
  constexpr int RW = 32 / WM;                           // map rows of one wavefront's positions (not 4-wide maps)
  constexpr int kLoads = KS ? 3 : 2;                    // of a wavefront per step
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 31, h = lane >> 5, g = lane >> 4, s = lane & 15;
  const bool up = h != 0;
  const int tiles_ci = KS ? 1 : (p.Cin + 63) / 64;
  const int tile_co = KS ? tile : tile / tiles_ci;
  const int co0 = tile_co * 64, ci0 = KS ? 0 : (tile - tile_co * tiles_ci) * 64;
  const int wco = (wave & 2) * 16, wci = KS ? 0 : (wave & 1) * 32;
  const int mine = KS ? (wave & 1) + (wave >> 2) * 2 : wave >> 2;   // this wavefront's share of a step's positions
  const int H = p.H, hw = H * WM;
  const int wk = ck.wk, nchunks = ck.n;

  // ---- the chunk's positions of X: npos from `first` (of the whole tensors) on, in image row row0
  const int upi = p.nimg == 1 ? H / p.R : 1;            // units per image when a unit is part of one image
  const int units_k = p.nimg == 1 ? (ck.end - ck.beg) * upi : (ck.end - ck.beg + p.nimg - 1) >> p.nimg_log;
  const int ubeg = ck.idx * p.upc, uend = min(units_k, ubeg + p.upc);
  int row0 = 0, npos, below = 0;                        // below: rows of the image that follow the chunk's last
  long first;
  if (p.nimg == 1) {
    const int img = exact_quotient(ubeg, p.by_upi), last = exact_quotient(uend, p.by_upi);
    row0 = (ubeg - img * upi) * p.R;
    npos = (uend - ubeg) * kUnit;
    below = uend - last * upi;
    first = (long)(ck.beg + img) * hw + row0 * WM;
  } else {
    const int img0 = ck.beg + (ubeg << p.nimg_log), img1 = min(ck.end, ck.beg + (uend << p.nimg_log));
    npos = (img1 - img0) * hw;
    first = (long)img0 * hw;
  }
  const int ylo = row0 > 0 ? -WM : 0, yn = npos + (below ? WM : 0) - ylo;   // the positions of dY that are needed: yn from ylo on
  const int steps = (npos + SP - 1) / SP;

  // ---- loads: a wavefront instruction brings 1 KB.  Of rows of 128 bytes every other pair has its halves swapped: the four
  // rows of a transposing read then fill the 64 banks once, as rows of 64 bytes do by themselves.
  const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem3;
  const uint32_t sY = base, sX = base + N * YS, sZ = sX + N * XS;
  const int oct8 = (lane & 7) ^ ((lane >> 2) & 4);
  const int ypos = wave * (SP / NW) + (lane >> 3);       // of the step; the second instruction: 8 further
  const int xoct = KS ? lane & 3 : oct8, xpos = KS ? wave * 16 + (lane >> 2) : ypos;
  const uint32_t yend = co0 + 8 * oct8 < p.Cout ? yn : 0, xend = ci0 + 8 * xoct < p.Cin ? npos : 0;
  // a step that is all there (of positions ylo + 0 .. yfull - 1 or 0 .. xfull - 1) needs no look at every lane
  const uint32_t yfull = co0 + 64 <= p.Cout ? max(yn - SP + 1, 0) : 0;
  const uint32_t xfull = ci0 + (KS ? 32 : 64) <= p.Cin ? max(npos - SP + 1, 0) : 0;
  int at = -SP;                                         // first position of the step that is loaded next
  const bf16_t* yp = p.dy + (first + at) * p.Cout + co0;
  const bf16_t* xp = p.src + (first + at) * p.Cin + ci0;
  const uint32_t yoff = (ypos * p.Cout + 8 * oct8) * 2, yoff8 = yoff + 16 * p.Cout, xoff = (xpos * p.Cin + 8 * xoct) * 2;
  const long ystep = (long)SP * p.Cout, xstep = (long)SP * p.Cin;
  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);
  uint32_t slot_to = N - 1;
  auto load_step = [&]() {
    const uint32_t yto = sY + slot_to * YS + wave * (YS / NW), xto = sX + slot_to * XS + wave * (XS / NW);
    if ((uint32_t)(at - ylo) < yfull && (uint32_t)at < xfull) {
      load_to_lds(yp, yoff, yto);
      if constexpr (KS) load_to_lds(yp, yoff8, yto + 1024);
      load_to_lds(xp, xoff, xto);
    } else {
      auto lane_at = [](const bf16_t* from, uint32_t offset) { return reinterpret_cast<const char*>(from) + offset; };
      const char* const none = reinterpret_cast<const char*>(zp);
      load_to_lds((uint32_t)(at + ypos - ylo) < yend ? lane_at(yp, yoff) : none, yto);
      if constexpr (KS) load_to_lds((uint32_t)(at + ypos + 8 - ylo) < yend ? lane_at(yp, yoff8) : none, yto + 1024);
      load_to_lds((uint32_t)(at + xpos) < xend ? lane_at(xp, xoff) : none, xto);
    }
    yp += ystep;
    xp += xstep;
    at += SP;
    slot_to = slot_to + 1 == N ? 0 : slot_to + 1;
  };
  __builtin_amdgcn_s_waitcnt(0x0F70);                   // vmcnt(0): the compiler's waits for its own loads would include these
#pragma unroll 1                                         // (code that nothing has run yet comes from memory too)
  for (int i = 0; i < N - 1; ++i) load_step();            // steps -1 .. N - 3
  if (tid < 16 * 128 / 16) *reinterpret_cast<u32x4*>(smem3 + N * (YS + XS) + tid * 16) = u32x4{0u, 0u, 0u, 0u};

  // ---- operand addresses.  For the transposing read, lane 16 g + s hands in position 8 .. + s / 4 of its half's sixteen and the
  // channels 16 (g % 2) + 4 (s % 4) .. + 3; it receives channel lane % 32 at four positions.
  const int chan = 32 * (g & 1) + 8 * (s & 3), swap = (s & 8) << 3;
  const uint32_t yin = (s >> 2) * 128 + ((wco * 2 + chan) ^ swap);
  const uint32_t yl = (32 * mine + 16 * h) * 128 + yin, zl = sZ + yin;
  const uint32_t xl = sX + (32 * mine + 16 * h + (s >> 2)) * XB + (KS ? chan : (wci * 2 + chan) ^ swap);

  v16f acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
  const bool want_bias = p.gb != nullptr && ci0 == 0;
  float bsum = 0.f;
  auto add_eight = [&](u32x4 q) {
#pragma unroll
    for (int d = 0; d < 4; ++d) bsum += bf16_lo(q[d]) + bf16_hi(q[d]);
  };

  // image row of this wavefront's first position (a step may hold several whole images)
  int hrow = row0 + mine * RW;
  while (WM != 4 && hrow >= H) hrow -= H;
  int hstep = SP / WM;
  while (WM != 4 && hstep >= H) hstep -= H;
  // ---- operands of the step at tY in the ring of dY and tX in that of X
  auto window_x = [&](uint32_t tX, int ks) { return tr_window(xl + tX + ks * 8 * XB, 4 * XB); };
  auto window_y = [&](uint32_t from, int ks) { return tr_window(from + ks * 1024, 512); };
  // where the rows of dY above (the wavefront's first row) and below (its last) begin, at image row r
  auto wrapped = [](uint32_t at) {                      // at < 2 N YS
    constexpr uint32_t all = N * YS;
    return all & (all - 1) ? min(at, at - all) : at & (all - 1);
  };
  auto row_above = [&](uint32_t tY, int r) {
    const bool none = r == 0 && (WM == 32 || !up);
    return none ? zl : sY + wrapped(tY + yl + (N * YS - WM * 128));
  };
  auto row_below = [&](uint32_t tY, int r) {            // (8-wide maps: of the second of the half's two rows)
    const bool none = r + RW == H && (WM == 32 || up);
    return none ? zl : sY + wrapped(tY + yl + (WM == 8 ? 16 : WM) * 128);
  };
  // at the start of step t: own loads of step t + 1 have arrived (those of N - 4 more may still be under way), then everyone's
  auto sync_step = [&]() { asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((N - 4) * kLoads) : "memory"); };
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((N - 3) * kLoads) : "memory");   // steps -1 and 0 have

  uint32_t tY = 0, tX = 0;
  auto advance = [&]() {
    tY = tY + YS == N * YS ? 0 : tY + YS;
    tX = tX + XS == N * XS ? 0 : tX + XS;
    hrow += hstep;
    if (hrow >= H) hrow -= H;
  };
  const bool odd = wave & 1;
  auto bias_of = [&](u32x4 a, u32x4 b) {               // (by value: an array chosen from inside would be one in scratch memory)
    if (!want_bias) return;
    if (KS) add_eight(a);
    add_eight(KS || odd ? b : a);
  };
  // a row of dY (two reduction steps) with the windows of X: the taps of filter row du
  u32x4 xl0, xm0, xr0, xl1, xm1, xr1;
  auto multiply = [&](int du, int ks, u32x4 fa) {
    const bf16x8 f = as_bf16x8(fa);
    acc[du * 3 + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, as_bf16x8(ks ? xm1 : xm0), acc[du * 3 + 1], 0, 0, 0);
    acc[du * 3 + 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, as_bf16x8(ks ? xl1 : xl0), acc[du * 3 + 0], 0, 0, 0);
    acc[du * 3 + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, as_bf16x8(ks ? xr1 : xr0), acc[du * 3 + 2], 0, 0, 0);
  };

  // the order of a region's instructions: behind each of `n` matrix instructions `v` vector instructions and `d` LDS reads
  auto spread = [](auto n, auto v, auto d) {
#pragma unroll
    for (int i = 0; i < decltype(n)::value; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (decltype(v)::value) __builtin_amdgcn_sched_group_barrier(0x002, decltype(v)::value, 0);
      if (decltype(d)::value) __builtin_amdgcn_sched_group_barrier(0x100, decltype(d)::value, 0);
    }
  };
#define OMNI_SPREAD(n, v, d) spread(std::integral_constant<int, n>{}, std::integral_constant<int, v>{}, std::integral_constant<int, d>{})

  if constexpr (WM == 32 || WM == 16) {
    u32x4 a0, a1, b0, b1, c0, c1;                       // rows of dY above, of and below the positions of X
    {
      const uint32_t above = row_above(0, hrow);
      a0 = window_y(above, 0);
      a1 = window_y(above, 1);
    }
    xm0 = window_x(0, 0);
    xm1 = window_x(0, 1);
    for (int t = 0; t < steps; ++t) {
      sync_step();
      b0 = window_y(sY + tY + yl, 0);
      b1 = window_y(sY + tY + yl, 1);
      uint32_t before = 0u, after = 0u;
      if constexpr (WM == 32) {                         // the sixteen columns of the other half are next to this one's
        const uint32_t r = from_partner(up ? xm0[0] : xm1[3], up);
        before = up ? r : 0u;
        after = up ? 0u : r;
      }
      xl0 = shifted_left(xm0, before);
      xr0 = shifted_right(xm0, xm1[0]);
      xl1 = shifted_left(xm1, xm0[3]);
      xr1 = shifted_right(xm1, after);
      multiply(2, 0, a0);
      multiply(2, 1, a1);
      const uint32_t below = row_below(tY, hrow);
      OMNI_SPREAD(2, 3, 2);
      OMNI_SPREAD(4, 6, 0);
      __builtin_amdgcn_sched_barrier(0);
      c0 = window_y(below, 0);
      c1 = window_y(below, 1);
      multiply(1, 0, b0);
      multiply(1, 1, b1);
      advance();
      const uint32_t above = row_above(tY, hrow);
      OMNI_SPREAD(2, 0, 2);
      OMNI_SPREAD(4, 2, 0);
      __builtin_amdgcn_sched_barrier(0);
      bias_of(b0, b1);
      load_step();
      __builtin_amdgcn_sched_barrier(0);
      const u32x4 n0 = window_x(tX, 0), n1 = window_x(tX, 1);
      a0 = window_y(above, 0);
      a1 = window_y(above, 1);
      multiply(0, 0, c0);
      multiply(0, 1, c1);
      OMNI_SPREAD(4, 0, 2);
      OMNI_SPREAD(2, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      xm0 = n0;
      xm1 = n1;
    }
  } else if constexpr (WM == 8) {
    // half h has rows 2 h and 2 h + 1 of the wavefront's four; y0 .. y3: rows 2 h - 1 .. 2 h + 2 of dY
    u32x4 y0, y1, y2, y3;
    y0 = window_y(row_above(0, hrow), 0);
    y1 = window_y(sY + yl, 0);
    xm0 = window_x(0, 0);
    xm1 = window_x(0, 1);
    for (int t = 0; t < steps; ++t) {
      sync_step();
      y2 = window_y(sY + tY + yl, 1);
      y3 = window_y(row_below(tY, hrow), 0);
      xl0 = shifted_left(xm0, 0u);
      xr0 = shifted_right(xm0, 0u);
      xl1 = shifted_left(xm1, 0u);
      xr1 = shifted_right(xm1, 0u);
      multiply(2, 0, y0);
      multiply(1, 0, y1);
      multiply(2, 1, y1);
      OMNI_SPREAD(2, 4, 2);
      OMNI_SPREAD(7, 3, 0);
      __builtin_amdgcn_sched_barrier(0);
      bias_of(y1, y2);
      load_step();
      advance();
      const uint32_t above = row_above(tY, hrow);
      __builtin_amdgcn_sched_barrier(0);
      const u32x4 n0 = window_x(tX, 0), n1 = window_x(tX, 1);
      y0 = window_y(above, 0);
      y1 = window_y(sY + tY + yl, 0);
      multiply(0, 0, y2);
      multiply(1, 1, y2);
      multiply(0, 1, y3);
      OMNI_SPREAD(4, 0, 2);
      OMNI_SPREAD(5, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      xm0 = n0;
      xm1 = n1;
    }
  } else {
    // half h has image h of the step's two; rows are two words; y: rows (0, 1), (1, 2) and (2, 3) of dY
    u32x4 y01, y12, y23;
    auto read_y = [&](uint32_t t4) {
      y01 = window_y(sY + t4 + yl, 0);
      y12 = tr_window(sY + t4 + yl + 512, 512);
      y23 = window_y(sY + t4 + yl, 1);
    };
    read_y(0);
    xm0 = window_x(0, 0);
    xm1 = window_x(0, 1);
    auto left4 = [](u32x4 q) {
      return u32x4{q[0] << 16, __builtin_amdgcn_alignbit(q[1], q[0], 16), q[2] << 16, __builtin_amdgcn_alignbit(q[3], q[2], 16)};
    };
    auto right4 = [](u32x4 q) {
      return u32x4{__builtin_amdgcn_alignbit(q[1], q[0], 16), q[1] >> 16, __builtin_amdgcn_alignbit(q[3], q[2], 16), q[3] >> 16};
    };
    for (int t = 0; t < steps; ++t) {
      sync_step();
      xl0 = left4(xm0);
      xr0 = right4(xm0);
      xl1 = left4(xm1);
      xr1 = right4(xm1);
      const u32x4 top = {0u, 0u, y01[0], y01[1]}, bottom = {y23[2], y23[3], 0u, 0u};
      const u32x4 z01 = y01, z12 = y12, z23 = y23;
      multiply(1, 0, z01);
      multiply(2, 1, z12);
      OMNI_SPREAD(6, 4, 0);
      __builtin_amdgcn_sched_barrier(0);
      load_step();
      advance();
      __builtin_amdgcn_sched_barrier(0);
      read_y(tY);
      const u32x4 n0 = window_x(tX, 0), n1 = window_x(tX, 1);
      multiply(1, 1, z23);
      multiply(0, 0, z12);
      multiply(2, 0, top);
      multiply(0, 1, bottom);
      OMNI_SPREAD(5, 1, 2);
      OMNI_SPREAD(7, 1, 0);
      __builtin_amdgcn_sched_barrier(0);
      bias_of(z01, z23);
      __builtin_amdgcn_sched_barrier(0);
      xm0 = n0;
      xm1 = n1;
    }
  }
#undef OMNI_SPREAD
  // nothing may still be on its way to LDS when it is used again or given back
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  if (want_bias) {
    // the shares of a channel's positions meet: by wavefront, then by half
    float* share = reinterpret_cast<float*>(smem3);
    const int of = KS ? mine : mine * 2 + (wave & 1);
    share[(of * 2 + h) * 64 + wco + j] = bsum;
    __syncthreads();
    if (tid < 64) {
      bsum = share[tid];
#pragma unroll
      for (int i = 1; i < NW; ++i) bsum += share[i * 64 + tid];
    }
  }
  // ---- the block's sums: to the chunk's partial tile or, of a worker in one chunk, to its gradient
  float* const to = p.partial + ((size_t)tile * ck.total + ck.row) * kTile3Stride;
  float* const gw = p.gw + (size_t)wk * p.worker_stride;
  const int quad = wave & (KS ? 2 : 3);                  // quadrant of the tile
  // registers 4 i .. + 3 of the block's 144, i = 4 tap + q
  auto four = [&](int i) { return v4f{acc[i / 4][i % 4 * 4], acc[i / 4][i % 4 * 4 + 1], acc[i / 4][i % 4 * 4 + 2], acc[i / 4][i % 4 * 4 + 3]}; };
  auto put = [&](auto first, auto count) {
    const int ci = ci0 + wci + j;
    if (ci >= p.cin_real) return;                        // (the second stage reads the lanes that hold a gradient only)
    constexpr int from = decltype(first)::value, after = from + decltype(count)::value;
    if (nchunks > 1) {
#pragma unroll
      for (int i = from; i < after; ++i) *reinterpret_cast<v4f*>(to + partial3_at(i / 4, i % 4, quad, lane)) = four(i);
      return;
    }
    float* const at = gw + ((size_t)(co0 + wco + 4 * h) * 9) * p.cin_real + ci;
#pragma unroll
    for (int i = from; i < after; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (co0 + wco + 4 * h + 8 * (i % 4) + e < p.Cout) at[((8 * (i % 4) + e) * 9 + i / 4) * p.cin_real] = acc[i / 4][i % 4 * 4 + e];
  };
  // The shares of the positions meet by halves: of what a wavefront and its partner both hold, each sends one half through LDS
  // and adds and keeps the other (6100 cycles for two shares; with all shares in LDS, three taps at a time, 9600).
  v4f* const slots = reinterpret_cast<v4f*>(smem3);      // [wave][18][lane]
  auto meet = [&](auto sent, auto kept, auto count, int partner) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < decltype(count)::value; ++i) slots[(wave * 18 + i) * 64 + lane] = four(decltype(sent)::value + i);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < decltype(count)::value; ++i) {
      const v4f other = slots[(partner * 18 + i) * 64 + lane];
      const int to4 = decltype(kept)::value + i;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[to4 / 4][to4 % 4 * 4 + e] += other[e];
      if (i % 9 == 8) __builtin_amdgcn_sched_barrier(0);   // (eighteen reads in flight do not fit the registers)
    }
  };
#define OMNI_C(n) std::integral_constant<int, n>{}
  if constexpr (SHARES == 1) {
    put(OMNI_C(0), OMNI_C(36));
  } else if constexpr (SHARES == 2) {
    const int partner = KS ? wave ^ 1 : wave ^ 4;
    if (mine == 0) {
      meet(OMNI_C(18), OMNI_C(0), OMNI_C(18), partner);
      put(OMNI_C(0), OMNI_C(18));
    } else {
      meet(OMNI_C(0), OMNI_C(18), OMNI_C(18), partner);
      put(OMNI_C(18), OMNI_C(18));
    }
  } else {
    auto quarter = [&](auto kept, auto sent) {           // of the half that is left
      meet(sent, kept, OMNI_C(9), wave ^ 4);
      put(kept, OMNI_C(9));
    };
    if (mine & 1) {
      meet(OMNI_C(0), OMNI_C(18), OMNI_C(18), wave ^ 1);
      if (mine & 2) quarter(OMNI_C(27), OMNI_C(18)); else quarter(OMNI_C(18), OMNI_C(27));
    } else {
      meet(OMNI_C(18), OMNI_C(0), OMNI_C(18), wave ^ 1);
      if (mine & 2) quarter(OMNI_C(9), OMNI_C(0)); else quarter(OMNI_C(0), OMNI_C(9));
    }
  }
#undef OMNI_C
  if (tid < 64) {
    if (nchunks > 1) to[kTile3Floats + tid] = bsum;
    else if (want_bias && co0 + tid < p.Cout) p.gb[(size_t)wk * p.worker_stride + co0 + tid] = bsum;
  }
}

}  // namespace
}  // namespace omni
