// Input gradient of a residual block's ENTRY in bf16 (fp32 accumulation): the block input x feeds a
// 3x3 / stride-2 / pad-1 convolution and, beside it, the 1x1 / stride-2 projection of the shortcut; both
// send gradients back to x (the inner F(.) of the gradient line of procedure Train, Algorithm 1):
//
//   dx[n, h, w, ci] = mask * ( sum_{u,v,co} dy[n, (h+1-u)/2, (w+1-v)/2, co] * wt[ci][u][v][co]      (both quotients whole)
//                            + [h, w even] sum_co dys[n, h/2, w/2, co] * wts[ci][co] )
//
// Launched separately through the generic kernel these were its slowest calls (two passes over the
// full-resolution dx, each re-reading the mask; 128-row tiles with two to eight reduction slabs each).
// Here ONE pass writes dx:
//   * a workgroup owns 512 positions of dx (whole rows of whole images) x 64 channels; the positions
//     split into the four parity classes (h mod 2, w mod 2) of 128 each, and a wavefront takes 32 of
//     every class: a class meets only the filter taps of matching parity (1, 2, 2 or 4 of the 9), so
//     no dead tap is ever multiplied, and the classes' different tap counts balance inside every wavefront;
//   * the half-resolution patch of dy (one extra row and column: odd positions reach one further) and the
//     weights of all nine taps are staged per slice of 32 reduction channels, as in conv3_wide_bf16.hip;
//     the shortcut's slices follow with a patch of dys and one weight slab, feeding class (0, 0) only;
//   * the product is formed transposed and written straight from registers in 16-byte pieces, with the
//     ReLU mask of x (and an addend or the old dx, if another consumer of x wrote first) fetched per piece.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "bf16.h"
#include "bn_sums_device.h"
#include "common.h"
#include "kernels.h"
#include "lds_limit.h"
#include "lds_load_device.h"
#include "lines_device.h"
#include "quotient.h"

namespace omni {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

constexpr int kThreads = 256;
constexpr int kUnit = 512;        // positions of dx per unit
constexpr int kTN = 64;           // channels of dx per workgroup
constexpr int KC = 32;            // reduction channels per slice
constexpr int kRow = KC + 8;      // elements per LDS row
constexpr int OC = KC / 8;
constexpr int KK = KC / 16;
constexpr int NPP = 4;            // patch pieces per thread (up to 256 patch positions)

struct S2Params {
  const bf16_t* dy;    // [rows][H/2][W/2][Cs]
  const bf16_t* wt;    // [N][9][Cs]
  const bf16_t* dys;   // [rows][H/2][W/2][Cs2] or null
  const bf16_t* wts;   // [N][Cs2]
  bf16_t* dx;          // [rows*H*W][N]
  int rows, H, W, Cs, Cs2, N;
  int R, nimg;         // a unit is nimg images x R rows of dx; nimg * R * W = 512
  int units, upw;
  const void* zero;
  const bf16_t* mask;
  const uint8_t* mask_bits;   // may be null: the mask at one bit per element, [rows*H*W][N/8] (N a multiple of 64)
  const bf16_t* addend;
  int accumulate;
};

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__global__ __launch_bounds__(kThreads, 1) void conv3s2_dgrad_kernel(S2Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smemS[];
  const int W = p.W, H = p.H, R = p.R;
  const int H2 = H >> 1, W2 = W >> 1, R2 = R >> 1;
  const int PW2 = W2 + 1, PR2 = R2 + 1;
  const int npatch = p.nimg * PR2 * PW2;
  bf16_t* sP = reinterpret_cast<bf16_t*>(smemS);          // [npatch][kRow]
  bf16_t* sW = sP + (size_t)npatch * kRow;                // [9][64][kRow]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 31, h = lane >> 5;
  const int tiles_n = (p.N + kTN - 1) / kTN;
  // (workgroup b runs on XCD b % 8: the channel tiles of a group of units, which read the same patches, share one)
  const int on_xcd = blockIdx.x >> 3;
  const int tile_n = on_xcd % tiles_n;
  const int group = (on_xcd / tiles_n) * 8 + (blockIdx.x & 7);
  if (group * p.upw >= p.units) return;
  const int col0 = tile_n * kTN;
  const int ubeg = group * p.upw, uend = min(p.units, ubeg + p.upw);
  const int nslice = p.Cs / KC, nslice2 = p.dys ? p.Cs2 / KC : 0;
  const int nall = nslice + nslice2;

  // ---- patch staging tasks: piece x = tid + 256 t -> patch position x / OC, channel octet x % OC
  int prel[NPP];
  uint32_t img8 = 0, prow8 = 0, pcol_ok = 0;
  const int npieces = npatch * OC;
#pragma unroll
  for (int t = 0; t < NPP; ++t) {
    const int x = tid + t * kThreads;
    const int pp = min(x, npieces - 1) / OC;
    const int il = pp / (PR2 * PW2), rem = pp - il * (PR2 * PW2);
    const int pr = rem / PW2, pc = rem - pr * PW2;
    prel[t] = (il * H2 + pr) * W2 + pc;   // source position relative to the unit's first (channels: see load_slice)
    img8 |= (uint32_t)il << (8 * t);
    prow8 |= (uint32_t)pr << (8 * t);
    pcol_ok |= (x < npieces && pc < W2 ? 1u : 0u) << t;   // (the extra column lies outside the image)
  }
  const int poct = tid % OC;   // (256 is a multiple of OC: a thread's pieces all carry the same octet)
  // ---- weight staging: this thread carries row tid / OC, octet tid % OC of every tap's slab
  const int wrow = tid / OC;
  const bool wvalid = col0 + wrow < p.N;
  bf16_t* const wdst = sW + wrow * kRow + poct * 8;
  // ---- this wavefront's positions: the 32 class positions wave*32 + j of every parity class
  const int per_img = R2 * W2;
  const int q = wave * 32 + j;
  const int qil = q / per_img, qrem = q - qil * per_img;
  const int qi = qrem / W2, qj = qrem - qi * W2;
  const int pbase = ((qil * PR2 + qi) * PW2 + qj) * kRow + h * 8;
  int ipos[4];   // position within the unit of class (ph, pw) = (a >> 1, a & 1)
#pragma unroll
  for (int a = 0; a < 4; ++a) ipos[a] = (qil * R + 2 * qi + (a >> 1)) * W + 2 * qj + (a & 1);
  const bf16_t* const wfrag = sW + j * kRow + h * 8;

  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);
  // Two staging sets: a slice is requested TWO slices before it is needed (a slice is at most 36 matrix instructions
  // per wavefront, about half a microsecond: one slice of distance left every slice waiting for memory).
  u32x4 rp[2][NPP], rw[2][9];
  auto unit_geom = [&](int unit, int& n0, int& r0, int& nvalid) {
    if (p.nimg == 1) {
      const int upi = H / R, img = unit / upi;
      n0 = img; r0 = (unit - img * upi) * R; nvalid = 1;
    } else {
      n0 = unit * p.nimg; r0 = 0; nvalid = min(p.nimg, p.rows - n0);
    }
  };
  // slice s of `unit`: s < nslice: 32 channels of dy with all nine taps' weights; else of dys with its one slab
  auto load_slice = [&](int set, int unit, int s) {
    const bool main = s < nslice;
    const bf16_t* src = main ? p.dy : p.dys;
    const int cs_total = main ? p.Cs : p.Cs2;
    const int c0 = (main ? s : s - nslice) * KC;
    const bf16_t* wsrc = main ? p.wt + ((long)(col0 + wrow) * 9 * p.Cs + c0 + poct * 8)
                              : p.wts + ((long)(col0 + wrow) * p.Cs2 + c0 + poct * 8);
#pragma unroll
    for (int t = 0; t < 9; ++t)
      rw[set][t] = *reinterpret_cast<const u32x4*>((wvalid && (main || t == 0)) ? wsrc + (main ? t * p.Cs : 0) : zp);
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const long ubase = ((long)n0 * H2 + (r0 >> 1)) * W2;
#pragma unroll
    for (int t = 0; t < NPP; ++t) {
      const int il = (int)(img8 >> (8 * t)) & 255, pr = (int)(prow8 >> (8 * t)) & 255;
      const bool in = ((pcol_ok >> t) & 1u) && il < nvalid && (r0 >> 1) + pr < H2;
      rp[set][t] = *reinterpret_cast<const u32x4*>(in ? src + ((ubase + prel[t]) * cs_total + c0 + poct * 8) : zp);
    }
  };
  auto store_slice = [&](int set) {
#pragma unroll
    for (int t = 0; t < 9; ++t) *reinterpret_cast<u32x4*>(wdst + t * kTN * kRow) = rw[set][t];
#pragma unroll
    for (int t = 0; t < NPP; ++t) {
      const int x = tid + t * kThreads;
      if (x < npieces) *reinterpret_cast<u32x4*>(sP + (x / OC) * kRow + (x % OC) * 8) = rp[set][t];
    }
  };
  // the slice `ahead` slices after (unit, s), running on into the next unit of this workgroup
  auto load_ahead = [&](int set, int unit, int s, int ahead) {
    int u = unit, t = s + ahead;
    if (t >= nall) { t -= nall; u = min(unit + 1, uend - 1); }
    load_slice(set, u, t);
  };

  // (nall is even -- the launcher sees to it -- so slice s of every unit lives in set s & 1)
  load_slice(0, min(ubeg, p.units - 1), 0);
  store_slice(0);
  load_ahead(1, min(ubeg, p.units - 1), 0, 1);
  __syncthreads();

  for (int unit = ubeg; unit < uend; ++unit) {
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const long out_base = ((long)n0 * H + r0) * W;
    const int npos = nvalid * R * W;

    v16f acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    auto slice = [&](int s, auto set_tag) {
      constexpr int SET = decltype(set_tag)::value;
      load_ahead(SET, unit, s, 2);   // (set SET held this slice until the end of the slice before: free now)
      if (s < nslice) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          // class (ph, pw) meets tap (u, v) when ph + 1 - u and pw + 1 - v are even; its source lies (du, dv) =
          // ((ph + 1 - u) / 2, (pw + 1 - v) / 2) from the class position's own half-resolution coordinates
#pragma unroll
          for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int v = 0; v < 3; ++v) {
              const int ph = (u + 1) & 1, pw = (v + 1) & 1;
              const int du = (ph + 1 - u) >> 1, dv = (pw + 1 - v) >> 1;
              const int a = ph * 2 + pw;
              const bf16x8 fa = as_bf16x8(*reinterpret_cast<const u32x4*>(sP + pbase + (du * PW2 + dv) * kRow + kk * 16));
#pragma unroll
              for (int b = 0; b < 2; ++b) {
                const bf16x8 fb = as_bf16x8(*reinterpret_cast<const u32x4*>(wfrag + ((u * 3 + v) * kTN + b * 32) * kRow + kk * 16));
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa, acc[a][b], 0, 0, 0);
              }
            }
        }
      } else {
        // the shortcut's 1x1 / stride-2 projection reaches the even-even positions only
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const bf16x8 fa = as_bf16x8(*reinterpret_cast<const u32x4*>(sP + pbase + kk * 16));
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const bf16x8 fb = as_bf16x8(*reinterpret_cast<const u32x4*>(wfrag + (b * 32) * kRow + kk * 16));
            acc[0][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb, fa, acc[0][b], 0, 0, 0);
          }
        }
      }
      __syncthreads();
      store_slice(SET ^ 1);   // the next slice, requested a slice ago
      __syncthreads();
    };
    for (int s = 0; s < nall; s += 2) {
      slice(s, std::integral_constant<int, 0>{});
      slice(s + 1, std::integral_constant<int, 1>{});
    }

    // ---- epilogue, straight from registers: after the swap of the wavefront's halves
    // lane (j, h) holds channels b*32 + q*16 + 8h .. +7 of its position of class a
    u32x4 em[2][4], ea[2][4];   // mask and addend / old dx of class a: fetched one class ahead
    u32x2 eb[2];                // the mask as bits: the 8 bytes of the tile's 64 channels at this lane's position
    auto load_epi = [&](int a, int set) {
      const size_t row = (size_t)(out_base + ipos[a]) * p.N;
      const bf16_t* other = p.addend ? p.addend : (p.accumulate ? p.dx : nullptr);
      const bf16_t* mask = p.mask_bits ? nullptr : p.mask;
      eb[set] = *reinterpret_cast<const u32x2*>((ipos[a] < npos && p.mask_bits)
                                                    ? p.mask_bits + ((size_t)(out_base + ipos[a]) * (p.N >> 3) + (col0 >> 3))
                                                    : static_cast<const uint8_t*>(p.zero));
#pragma unroll
      for (int bq = 0; bq < 4; ++bq) {
        const int c = col0 + (bq >> 1) * 32 + (bq & 1) * 16 + h * 8;
        const bool in = ipos[a] < npos && c < p.N;
        em[set][bq] = *reinterpret_cast<const u32x4*>((in && mask) ? mask + row + c : zp);
        ea[set][bq] = *reinterpret_cast<const u32x4*>((in && other) ? other + row + c : zp);
      }
    };
    load_epi(0, 0);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const bool row_in = ipos[a] < npos;
      const size_t row = (size_t)(out_base + ipos[a]) * p.N;
      if (a + 1 < 4) load_epi(a + 1, (a + 1) & 1);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int qq = 0; qq < 2; ++qq) {
          float val[8];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const u32x2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[a][b][8 * qq + e]),
                                                              __float_as_uint(acc[a][b][8 * qq + 4 + e]), false, false);
            val[e] = __uint_as_float(sw[0]);
            val[4 + e] = __uint_as_float(sw[1]);
          }
          const int c = col0 + b * 32 + qq * 16 + h * 8;
          if (!row_in || c >= p.N) continue;
          const u32x4 mk = em[a & 1][b * 2 + qq], ad = ea[a & 1][b * 2 + qq];
          if (p.addend) {
#pragma unroll
            for (int d = 0; d < 4; ++d) { val[2 * d] += bf16_lo(ad[d]); val[2 * d + 1] += bf16_hi(ad[d]); }
          }
          if (p.mask_bits) {
            const uint32_t byte = eb[a & 1][b] >> (8 * (2 * qq + h));
#pragma unroll
            for (int e = 0; e < 8; ++e) val[e] = ((byte >> e) & 1u) ? val[e] : 0.f;
          } else if (p.mask) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              val[2 * d] = bf16_lo(mk[d]) > 0.f ? val[2 * d] : 0.f;
              val[2 * d + 1] = bf16_hi(mk[d]) > 0.f ? val[2 * d + 1] : 0.f;
            }
          }
          if (p.accumulate) {
#pragma unroll
            for (int d = 0; d < 4; ++d) { val[2 * d] += bf16_lo(ad[d]); val[2 * d + 1] += bf16_hi(ad[d]); }
          }
          Piece<bf16_t>::store(p.dx + row + c, val);
        }
    }
  }
}

// ---- the same with weights in operand order and everything staged by loads that write LDS themselves (see conv3_wide_bf16.hip)
//
// What the kernel above waits for: a slice's weights and patch, through 26 registers of loads, and one wavefront per SIMD to cover it
// (matrix pipe busy 0.15).  Here a slice of 32 channels of dy comes with the shortcut's, so that the projection is a tenth tap and
// no slice of its own; two workgroups share a compute unit; rows of the patch lie as in memory; and the batch norm below
// gets its sums here, where they took another pass over dx and its input.  2048 images of the ResNet-18 shape, the entries at 64, 128 and
// 256 channels: 731 us together and 260 for the sums -> 254 + 168 + 127 with them (the step 12.23 -> 11.72 ms), 233 + 153 + 120 with results and
// what the epilogue reads in whole lines (1.0 GB, 4.2 TB/s, in the first; the epilogue's vector instructions, the sums in double, were 0.45 of
// the time there, the matrix pipe is busy for 0.42 of the last).
struct S2RingParams {
  const bf16_t* dy;    // [rows][H/2][W/2][Cs]
  const bf16_t* wt;    // operand order, nine taps
  const bf16_t* dys;   // SC: [rows][H/2][W/2][Cs]
  const bf16_t* wts;   // SC: operand order, one tap
  bf16_t* dx;          // [rows*H*W][N]
  int rows, H, W, Cs, N;
  int R, nimg;         // a unit is nimg images x R rows of dx; nimg * R * W = 512, powers of two
  int w2log, r2log;    // log2 of W / 2 and R / 2
  int nx;              // patch instructions of 16 positions: those of the unit, and of the row below where the map goes on
  int units, upw, groups;
  uint32_t by_units;   // reciprocal_below(units of an image)
  const void* zero;
  const bf16_t* mask;
  const uint8_t* mask_bits;   // N a multiple of 64
  const bf16_t* addend;
  int accumulate;
  int gK;              // entries of units, groups and images, as in conv3_wide_bf16.hip
  int32_t gfirst[OMNI_MAX_WORKERS + 1], ufirst[OMNI_MAX_WORKERS + 1], ifirst[OMNI_MAX_WORKERS + 1];
  double* stat_partial;    // STATS: [group][N][2]
  const bf16_t* stat_x;    // ... [rows*H*W][N]
  const float* stat_norm;  // ... [worker][N][2]
};

constexpr uint32_t kHalfUnit = kUnit / 4 * 64;          // bytes of 32 channels of a unit's positions of dy
constexpr uint32_t ring_slot(int nx, bool sc) { return nx * 1024 + (sc ? kHalfUnit : 0) + 64; }   // (zeros at its end)
constexpr uint32_t ring_weights(bool sc) { return (sc ? 20 : 18) * 1024; }
constexpr uint32_t ring_bytes(int nx, bool sc) { return 2 * ring_slot(nx, sc) + 2 * ring_weights(sc); }

// SC: with the shortcut's share, whose slice comes with that of dy, a tenth tap of class (0, 0).  STATS: the sums of the batch norm
// below (see BnStatRequest; N a multiple of 64, the mask, if any, as bits).  SHARE: another share to add, or a mask that is not bits.
template <bool SC, bool STATS, bool SHARE>
__global__ __launch_bounds__(kThreads, 2) void conv3s2_ring_kernel(S2RingParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smemS[];
  const int W = p.W, H = p.H, R = p.R;
  const int H2 = H >> 1, W2 = W >> 1, R2 = R >> 1;
  const uint32_t slot = ring_slot(p.nx, SC);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 31, h = lane >> 5;
  const int tiles_n = (p.N + kTN - 1) / kTN;
  const int on_xcd = blockIdx.x >> 3;                    // (as above)
  const int tile_n = on_xcd % tiles_n;
  const int group = (on_xcd / tiles_n) * 8 + (blockIdx.x & 7);
  if (group >= p.groups) return;
  int gk = 0, ufirst = 0, uafter = p.units, ibeg = 0, iend = p.rows, gbeg = 0;
  if (STATS) {
    const int tg = p.gfirst[lane], tu = p.ufirst[lane], ti = p.ifirst[lane];
    gk = __popcll(__ballot(lane < p.gK && tg <= group)) - 1;
    const bool more = gk + 1 < p.gK;
    gbeg = __builtin_amdgcn_readlane(tg, gk);
    ufirst = __builtin_amdgcn_readlane(tu, gk);
    ibeg = __builtin_amdgcn_readlane(ti, gk);
    uafter = more ? __builtin_amdgcn_readlane(tu, gk + 1) : p.units;
    iend = more ? __builtin_amdgcn_readlane(ti, gk + 1) : p.rows;
  }
  const int col0 = tile_n * kTN;
  const int ubeg = ufirst + (group - gbeg) * p.upw, uend = min(uafter, ubeg + p.upw);
  const int nslice = p.Cs / KC, c16n = p.Cs >> 4;
  float* const sN = reinterpret_cast<float*>(smemS + ring_bytes(p.nx, SC));   // STATS: [64] means, [64] factors
  const uint32_t lds0 = lds_address(smemS);

  // ---- this wavefront's positions: 32 of every class, position q of the half-resolution grid.  The patch is that grid as it lies in
  // memory (rows without a column more): shift (du, dv) is du * W2 + dv positions on, outside the map the zeros at the slot's end.
  const int q = wave * 32 + j;
  const int qil = q >> (p.w2log + p.r2log), qi = (q >> p.w2log) & (R2 - 1), qj = q & (W2 - 1);
  uint32_t xaddr[SC ? 5 : 4];
  auto place_reads = [&](uint32_t from_slot, bool below) {   // below: the map goes on below the unit
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int at = q + (t >> 1) * W2 + (t & 1);
      const bool in = ((t & 1) == 0 || qj < W2 - 1) && ((t >> 1) == 0 || qi < R2 - 1 || below);
      xaddr[t] = lds0 + from_slot + (in ? at * 64 + (h ^ (at >> 2 & 3)) * 16 : (int)slot - 64);
    }
    if (SC) xaddr[SC ? 4 : 0] = lds0 + from_slot + p.nx * 1024 + q * 64 + (h ^ (q >> 2 & 3)) * 16;
  };

  auto unit_geom = [&](int unit, int& n0, int& r0, int& nvalid) {
    unit -= ufirst;
    if (p.nimg == 1) {
      const int img = quotient(unit, p.by_units, 1);
      n0 = ibeg + img; r0 = unit * R - img * H; nvalid = 1;
    } else {
      n0 = ibeg + unit * p.nimg; r0 = 0; nvalid = min(p.nimg, iend - n0);
    }
  };
  // ---- loads: an instruction of a wavefront brings 16 positions x 32 channels, or a weight block.  Positions that are not there
  // (rows below the map, images after the last) are the unit's first instead: nobody reads them.
  const int at0 = wave * 16 + (lane >> 2);
  const uint32_t piece = ((lane & 3) ^ (at0 >> 2 & 3)) * 16, lane_off = at0 * (p.Cs * 2) + piece;
  long lbase = 0;         // of the unit that is loaded next: its first position's element, its slice, how many positions there are
  int llimit = 0, lunit = ubeg, lslice = 0;
  auto load_unit = [&](int unit) {
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    lbase = ((long)n0 * H2 + (r0 >> 1)) * W2 * p.Cs;
    llimit = p.nimg == 1 ? min(R2 + 1, H2 - (r0 >> 1)) * W2 : nvalid * R2 * W2;
  };
  const bool third = wave + 8 < p.nx;
  uint32_t to_slot = 0;
  auto load_patch = [&]() {
    const uint32_t to = lds0 + to_slot + wave * 1024;
    const bf16_t* const from = p.dy + (lbase + lslice * KC);
    const bf16_t* const from_s = SC ? p.dys + (lbase + lslice * KC) : nullptr;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k == 2 && !third) break;
      const uint32_t off = at0 + 64 * k < llimit ? lane_off + (uint32_t)(128 * k * p.Cs) : piece;
      load_to_lds(from, off, to + k * 4096);
      if (SC && k < 2) load_to_lds(from_s, off, to + p.nx * 1024 + k * 4096);
    }
    to_slot = slot - to_slot;
    if (++lslice == nslice) {
      lslice = 0;
      lunit = min(lunit + 1, uend - 1);                  // (after the last unit: that once more, for nothing)
      load_unit(lunit);
    }
  };
  // weight instruction wave + 4 k: of the tile's first or second 32 channels, taps in turn, the shortcut's last
  const int wblk = col0 + 32 * (wave & 1) < p.N ? wave & 1 : 0;   // (a tile of which only the first half exists)
  const int wrow = (col0 >> 5) + wblk;
  const char* const wsrc = reinterpret_cast<const char*>(p.wt) + ((size_t)(wrow * 9 + (wave >> 1)) * c16n << 10);
  const char* const wsrc_s = SC ? reinterpret_cast<const char*>(p.wts) + ((size_t)wrow * c16n << 10) : nullptr;
  const uint32_t wto = lds0 + 2 * slot + wave * 1024;
  auto load_weights = [&](int c16) {
    const char* from = wsrc + ((size_t)c16 << 10);
    uint32_t to = wto + (c16 & 1) * ring_weights(SC);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      if (k == 4 && wave >= 2) {
        if (!SC) break;
        from = wsrc_s + ((size_t)c16 << 10);
      }
      load_to_lds(from, lane * 16, to);
      from += (size_t)(2 * c16n) << 10;
      to += 4096;
    }
  };
  // own weights have arrived (the patch asked for after them may be under way), then everyone's
  auto weights_arrived = [&]() {
    if (SC) {
      if (third) asm volatile("s_waitcnt vmcnt(5)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
    } else {
      if (third) asm volatile("s_waitcnt vmcnt(3)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(2)\n\ts_barrier" ::: "memory");
    }
  };
  load_unit(ubeg);
  load_weights(0);
  load_patch();
  if (tid < 8) *reinterpret_cast<u32x4*>(smemS + ((tid >> 2) + 1) * slot - 64 + (tid & 3) * 16) = u32x4{0u, 0u, 0u, 0u};
  if (STATS && tid < 2 * kTN) sN[(tid & 1) * kTN + (tid >> 1)] = p.stat_norm[((size_t)gk * p.N + col0) * 2 + tid];
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");

  uint32_t read_slot = 0;
  double stat_sum[2] = {0.0, 0.0};
  for (int unit = ubeg; unit < uend; ++unit) {
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    place_reads(read_slot, r0 + R < H);
    v16f acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    // sixteen channels: the taps in an order in which neighbours feed different classes and the patch's shifts are first needed
    // one after the other; fragments are read two taps ahead
    auto sixteen = [&](auto which) {
      constexpr uint32_t half = decltype(which)::value;
      constexpr int kSteps = SC ? 10 : 9;
      const uint32_t wl = lds0 + 2 * slot + half * ring_weights(SC) + lane * 16;
      auto tap_at = [](int i) { return i == 0 ? 4 : i == 1 ? 8 : i == 2 ? 5 : i == 3 ? 7 : SC ? (i == 4 ? 9 : i == 5 ? 6 : 9 - i) : (i == 4 ? 6 : 8 - i); };
      // class (ph, pw) meets tap (u, v) when ph + 1 - u and pw + 1 - v are even; its source lies half of these away
      auto class_at = [&](int i) { const int t = tap_at(i); return t == 9 ? 0 : (t / 3 + 1) % 2 * 2 + (t % 3 + 1) % 2; };
      auto shift_at = [&](int i) {
        const int t = tap_at(i), u = t / 3, v = t % 3;
        return t == 9 ? 4 : ((u + 1) % 2 + 1 - u) / 2 * 2 + ((v + 1) % 2 + 1 - v) / 2;
      };
      auto read = [](uint32_t at) {
        typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
        return as_bf16x8(*(lds_u32x4*)(uintptr_t)at);
      };
      uint32_t second_half = half * 32;
      if (half) asm volatile("" : "+s"(second_half));     // (addresses of either half kept all along would not fit the registers)
      bf16x8 fa[5], fb[3][2];
      auto fetch = [&](int i) {
#pragma unroll
        for (int b = 0; b < 2; ++b) fb[i % 3][b] = read(wl + (tap_at(i) * 2 + b) * 1024);
        const int s = shift_at(i);
        if (i == 0 || s != shift_at(i - 1)) fa[s] = read(half ? xaddr[SC ? s : s & 3] ^ second_half : xaddr[SC ? s : s & 3]);
      };
      fetch(0);
      fetch(1);
#pragma unroll
      for (int i = 0; i < kSteps; ++i) {
        if (i + 2 < kSteps) fetch(i + 2);
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[class_at(i)][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[i % 3][b], fa[shift_at(i)], acc[class_at(i)][b], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // ... and a read or two
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // what the epilogue reads, in whole lines (lines_device.h): a lane has eight channels at four of the half-resolution positions, which
    // for class a are dx positions pos[r] + (a >> 1) W + (a & 1): the mask's bits, and for STATS the batch norm's input
    int lane_q = wave * 32 + lines_base<2>(lane);
    uint32_t pos[4];
    bool live[4];
    auto place_results = [&]() {
      asm volatile("" : "+v"(lane_q));                    // (nothing formed from it before)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at = lane_q + lines_position<2>(r), il = at >> (p.w2log + p.r2log);
        pos[r] = ((uint32_t)n0 * H + r0) * W + (il * R + 2 * ((at >> p.w2log) & (R2 - 1))) * W + 2 * (at & (W2 - 1));
        live[r] = il < nvalid;
      }
    };
    auto shift_of = [&](int a) { return (a >> 1) * W + (a & 1); };
    const int lane_c = lines_channel<2>(lane);
    uint8_t eb[2][4];
    u32x4 xs[2][STATS ? 4 : 1];
    auto load_bits = [&](int a) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        eb[a & 1][r] = 255;
        if (p.mask_bits)
          eb[a & 1][r] = *(live[r] ? p.mask_bits + ((size_t)(shift_of(a) * (p.N >> 3) + (col0 >> 3)) + pos[r] * (p.N >> 3) + (lane_c >> 3))
                                   : static_cast<const uint8_t*>(p.zero));
      }
    };
    auto load_x = [&](int a) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        xs[a & 1][STATS ? r : 0] = *reinterpret_cast<const u32x4*>(
            live[r] ? p.stat_x + (size_t)(shift_of(a) * p.N + col0) + (pos[r] * p.N + lane_c) : static_cast<const bf16_t*>(p.zero));
    };
    for (int cs = 0; cs < nslice; ++cs) {
      const bool last = cs + 1 == nslice;
      // (a unit's first slice had arrived before the last unit's results were stored)
      if (cs == 0) asm volatile("s_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      load_weights(2 * cs + 1);
      load_patch();
      __builtin_amdgcn_sched_barrier(0);
      sixteen(std::integral_constant<uint32_t, 0>{});
      weights_arrived();
      load_weights(last ? 0 : 2 * cs + 2);
      __builtin_amdgcn_sched_barrier(0);
      sixteen(std::integral_constant<uint32_t, 1>{});
      const uint32_t other_slot = slot - read_slot;
#pragma unroll
      for (int t = 0; t < (SC ? 5 : 4); ++t) xaddr[t] += other_slot - read_slot;
      read_slot = other_slot;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the next unit's first slice, before results are stored

    // ---- epilogue, straight from registers, a class at a time
    place_results();
    load_bits(0);
    if (STATS) load_x(0);
    double t[2][8];                 // STATS: this lane's sums of its channels
#pragma unroll
    for (int e = 0; e < 8; ++e) t[0][e] = t[1][e] = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      float val[4][8];
      lines_of<2>(acc[a], val);
      u32x4 kept[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (!live[r] || (!STATS && col0 + lane_c >= p.N)) continue;
        const size_t to = (size_t)(shift_of(a) * p.N + col0) + (pos[r] * p.N + lane_c);
        float(&v)[8] = val[r];
        u32x4 ad = {0u, 0u, 0u, 0u};
        if (SHARE && (p.addend || p.accumulate)) {
          ad = *reinterpret_cast<const u32x4*>((p.addend ? p.addend : p.dx) + to);
          if (p.addend) {
#pragma unroll
            for (int d = 0; d < 4; ++d) { v[2 * d] += bf16_lo(ad[d]); v[2 * d + 1] += bf16_hi(ad[d]); }
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ((eb[a & 1][r] >> e) & 1u) ? v[e] : 0.f;
        if (SHARE && !p.mask_bits && p.mask) {
          const u32x4 mk = *reinterpret_cast<const u32x4*>(p.mask + to);
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            v[2 * d] = bf16_lo(mk[d]) > 0.f ? v[2 * d] : 0.f;
            v[2 * d + 1] = bf16_hi(mk[d]) > 0.f ? v[2 * d + 1] : 0.f;
          }
        }
        if (SHARE && p.accumulate) {
#pragma unroll
          for (int d = 0; d < 4; ++d) { v[2 * d] += bf16_lo(ad[d]); v[2 * d + 1] += bf16_hi(ad[d]); }
        }
        u32x4 stored;
#pragma unroll
        for (int d = 0; d < 4; ++d) stored[d] = pack_bf16(v[2 * d], v[2 * d + 1]);
        *reinterpret_cast<u32x4*>(p.dx + to) = stored;
        kept[r] = stored;
      }
      __builtin_amdgcn_sched_barrier(0);
      if (a < 3) {                                        // (in the registers that have gone)
        load_bits(a + 1);
        if (STATS) load_x(a + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (STATS) {
        v4f mean[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) mean[d] = *reinterpret_cast<const v4f*>(sN + lane_c + 4 * d);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (live[r]) bn_sums_add(t, kept[r], xs[a & 1][r], mean);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (STATS) lines_sums(t, lane, stat_sum);
  }
  if (STATS) {
    // the four wavefronts' sums meet in LDS (once nobody reads patch or weights any more), added in wavefront order
    __syncthreads();
    double* red = reinterpret_cast<double*>(smemS);       // [4][2][64]
#pragma unroll
    for (int i = 0; i < 2; ++i) red[(wave * 2 + lines_sum(lane)) * 64 + lines_sum_channel(lane) + i] = stat_sum[i];
    __syncthreads();
    if (tid < 128) {
      const int c = tid & 63, w = tid >> 6;
      const double tot = ((red[(0 * 2 + w) * 64 + c] + red[(1 * 2 + w) * 64 + c]) + red[(2 * 2 + w) * 64 + c]) +
                         red[(3 * 2 + w) * 64 + c];
      const double factor = w == 1 ? (double)sN[kTN + c] : 1.0;
      p.stat_partial[((size_t)group * p.N + col0 + c) * 2 + w] = tot * factor;
    }
  }
}

template <bool SC, bool STATS, bool SHARE>
void launch_ring_variant(hipStream_t st, const S2RingParams& p, int tiles_n) {
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&conv3s2_ring_kernel<SC, STATS, SHARE>), kLdsOfComputeUnit);
  const dim3 grid(((p.groups + 7) / 8) * 8 * tiles_n);
  hipLaunchKernelGGL((conv3s2_ring_kernel<SC, STATS, SHARE>), grid, dim3(kThreads), ring_bytes(p.nx, SC) + 2 * kTN * sizeof(float),
                     st, p);
}

template <bool SC, bool STATS>
void launch_ring(hipStream_t st, const S2RingParams& p, int tiles_n) {
  if (p.addend || p.accumulate || (p.mask && !p.mask_bits)) launch_ring_variant<SC, STATS, true>(st, p, tiles_n);
  else launch_ring_variant<SC, STATS, false>(st, p, tiles_n);
}

int log2_of(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

}  // namespace

bool conv3s2_dgrad_supported(int rows, int H, int W, int Cin, int Cout, int Cout_sc) {
  if (H % 2 || W % 2 || Cin % 8 != 0 || Cin <= 32 || Cout % KC != 0 || Cout_sc % KC != 0) return false;
  if ((Cout / KC + Cout_sc / KC) % 2 != 0) return false;   // (slices alternate between two staging sets)
  if ((long)rows * H * W * std::max(Cin, std::max(Cout, Cout_sc)) >= (1L << 31)) return false;   // 32-bit element offsets
  if (W < 4 || W > kUnit || kUnit % W != 0) return false;
  const int R = std::min(H, kUnit / W);
  if (R % 2 || H % R != 0 || kUnit % (R * W) != 0) return false;
  const int nimg = kUnit / (R * W);
  if ((nimg > 1 && R != H) || nimg > 255) return false;
  const int npatch = nimg * (R / 2 + 1) * (W / 2 + 1);
  if (npatch * OC > NPP * kThreads || R / 2 + 1 > 255) return false;
  const int tiles_n = (Cin + kTN - 1) / kTN;
  const int units = nimg == 1 ? rows * (H / R) : (rows + nimg - 1) / nimg;
  return (long)units * tiles_n >= 32;   // (less work than that: the generic kernel spreads it better)
}

// Of those, the ones whose weights are wanted in operand order: whole blocks of 32 channels, the shortcut's as many as the other's.
bool conv3s2_dgrad_ring_takes(int rows, int H, int W, int Cin, int Cout, int Cout_sc) {
  if (!conv3s2_dgrad_supported(rows, H, W, Cin, Cout, Cout_sc) || Cin % 32 != 0 || (Cout_sc && Cout_sc != Cout)) return false;
  const int R = std::min(H, kUnit / W);
  if (R < H && 128 + W / 2 > 12 * 16) return false;
  return R == H || reciprocal_below(H / R, (long)rows * (H / R)) != 0;
}

void conv3s2_dgrad_ring_bf16(hipStream_t st, const bf16_t* dy, const bf16_t* wt, int Cout, const bf16_t* dy_sc, const bf16_t* wt_sc,
                             bf16_t* dx, int rows, int H, int W, int Cin, const bf16_t* mask, const uint8_t* mask_bits,
                             bool accumulate, const bf16_t* addend, const void* zero, BnStatRequest* stats) {
  S2RingParams p{};
  p.dy = dy; p.wt = wt; p.dys = dy_sc; p.wts = wt_sc; p.dx = dx;
  p.rows = rows; p.H = H; p.W = W; p.Cs = Cout; p.N = Cin;
  p.R = std::min(H, kUnit / W);
  p.nimg = kUnit / (p.R * W);
  p.w2log = log2_of(W / 2); p.r2log = log2_of(p.R / 2);
  p.nx = (kUnit / 4 + (p.R < H ? W / 2 : 0) + 15) / 16;
  p.zero = zero; p.mask = mask; p.addend = addend; p.accumulate = accumulate ? 1 : 0;
  p.mask_bits = (mask && Cin % kTN == 0) ? mask_bits : nullptr;
  const int tiles_n = (Cin + kTN - 1) / kTN, upi = H / p.R;
  auto units_of = [&](long n) { return (int)(p.nimg == 1 ? n * upi : (n + p.nimg - 1) / p.nimg); };
  const int units = units_of(rows);
  p.by_units = reciprocal_below(upi, units);
  int upw = 1;
  while (upw < 8 && (long)units * tiles_n / (upw * 2) >= 1024) upw *= 2;
  p.gK = 1;
  p.ufirst[1] = units;
  p.ifirst[1] = rows;
  bool with_stats = false;
  if (stats && stats->partial && stats->seg && stats->x && Cin % kTN == 0 && (!mask || p.mask_bits) &&
      stats->seg->off[stats->seg->K] == rows) {
    const Segments& seg = *stats->seg;
    int u = upw;
    auto groups_at = [&](int per) {
      long n = 0;
      for (int k = 0; k < seg.K; ++k) n += (units_of(seg.off[k + 1] - seg.off[k]) + per - 1) / per;
      return n;
    };
    while (groups_at(u) > (long)seg.K * kBnMaxSplits && u < 64) u *= 2;
    if (groups_at(u) <= (long)seg.K * kBnMaxSplits) {
      with_stats = true;
      upw = u;
      p.gK = seg.K;
      for (int k = 0; k < seg.K; ++k) p.ufirst[k + 1] = p.ufirst[k] + units_of(seg.off[k + 1] - seg.off[k]);
      for (int k = 0; k <= seg.K; ++k) p.ifirst[k] = seg.off[k];
      p.stat_partial = stats->partial;
      p.stat_x = stats->x;
      p.stat_norm = stats->stats;
    }
  }
  p.units = p.ufirst[p.gK]; p.upw = upw;
  for (int k = 0; k < p.gK; ++k) p.gfirst[k + 1] = p.gfirst[k] + (p.ufirst[k + 1] - p.ufirst[k] + upw - 1) / upw;
  p.groups = p.gfirst[p.gK];
  if (dy_sc) {
    if (with_stats) launch_ring<true, true>(st, p, tiles_n);
    else launch_ring<true, false>(st, p, tiles_n);
  } else {
    if (with_stats) launch_ring<false, true>(st, p, tiles_n);
    else launch_ring<false, false>(st, p, tiles_n);
  }
  if (with_stats) {
    for (int k = 0; k <= p.gK; ++k) stats->table.first[k] = p.gfirst[k];
    stats->done = true;
  }
}

bool conv3s2_dgrad_bf16(hipStream_t st, const bf16_t* dy, const bf16_t* wt, int Cout, const bf16_t* dy_sc,
                        const bf16_t* wt_sc, int Cout_sc, bf16_t* dx, int rows, int H, int W, int Cin,
                        const bf16_t* mask, bool accumulate, const bf16_t* addend, const void* zero,
                        const uint8_t* mask_bits) {
  if (!conv3s2_dgrad_supported(rows, H, W, Cin, Cout, dy_sc ? Cout_sc : 0)) return false;
  if (dy_sc && !wt_sc) return false;
  const int R = std::min(H, kUnit / W);
  const int nimg = kUnit / (R * W);
  const int npatch = nimg * (R / 2 + 1) * (W / 2 + 1);
  const int tiles_n = (Cin + kTN - 1) / kTN;
  const int units = nimg == 1 ? rows * (H / R) : (rows + nimg - 1) / nimg;
  S2Params p{};
  p.dy = dy; p.wt = wt; p.dys = dy_sc; p.wts = wt_sc; p.dx = dx;
  p.rows = rows; p.H = H; p.W = W; p.Cs = Cout; p.Cs2 = dy_sc ? Cout_sc : 0; p.N = Cin;
  p.R = R; p.nimg = nimg; p.zero = zero; p.mask = mask; p.addend = addend; p.accumulate = accumulate ? 1 : 0;
  p.mask_bits = (mask && Cin % kTN == 0) ? mask_bits : nullptr;
  int upw = 1;
  while (upw < 8 && (long)units * tiles_n / (upw * 2) >= 1024) upw *= 2;
  p.units = units; p.upw = upw;
  const int groups = (units + upw - 1) / upw;
  const dim3 grid(((groups + 7) / 8) * 8 * tiles_n);
  const size_t lds = ((size_t)npatch + 9 * kTN) * kRow * sizeof(bf16_t);
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&conv3s2_dgrad_kernel), kLdsOfComputeUnit);
  hipLaunchKernelGGL(conv3s2_dgrad_kernel, grid, dim3(kThreads), lds, st, p);
  return true;
}

}  // namespace omni
