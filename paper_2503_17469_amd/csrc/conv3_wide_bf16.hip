// Forward and stride-1 input gradient of 3x3 / pad-1 convolutions in bf16 (fp32 accumulation): the
// wide-tile variant of the patch-resident implicit GEMM (same contraction as conv_bf16.hip's kernel D:
// the inner F(.) of the gradient line of procedure Train, Algorithm 1).
//
//   out[m][co] = sum_{u,v,ci} src[n, h+u-1, w+v-1, ci] * wgt[co][u][v][ci]        (dgrad: taps mirrored)
//
// A unit is 256 positions (two workgroups per compute unit, 256 registers per lane) or, where two of those do not fit LDS
// (4-wide maps), 512 (one workgroup, one wavefront per SIMD, 512 registers); a workgroup owns a unit x 64 output channels, a
// wavefront a quarter of the positions.  What limits such a product is not a unit of the machine but waiting, so:
//
//   * the next reduction step's fragments are read under the matrix instructions of this one (two register sets);
//   * the reduction is staged 32 channels at a time, by loads that write LDS themselves (NP = 0): no registers, no store
//     instructions and no wait for either.  A slice's patch goes to the other of two slots while this one's is read; its
//     weights come 16 channels at a time, one half being read while the other is filled, in the order the matrix instruction
//     wants them, which the cast to bf16 lays out.  Two barriers per slice;
//   * where those loads do not fit (other map widths, channel counts that are no multiple of 32, a single slice), a slice
//     comes through registers: its patch AND the weights of all nine taps (9 x 64 x 32) into LDS together, no barrier and no
//     wait inside a slice.  The memory counter retires loads in order: weight slabs requested tap by tap, in between the
//     loads of the next patch, waited for those as well (about 1 us per tap, measured).  All loads of the next slice are
//     issued together when a slice begins and are first needed when it ends, where two barriers separate the last fragment
//     read from the stores that replace patch and weights;
//   * the product is formed TRANSPOSED (weights as the left operand): a lane then holds, for one
//     position, runs of four consecutive channels; exchanges within the wavefront (lines_device.h) turn that into whole
//     lines of the output per instruction -- no staging of the output tile through LDS.
//
// 2048 images of the ResNet-18 shape, 154.6 GFLOP per launch, each alone, staged through registers / by loads that write LDS / and
// stored in whole lines: forward with the batch norm's sums 216 / 187 / 175 us at 64 channels (32x32 maps; 706 MB, 4.0 TB/s),
// 190 / 154 / 151 at 128, 172 / 136 / 138 at 256 (1.1 PFLOP/s, matrix pipe busy 0.66 at the 1.63 GHz that the chip then holds);
// input gradient with mask, shortcut's gradient and sums 294 / 261 / 248 (1.2 GB, 4.9 TB/s), 224 / 188 / 183, 199 / 160 / 158.
// At 64 channels memory and vector instructions (the sums are in double) bind, at 256 the matrix pipe.
// 128 images: 22-24 -> 19-21 and 26-29 -> 24-26.5, a third of it the first loads.
//
// 1024 images of three conv layers 3-32-64-128, 32x32: forward 32 -> 64 on 16x16 with pooling 20.6 us (one slice, through registers),
// 64 -> 128 on 8x8 19.5 -> 17.3, input gradients 64 -> 32 21.7 -> 20.0 and 128 -> 64 18.2 -> 15.5.  Of a workgroup's 30000 cycles
// in the first, 6000 are the first loads, 4600 per unit the matrix pipe (two workgroups on it) and 5000 the epilogue's vector
// instructions, half of them pooling; indexes by division were 2600.
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
#include "pool_device.h"
#include "quotient.h"

namespace omni {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

constexpr int kThreads = 256;

struct WideParams {
  const bf16_t* src;   // [rows][H][W][Cs]
  const bf16_t* wgt;   // [N][9][Cs]; staged by loads that write LDS: in operand order, blocks [N/32][9][Cs/16]
  bf16_t* out;         // [rows*H*W][N]
  int rows, H, W, Cs, N;
  int R, nimg;         // a unit is nimg images x R rows; nimg * R * W = 128 MA
  int units, upw;      // units in all, units per workgroup
  int groups;          // of upw units (see below)
  int flip;            // 1: dgrad (mirrored taps)
  int wlog;            // log2 of W
  uint32_t by_rows;    // 2^22 / (R + 2) rounded up
  uint32_t by_patch, by_row, by_r;   // 2^22 / d rounded up, for division of a patch position by a patch and by a patch row, and of a row by R
  uint32_t by_units;   // reciprocal_below(units of an image)
  const void* zero;    // zeros for absent pieces
  const float* bias;
  const bf16_t* mask;     // [rows*H*W][N] or null: the value passes where mask > 0
  const uint8_t* mask_bits;   // BITS: [rows*H*W][N/8], the mask at one bit per element (N a multiple of 64)
  const bf16_t* addend;   // [rows*H*W][N] or null: added to the product before the mask
  int relu, accumulate;
  // Workgroup g (after the XCD mapping below) takes units of ONE entry of this table: entry k owns the units
  // ufirst[k] .. ufirst[k+1]-1 and the groups gfirst[k] .. gfirst[k+1]-1 of upw units each.  One entry that
  // spans everything, or one per worker when the layer's batch-norm sums are wanted (a group's sums then
  // belong to one worker).
  int gK;
  int32_t gfirst[OMNI_MAX_WORKERS + 1], ufirst[OMNI_MAX_WORKERS + 1];
  int32_t ifirst[OMNI_MAX_WORKERS + 1];   // the entries' images
  bf16_t* pool;           // POOL: [rows*(H/2)*(W/2)][N], the 2 x 2 max pooling of `out`
  uint8_t* pool_code;     // ... and where its gradient goes (pool_code_of)
  const uint8_t* unpool_code;   // plain: see UnpoolRequest
  bf16_t* unpool;
  double* stat_partial;   // STATS: [group][N][2] sums of the stored output and of its squares (BWD: see BnStatRequest)
  const bf16_t* stat_x;   // STATS and BWD: [rows*H*W][N]
  const float* stat_norm; // ... [worker][N][2]
};

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// NP: 16-byte patch pieces per thread.  W8: maps 8 wide (the wavefront takes the map rows of every 64
// positions in the order 0 4 1 5 2 6 3 7: rows 4 apart are complementary in the LDS banks, neighbours are
// not).  BWD: mask / addend / accumulate in the epilogue.
constexpr int KC = 32;            // reduction channels per slice
constexpr int kRow = KC + 8;      // elements per LDS row (80 bytes): sixteen 16-byte reads of consecutive rows cover all banks
constexpr int OC = KC / 8;        // 16-byte pieces per patch position and per weight row
constexpr int KK = KC / 16;       // reduction steps per tap
// With loads that write LDS themselves (NP = 0): patches of 32 channels, rows of 64 bytes, no column halo, in two slots; weights of 16
// channels, in the order the matrix instruction wants them (blocks of 64 lanes x 8 elements, see frag_offset), in two halves.  Both are
// whole cache lines a wavefront: with patches of 16 channels, 32 bytes a position, a load took 200 cycles and bound the kernel.
constexpr int kDmaPatch = 320;                              // positions at most
constexpr uint32_t kDmaSlot = kDmaPatch * 64 + 64;          // (with the zeros that absent columns are read from)
constexpr uint32_t dma_weights(int nb) { return 9 * nb * 1024; }
constexpr uint32_t dma_lds(int nb) { return 2 * kDmaSlot + 2 * dma_weights(nb); }

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// pool_code_of for two channels of bf16 values that are not negative (a ReLU's): their bits are in the order of their values.
__device__ inline uint32_t pool_pair(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t& code) {
  const u16x2 va = __builtin_bit_cast(u16x2, a), vb = __builtin_bit_cast(u16x2, b), vc = __builtin_bit_cast(u16x2, c),
              vd = __builtin_bit_cast(u16x2, d), one = {1, 1}, four = {4, 4};
  const u16x2 m = __builtin_elementwise_max(__builtin_elementwise_max(va, vb), __builtin_elementwise_max(vc, vd));
  const u16x2 na = __builtin_elementwise_min((u16x2)(m - va), one), nb = __builtin_elementwise_min((u16x2)(m - vb), one),
              nc = __builtin_elementwise_min((u16x2)(m - vc), one);       // 1: less than the maximum
  // first of those equal to it; 4 where it is zero (then na = 0)
  const u16x2 k = na * (nb * nc + nb) + na;
  code = __builtin_bit_cast(uint32_t, (u16x2)(k + (four - four * __builtin_elementwise_min(m, one))));
  return __builtin_bit_cast(uint32_t, m);
}

// v of the even (quad_perm [0,0,2,2], 0xA0) or the odd ([1,1,3,3], 0xF5) lane of a pair
template <int CTRL>
__device__ inline uint32_t beside(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// MA: 32-position blocks per wavefront: 4 (a unit of 512 positions, one workgroup per compute unit) or 2 (256
// positions, two workgroups per compute unit, whose load, store and compute phases overlap each other's).
// STATS (MA = 2, no bias, no ReLU): the per-channel sums of the group's stored outputs and of their squares go to
// p.stat_partial, the first pass of the batch norm that follows, without reading the tensor back.  With BWD: the sums
// of the stored gradient and of its product with the normalised input, the first pass of the batch norm's backward,
// for one read of that input instead of two tensors (its means and factors wait in LDS).
// BITS (input gradient): the ReLU mask is read as one bit per element, 8 bytes per position and channel tile
// instead of 128.
// NB: 32-channel blocks of output per workgroup: 2, or 1 for layers with at most 32 outputs (three workgroups per compute unit).
// POOL (forward, 16- and 8-wide maps): the 2 x 2 max pooling and its codes too, see the epilogue.
// ONE: the reduction is a single slice, whose weights stay in LDS for all units of the workgroup.
template <int MA, int NP, bool W8, bool BWD, bool STATS = false, bool BITS = false, int NB = 2, bool POOL = false, bool ONE = false>
__global__ __launch_bounds__(kThreads, MA == 4 ? 1 : NB == 1 ? 3 : 2) void conv3_wide_kernel(WideParams p) {
  static_assert(!STATS || (MA == 2 && (!BWD || BITS)), "statistics come with the 256-position unit only");
  static_assert(NB == 2 || (!BWD && !STATS), "the narrow tile has neither mask nor sums");
  static_assert(!POOL || (!BWD && !STATS), "pooling is a forward epilogue");
  constexpr int kTN = 32 * NB;    // output channels per workgroup
  constexpr bool DMA = NP == 0;
  constexpr bool UNPOOL = MA == 2 && (DMA || ONE) && !BWD && !STATS && !POOL;   // may expand a pooling's gradient (the others' registers are full)
  constexpr bool STOP = ONE;   // no loads for a unit that does not come (the other variants would spill at the branch)
  constexpr int RW = (9 * kTN * OC + kThreads - 1) / kThreads;   // weight pieces per thread and slice
  static_assert(!DMA || (MA == 2 && !ONE), "units of 256 positions");
  static_assert(!BITS || BWD, "mask bits belong to the input gradient");
  constexpr int WPOS = 32 * MA;   // positions per wavefront
  extern __shared__ __attribute__((aligned(16))) unsigned char smemW[];
  const int W = p.W, H = p.H, R = p.R;
  const int PW = W + 2, PR = R + 2;
  const int npatch = p.nimg * PR * PW;
  bf16_t* sP = reinterpret_cast<bf16_t*>(smemW);          // [npatch][kRow]
  bf16_t* sW = sP + (size_t)npatch * kRow;                // [9][64][kRow]
  float* sN = DMA ? reinterpret_cast<float*>(smemW + dma_lds(NB))
                  : reinterpret_cast<float*>(sW + 9 * kTN * kRow);   // STATS and BWD: [64] means, [64] factors; forward: [64] biases
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 31, h = lane >> 5;
  const int tiles_n = (p.N + kTN - 1) / kTN;
  // Workgroups are dealt to the 8 XCDs round-robin by index, and every XCD has an L2 of its own.  The
  // channel tiles of one group of units all read the same patches: they must run on ONE XCD, next to each
  // other in time, or every patch crosses the fabric once per channel tile (at 512 channels: eight times).
  // Workgroup b runs on XCD b % 8; there it is the (b / 8)-th: channel tile fastest, then the XCD's groups.
  const int on_xcd = blockIdx.x >> 3;
  const int tile_n = on_xcd % tiles_n;
  const int group = (on_xcd / tiles_n) * 8 + (blockIdx.x & 7);
  if (group >= p.groups) return;   // (the grid is rounded up to whole rounds of 8 groups)
  // (the tables lie in lines of arguments of their own, 640 cycles each at first touch: without sums there is one entry)
  int gk = 0, ufirst = 0, uafter = p.units, ibeg = 0, iend = p.rows, gbeg = 0;
  if (STATS) {                                            // (all lanes at once: entry by entry, eight workers' took 5000 cycles)
    const int tg = p.gfirst[lane], tu = p.ufirst[lane], ti = p.ifirst[lane];   // (65 entries)
    gk = __popcll(__ballot(lane < p.gK && tg <= group)) - 1;
    const bool more = gk + 1 < p.gK;
    gbeg = __builtin_amdgcn_readlane(tg, gk);
    ufirst = __builtin_amdgcn_readlane(tu, gk);
    ibeg = __builtin_amdgcn_readlane(ti, gk);
    uafter = more ? __builtin_amdgcn_readlane(tu, gk + 1) : p.units;
    iend = more ? __builtin_amdgcn_readlane(ti, gk + 1) : p.rows;
  }
  const int col0 = tile_n * kTN;
  const int K = 9 * p.Cs;
  const int ubeg = ufirst + (group - gbeg) * p.upw, uend = min(uafter, ubeg + p.upw);
  const int nslice = p.Cs / KC;

  // ---- patch staging tasks: piece x = tid + 256 t -> patch position x / OC, channel octet x % OC
  int prel[NP > 0 ? NP : 1];
  uint32_t col_ok = 0, top = 0, bottom = 0;
  uint32_t img8[(NP + 3) / 4 + 1];
#pragma unroll
  for (int t = 0; t < (NP + 3) / 4; ++t) img8[t] = 0;
  const int npieces = npatch * OC;
#pragma unroll
  for (int t = 0; t < NP; ++t) {
    const int x = tid + t * kThreads;
    const int pp = min(x, npieces - 1) / OC, oct = x % OC;
    const int il = (int)(((uint32_t)pp * p.by_patch) >> 22), rem = pp - il * (PR * PW);
    const int pr = (int)(((uint32_t)rem * p.by_row) >> 22), pc = rem - pr * PW;
    prel[t] = ((il * H + pr - 1) * W + pc - 1) * p.Cs + oct * 8;
    col_ok |= (x < npieces && pc >= 1 && pc <= W ? 1u : 0u) << t;
    top |= (pr == 0 ? 1u : 0u) << t;
    bottom |= (pr == PR - 1 ? 1u : 0u) << t;
    img8[t / 4] |= (uint32_t)il << (8 * (t % 4));
  }
  // ---- weight staging: piece tid + 256 t is octet tid % OC of row (tid + 256 t) / OC, rows being tap by tap the tile's channels;
  // 256 pieces are one tap's (two of the narrow tile: threads of the second half are a tap ahead)
  constexpr int kTaps = kThreads / (kTN * OC);            // taps per pass
  const int wrow = tid / OC, woct = tid % OC, wtap = NB == 2 ? 0 : wrow / kTN;
  const bool wvalid = col0 + wrow % kTN < p.N;
  const long woff = wvalid ? (long)(col0 + wrow % kTN) * K + (long)wtap * p.Cs + woct * 8 : 0;
  bf16_t* const wdst = sW + wrow * kRow + woct * 8;
  // ---- fragment addresses: this wavefront's positions wave*128 + a*32 + j
  auto row_order = [](int t) { return (t >> 1) + 4 * (t & 1); };   // t: 0..7
  int pbase[MA];
  const uint32_t lds0 = lds_address(smemW), zeros = lds0 + kDmaPatch * 64;
  uint32_t xaddr[DMA ? 9 : 1][MA];                        // DMA: where tap t of block a's positions lies in a buffer
  // how the four pieces of a patch position are moved (xor) so that sixteen lanes' reads cover all banks
  auto moved = [](int at) { return W8 ? (at >> 2 & 1) | (at >> 3 & 2) : at >> 2 & 3; };
#pragma unroll
  for (int a = 0; a < MA; ++a) {
    int pos = wave * WPOS + a * 32 + j;
    if (W8 && !DMA) pos = wave * WPOS + (a >> 1) * 64 + row_order((a & 1) * 4 + (j >> 3)) * 8 + (j & 7);
    // (rows 0 2 1 3: of sixteen lanes the rows are two apart, and the rows of a pooling window are lanes j and j ^ 16)
    if (W8 && DMA) pos = wave * WPOS + a * 32 + ((j & 7) | (j & 8) << 1 | (j & 16) >> 1);
    const int rr = pos >> p.wlog, w = pos - (rr << p.wlog);
    const int il = (int)(((uint32_t)rr * p.by_r) >> 22), r = rr - il * R;
    pbase[a] = ((il * PR + r) * PW + w) * kRow + h * 8;   // patch origin is (-1, -1): tap (u, v) adds u*PW + v
    if constexpr (DMA) {
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int at = (il * PR + r + t / 3) * W + w + t % 3 - 1;
        const bool in = (t % 3 > 0 || w > 0) && (t % 3 < 2 || w < W - 1);
        xaddr[DMA ? t : 0][a] = in ? lds0 + at * 64 + (h ^ moved(at)) * 16 : zeros;
      }
    }
  }
  const bf16_t* const wfrag = sW + j * kRow + h * 8;
  // ---- in the epilogue a lane has eight channels at 2 NB positions of every block (lines_device.h): position place(a, r) of the unit
  constexpr int NR = 2 * NB;
  int lane_pos = wave * WPOS + (lane & 7), lane_c = lines_channel<NB>(lane);
  if (NB == 1) lane_pos += (lane >> 3 & 1) * (W8 && DMA ? 16 : W8 ? 32 : 8);
  const int lane_pooled = POOL ? (lane_pos >> p.wlog >> 1) * (W >> 1) + ((lane_pos & (W - 1)) >> 1) : 0;
  auto place = [](int a, int r) {
    const int p3 = r >> 1, p4 = r & 1;   // the bits of the lane that had it
    return W8 && DMA ? a * 32 + p3 * 16 + p4 * 8 : W8 ? (a >> 1) * 64 + (a & 1) * 16 + p4 * 8 + p3 * 32 : a * 32 + p3 * 8 + p4 * 16;
  };

  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);
  u32x4 rp[NP > 0 ? NP : 1], rw[ONE ? 1 : RW];
  auto unit_geom = [&](int unit, int& n0, int& r0, int& nvalid) {
    unit -= ufirst;
    if (p.nimg == 1) {
      const int img = quotient(unit, p.by_units, 1);
      n0 = ibeg + img; r0 = unit * R - img * H; nvalid = 1;
    } else {
      n0 = ibeg + unit * p.nimg; r0 = 0; nvalid = min(p.nimg, iend - n0);
    }
  };
  // everything slice cs of `unit` needs, on its way to registers (all loads are unconditional)
  auto load_w = [&](int t, int cs) {
    const bool in = wvalid && (NB == 2 || kTaps * t + wtap < 9);
    return *reinterpret_cast<const u32x4*>(in ? p.wgt + (woff + (long)(kTaps * t) * p.Cs + cs * KC) : zp);
  };
  auto store_w = [&](int t, u32x4 v) {
    if (NB == 2 || kTaps * t + wtap < 9) *reinterpret_cast<u32x4*>(wdst + t * kTaps * kTN * kRow) = v;
  };
  auto load_slice = [&](int unit, int cs) {
    if constexpr (!ONE) {
#pragma unroll
      for (int t = 0; t < RW; ++t) rw[t] = load_w(t, cs);
    }
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const int ubase = (n0 * H + r0) * W * p.Cs + cs * KC;
    const uint32_t pvalid = col_ok & ~(r0 == 0 ? top : 0u) & ~(r0 + R == H ? bottom : 0u);
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const int il = (int)(img8[t / 4] >> (8 * (t % 4))) & 255;
      const bool in = ((pvalid >> t) & 1u) && il < nvalid;
      rp[t] = *reinterpret_cast<const u32x4*>(in ? p.src + (ubase + prel[t]) : zp);
    }
  };
  auto store_slice = [&]() {
    if constexpr (!ONE) {
#pragma unroll
      for (int t = 0; t < RW; ++t) store_w(t, rw[t]);
    }
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const int x = tid + t * kThreads;
      if (x < npieces) *reinterpret_cast<u32x4*>(sP + (x / OC) * kRow + (x % OC) * 8) = rp[t];
    }
  };

  if (STATS && BWD && tid < 2 * kTN) sN[(tid & 1) * kTN + (tid >> 1)] = p.stat_norm[((size_t)gk * p.N + col0) * 2 + tid];
  constexpr bool AFFINE = !BWD && !STATS;   // bias and ReLU exist in the plain forward only
  const float bias = AFFINE && p.bias ? p.bias[min(col0 + (tid & (kTN - 1)), p.N - 1)] : 0.f;
  // ---- DMA: a patch instruction of a wavefront brings 16 positions, a weight instruction a block
  constexpr int kXI = kDmaPatch / 16 / 4;                 // patch instructions per wavefront at most
  const bf16_t* xptr[DMA ? kXI : 1];                      // of the unit that is loaded next
  uint32_t xstep[DMA ? kXI : 1];                          // 0 where there is nothing and a zero is loaded
  const int nx = (p.nimg * PR * W + 15) / 16;
  const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto load_unit = [&](int unit) {
    if constexpr (DMA) {
      int n0, r0, nvalid;
      unit_geom(unit, n0, r0, nvalid);
      int at0 = wave * 16 + (lane >> 2);
      asm volatile("" : "+v"(at0));                       // (places and pieces kept from unit to unit would not fit the registers)
#pragma unroll
      for (int k = 0; k < kXI; ++k) {
        const int at = at0 + 64 * k;
        const int row = at >> p.wlog, w = at & (W - 1), il = (int)(((uint32_t)row * p.by_rows) >> 22), pr = row - il * PR;
        const int hr = r0 + pr - 1;
        const bool in = unit < uend && il < nvalid && hr >= 0 && hr < H;
        xptr[k] = in ? p.src + (((size_t)(n0 + il) * H + hr) * W + w) * p.Cs + ((lane & 3) ^ moved(at)) * 8 : zp;
        xstep[k] = in ? KC : 0;
      }
    }
  };
  // the patch of the next slice (unit by unit) to the next slot, and the weights of sixteen channels to either half
  uint32_t to_slot = 0;
  int lunit = ubeg, lslice = 0;
  auto load_patch = [&]() {
    if constexpr (DMA) {
#pragma unroll
      for (int k = 0; k < kXI; ++k) {
        if (k == kXI - 1 && (int)wave_u + 4 * k >= nx) break;   // (more than 16 in all)
        load_to_lds(xptr[k], lds0 + to_slot + (wave_u + 4 * k) * 1024);
        xptr[k] += xstep[k];
      }
      to_slot = kDmaSlot - to_slot;
      if (++lslice == nslice) {
        lslice = 0;
        load_unit(++lunit);                               // (past the last unit: images that are not there, zeros)
      }
    }
  };
  // weight instruction wave + 4 k: two of a tap's blocks (NB == 1: one), taps in turn (flip: the last one first in LDS)
  const int c16n = p.Cs >> 4, wtap0 = NB == 2 ? wave_u >> 1 : wave_u, wblk = NB == 2 ? wave_u & 1 : 0;
  const int wexists = col0 + 32 * wblk < p.N ? wblk : 0;  // (a tile of which only the first half exists)
  const char* const wsrc = reinterpret_cast<const char*>(p.wgt) + ((size_t)(((col0 >> 5) + wexists) * 9 + wtap0) * c16n << 10);
  const uint32_t wstride = (uint32_t)((NB == 2 ? 2 : 4) * c16n) << 10;
  const uint32_t wto = lds0 + 2 * kDmaSlot + ((p.flip ? 8 - wtap0 : wtap0) * NB + wblk) * 1024;
  const int wstep = p.flip ? -4096 : 4096;
  auto load_weights = [&](int c16) {
    if constexpr (DMA) {
      constexpr int kWI = 9 * NB;
      const char* from = wsrc + ((size_t)c16 << 10);
      uint32_t to = wto + (c16 & 1) * dma_weights(NB);
#pragma unroll
      for (int k = 0; k < (kWI + 3) / 4; ++k) {
        if (k == (kWI + 3) / 4 - 1 && (int)wave_u + 4 * k >= kWI) break;
        load_to_lds(from, lane * 16, to);
        from += wstride;
        to += wstep;
      }
    }
  };
  // own weights have arrived (the patch asked for after them may be under way), then everyone's
  const int xloads = (nx - (int)wave_u + 3) / 4;
  auto weights_arrived = [&]() {
    if (xloads <= 4) asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(5)\n\ts_barrier" ::: "memory");
  };
  if constexpr (DMA) {
    load_unit(ubeg);
    load_weights(0);
    load_patch();
    if (tid < 8)
      *reinterpret_cast<u32x4*>(smemW + (tid >> 2) * kDmaSlot + kDmaPatch * 64 + (tid & 3) * 16) = u32x4{0u, 0u, 0u, 0u};
  } else {
    load_slice(ubeg, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (AFFINE && tid < kTN) sN[tid] = bias;
  if constexpr (ONE) {
    u32x4 w1[RW];
#pragma unroll
    for (int t = 0; t < RW; ++t) w1[t] = load_w(t, 0);
#pragma unroll
    for (int t = 0; t < RW; ++t) store_w(t, w1[t]);
  }
  if constexpr (DMA) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  } else {
    store_slice();
    __syncthreads();
  }

  uint32_t to_other = kDmaSlot;   // DMA: from the slot that is read to the other
  double stat_sum[2] = {0.0, 0.0};   // STATS: this lane's sums of two channels over the group's units

  for (int unit = ubeg; unit < uend; ++unit) {
    int n0, r0, nvalid;
    unit_geom(unit, n0, r0, nvalid);
    const long out_base = ((long)n0 * H + r0) * W;   // the unit's positions are contiguous rows of `out`
    const int npos = nvalid * R * W;                 // live positions of this unit

    v16f acc[MA][NB];
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    // epilogue operands of the input gradient (mask; addend or the old output), one 16-byte piece per position of a block row a,
    // in two sets.  MA = 4: the first set is fetched during the last taps, the others one block row ahead.  MA = 2 (256
    // registers per lane): a full set that is live inside the tap loop spills, so both block rows are fetched when the
    // loop has ended and the other workgroup's matrix instructions cover the wait; with the mask as bits the first one does
    // travel under the last taps (except on 8-wide maps, where the seventh patch piece takes the room).
    u32x4 em[2][BWD && !BITS ? NR : 1], ea[2][BWD ? NR : 1];
    uint8_t eb[2][NR];   // BITS: the mask bits of this lane's channels
    // element or byte `unit's + lane's` of a tensor with `per` of them per position
    auto lane_at = [&](int per, int c) { return (uint32_t)(lane_pos * per + c); };
    auto load_epi = [&](int a, int set) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const bool in = lane_pos + place(a, r) < npos && col0 + lane_c < p.N;
        const size_t unit_at = (size_t)(out_base + place(a, r)) * p.N + col0;
        if (BITS) eb[set][r] = *(in ? p.mask_bits + (unit_at >> 3) + lane_at(p.N >> 3, lane_c >> 3) : static_cast<const uint8_t*>(p.zero));
        if (!BITS) em[set][r] = *reinterpret_cast<const u32x4*>((in && p.mask) ? p.mask + unit_at + lane_at(p.N, lane_c) : zp);
        const bf16_t* other = p.addend ? p.addend : (p.accumulate ? p.out : nullptr);
        ea[set][r] = *reinterpret_cast<const u32x4*>((in && other) ? other + unit_at + lane_at(p.N, lane_c) : zp);
      }
    };

    if constexpr (DMA) {
      // sixteen channels: nine taps, the next tap's fragments read under this one's matrix instructions
      auto sixteen = [&](auto which) {
        constexpr uint32_t half = decltype(which)::value;
        const uint32_t wl = lds0 + 2 * kDmaSlot + half * dma_weights(NB) + lane * 16;
        auto read = [](uint32_t at) {
          typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
          return as_bf16x8(*(lds_u32x4*)(uintptr_t)at);
        };
        uint32_t second_half = half * 32;
        if (half) asm volatile("" : "+s"(second_half));   // (as above)
        auto patch_at = [&](int tap, int a) { return half ? xaddr[DMA ? tap : 0][a] ^ second_half : xaddr[DMA ? tap : 0][a]; };
        auto tap_of = [](int t) { return 8 - t; };   // the last tap first
        bf16x8 fa[2][MA], fb[2][NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) fb[0][b] = read(wl + (tap_of(0) * NB + b) * 1024);
#pragma unroll
        for (int a = 0; a < MA; ++a) fa[0][a] = read(patch_at(tap_of(0), a));
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const int cur = tap & 1, nxt = cur ^ 1;
          if (tap < 8) {
#pragma unroll
            for (int b = 0; b < NB; ++b) fb[nxt][b] = read(wl + (tap_of(tap + 1) * NB + b) * 1024);
#pragma unroll
            for (int a = 0; a < MA; ++a) fa[nxt][a] = read(patch_at(tap_of(tap + 1), a));
          }
#pragma unroll
          for (int a = 0; a < MA; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][b], fa[cur][a], acc[a][b], 0, 0, 0);
          if (tap < 8) {
#pragma unroll
            for (int i = 0; i < MA * NB; ++i) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction
              __builtin_amdgcn_sched_group_barrier(0x100, NB == 2 ? 1 : 2, 0);   // ... and a read or two
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
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
        if (BWD && BITS && last) {
          load_epi(0, 0);
          load_epi(1, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        sixteen(std::integral_constant<uint32_t, 1>{});
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
          for (int a = 0; a < MA; ++a) xaddr[DMA ? t : 0][a] += to_other;
        to_other = -to_other;
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the next unit's first slice, before results are stored
    } else {
      for (int cs = 0; cs < nslice; ++cs) {
        const bool last_slice = cs + 1 == nslice, more = !STOP || !last_slice || unit + 1 < uend;
        // the next slice (of this unit, or the first of the next unit) sets out now: it is needed when this one ends
        if (more) load_slice(last_slice ? min(unit + 1, uend - 1) : unit, last_slice ? 0 : cs + 1);
        bf16x8 fa[2][MA], fb[2][NB];   // two fragment sets: one feeds the matrix pipe while the other is read
        {
          const int toff0 = (p.flip ? 2 * PW + 2 : 0) * kRow;
#pragma unroll
          for (int b = 0; b < NB; ++b) fb[0][b] = as_bf16x8(*reinterpret_cast<const u32x4*>(wfrag + b * 32 * kRow));
#pragma unroll
          for (int a = 0; a < MA; ++a) fa[0][a] = as_bf16x8(*reinterpret_cast<const u32x4*>(sP + pbase[a] + toff0));
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const int u = tap / 3, v = tap - u * 3;
          const int toff = (p.flip ? (2 - u) * PW + (2 - v) : u * PW + v) * kRow;
          const int un = (tap + 1) / 3, vn = (tap + 1) - un * 3;
          const int toff_next = (p.flip ? (2 - un) * PW + (2 - vn) : un * PW + vn) * kRow;
          if (BWD && (MA == 4 || (BITS && !W8 && !STATS)) && tap == 6 && last_slice) load_epi(0, 0);
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            const int step = tap * KK + kk;
            const int cur = step & 1, nxt = cur ^ 1;
            // (read in the order of first use: both weight fragments, then the patch fragments)
            if (kk + 1 < KK) {
#pragma unroll
              for (int b = 0; b < NB; ++b)
                fb[nxt][b] = as_bf16x8(*reinterpret_cast<const u32x4*>(wfrag + (tap * kTN + b * 32) * kRow + (kk + 1) * 16));
#pragma unroll
              for (int a = 0; a < MA; ++a)
                fa[nxt][a] = as_bf16x8(*reinterpret_cast<const u32x4*>(sP + pbase[a] + toff + (kk + 1) * 16));
            } else if (tap < 8) {
#pragma unroll
              for (int b = 0; b < NB; ++b)
                fb[nxt][b] = as_bf16x8(*reinterpret_cast<const u32x4*>(wfrag + ((tap + 1) * kTN + b * 32) * kRow));
#pragma unroll
              for (int a = 0; a < MA; ++a)
                fa[nxt][a] = as_bf16x8(*reinterpret_cast<const u32x4*>(sP + pbase[a] + toff_next));
            }
            // transposed product: rows = output channels, columns = positions
#pragma unroll
            for (int a = 0; a < MA; ++a)
#pragma unroll
              for (int b = 0; b < NB; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][b], fa[cur][a], acc[a][b], 0, 0, 0);
            // issue order of this step: a fragment read of the next step behind each of the first matrix
            // instructions (left to itself the scheduler reads every fragment right before its use and waits)
            if (step + 1 < 9 * KK) {
#pragma unroll
              for (int i = 0; i < MA + NB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
              }
              if (MA * NB > MA + NB) __builtin_amdgcn_sched_group_barrier(0x008, MA * NB - MA - NB, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        // the slice is done: the next one replaces patch and weights once every wavefront has read its last fragment
        if (more) {
          __syncthreads();
          store_slice();
          __syncthreads();
        }
      }
    }

    // ---- epilogue, straight from registers, in whole lines (lines_device.h).  Register v of block (a, b) in lane (j, h) is channel
    // b*32 + 8 (v/4) + 4 h + v%4 of the position that lane took; afterwards a lane has channels lane_c .. +7 of positions place(a, r).
    // POOL: of a 2 x 2 window the rows are a lane's r and r + 1 (their lanes' bit 4, also in the orders that 8-wide maps are taken in),
    // the columns two neighbouring lanes', of which each does half of the eight channels.  Values as stored, none negative.
    auto pool_rows = [&](int a, int r, const u32x4& upper, const u32x4& lower) {
      const bool odd = lane & 1;
      // of the even and of the odd lane's column, this lane's half of the channels
      auto left = [&](const u32x4& v, int d) {
        const uint32_t even = beside<0xA0>(v[2 + d]);      // (all lanes take part)
        return odd ? even : v[d];
      };
      auto right = [&](const u32x4& v, int d) {
        const uint32_t other = beside<0xF5>(v[d]);
        return odd ? v[2 + d] : other;
      };
      uint32_t m[2], c2[2];
#pragma unroll
      for (int d = 0; d < 2; ++d) m[d] = pool_pair(left(upper, d), right(upper, d), left(lower, d), right(lower, d), c2[d]);
      if (lane_pos + place(a, r) < npos && col0 + lane_c < p.N) {
        // (a pair of rows of 8 or 16 is 4 or 8 pooled positions)
        const int ahead = W8 ? place(a, r) / 4 : place(a, r) / 32 * 8 + place(a, r) % 32 / 2;
        const size_t unit_at = ((((size_t)n0 * H + r0) >> 1) * (W >> 1) + ahead) * p.N + col0;
        const uint32_t lane_to = lane_pooled * p.N + lane_c + (odd ? 4 : 0);
        *reinterpret_cast<u32x2*>(p.pool + unit_at + lane_to) = u32x2{m[0], m[1]};
        *reinterpret_cast<uint32_t*>(p.pool_code + unit_at + lane_to) = __builtin_amdgcn_perm(c2[1], c2[0], 0x06040200u);
      }
    };
    // (offsets formed from these before the units would be kept in registers all along, and do not fit)
    if (STATS || POOL) asm("" : "+v"(lane_pos), "+v"(lane_c));
    constexpr bool early = DMA ? BITS : BITS && !W8 && !STATS;
    if (BWD && MA == 2 && !early) load_epi(0, 0);
    if (BWD && MA == 2 && !(DMA && early)) load_epi(1, 1);
    u32x4 xs[MA][STATS && BWD ? NR : 1];   // STATS and BWD: the batch norm's input at this lane's positions
    auto load_x = [&](int a) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
        xs[a][STATS && BWD ? r : 0] = *reinterpret_cast<const u32x4*>(
            lane_pos + place(a, r) < npos ? p.stat_x + (size_t)(out_base + place(a, r)) * p.N + col0 + lane_at(p.N, lane_c) : zp);
    };
    if (STATS && BWD) load_x(0);
    if (STATS && BWD && DMA) load_x(1);
    u32x2 codes[UNPOOL ? MA : 1][NR];
    if constexpr (UNPOOL) {
      if (p.unpool) {
#pragma unroll
        for (int a = 0; a < MA; ++a)
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            const bool in = lane_pos + place(a, r) < npos && col0 + lane_c < p.N;
            codes[a][r] = *reinterpret_cast<const u32x2*>(in ? p.unpool_code + (size_t)(out_base + place(a, r)) * p.N + col0 +
                                                                   lane_at(p.N, lane_c)
                                                             : static_cast<const uint8_t*>(p.zero));
          }
      }
    }
    u32x4 kept[STATS ? MA : 1][NR];   // what was stored
#pragma unroll
    for (int a = 0; a < MA; ++a) {
      if (BWD && MA == 4 && a + 1 < MA) load_epi(a + 1, (a + 1) & 1);
      if (STATS && BWD && !DMA && a == 1) {   // (both block rows' at once would spill; with the seventh patch piece of 8-wide maps, either)
        if (W8) load_x(0);
        load_x(1);
      }
      u32x4(&stored)[NR] = kept[STATS ? a : 0];
      if constexpr (BWD) {
        float val[NR][8];
        lines_of<NB>(acc[a], val);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const u32x4 mk = em[a & 1][BITS ? 0 : r], ad = ea[a & 1][r];
          float(&v)[8] = val[r];
          if (p.addend) {
#pragma unroll
            for (int d = 0; d < 4; ++d) { v[2 * d] += bf16_lo(ad[d]); v[2 * d + 1] += bf16_hi(ad[d]); }
          }
          if (BITS) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = ((eb[a & 1][r] >> e) & 1u) ? v[e] : 0.f;
          } else if (p.mask) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              v[2 * d] = bf16_lo(mk[d]) > 0.f ? v[2 * d] : 0.f;
              v[2 * d + 1] = bf16_hi(mk[d]) > 0.f ? v[2 * d + 1] : 0.f;
            }
          }
          if (p.accumulate) {
#pragma unroll
            for (int d = 0; d < 4; ++d) { v[2 * d] += bf16_lo(ad[d]); v[2 * d + 1] += bf16_hi(ad[d]); }
          }
#pragma unroll
          for (int d = 0; d < 4; ++d) stored[r][d] = pack_bf16(v[2 * d], v[2 * d + 1]);
        }
      } else {
        if (AFFINE && p.bias) {
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int o = 0; o < 4; ++o) {
              const v4f add = *reinterpret_cast<const v4f*>(sN + b * 32 + o * 8 + h * 4);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[a][b][4 * o + e] += add[e];
            }
        }
        if (AFFINE && (POOL || p.relu)) {
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = fmaxf(acc[a][b][v], 0.f);   // (zero for NaN, as v > 0 ? v : 0)
        }
        uint32_t w[NB][8];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int d = 0; d < 8; ++d) w[b][d] = pack_bf16(acc[a][b][2 * d], acc[a][b][2 * d + 1]);
        lines_of<NB>(w, stored);
      }
#pragma unroll
      for (int r = 0; r < NR; ++r)   // N is a multiple of 8 (STATS: of 64): a piece is wholly inside or outside
        if (lane_pos + place(a, r) < npos && (STATS || col0 + lane_c < p.N))
          *reinterpret_cast<u32x4*>(p.out + (size_t)(out_base + place(a, r)) * p.N + col0 + lane_at(p.N, lane_c)) = stored[r];
      if constexpr (UNPOOL) {
        if (p.unpool) {
#pragma unroll
          for (int r = 0; r < NR; ++r)
            if (lane_pos + place(a, r) < npos && col0 + lane_c < p.N)
              unpool_store<4>(p.unpool, (size_t)out_base + (lane_pos + place(a, r)), (lane_pos + place(a, r)) & (W - 1), W, p.N, col0 + lane_c,
                           stored[r], codes[a][r]);
        }
      }
      if constexpr (POOL) {
#pragma unroll
        for (int r = 0; r < NR; r += 2) pool_rows(a, r, stored[r], stored[r + 1]);
      }
    }
    if constexpr (STATS) {
      __builtin_amdgcn_sched_barrier(0);   // (conversions to double drawn up into the loop above would spill)
      double t[2][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) t[0][e] = t[1][e] = 0.0;
      v4f mean[2];
      if (BWD) {
#pragma unroll
        for (int d = 0; d < 2; ++d) mean[d] = *reinterpret_cast<const v4f*>(sN + lane_c + 4 * d);
      }
#pragma unroll
      for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          if (lane_pos + place(a, r) >= npos) continue;
          if (BWD) bn_sums_add(t, kept[a][r], xs[a][r], mean);
          else bn_sums_add(t, kept[a][r]);
        }
      lines_sums(t, lane, stat_sum);
    }
  }
  if constexpr (DMA) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may be on its way to LDS when it is used again
  if (STATS) {
    // the four wavefronts' sums meet in LDS (once nobody reads patch or weights any more), added in wavefront order
    __syncthreads();
    double* red = reinterpret_cast<double*>(smemW);   // [4][2][64]
#pragma unroll
    for (int i = 0; i < 2; ++i) red[(wave * 2 + lines_sum(lane)) * 64 + lines_sum_channel(lane) + i] = stat_sum[i];
    __syncthreads();
    if (tid < 128) {
      const int c = tid & 63, w = tid >> 6;
      const double tot = ((red[(0 * 2 + w) * 64 + c] + red[(1 * 2 + w) * 64 + c]) + red[(2 * 2 + w) * 64 + c]) +
                         red[(3 * 2 + w) * 64 + c];
      const double factor = BWD && w == 1 ? (double)sN[kTN + c] : 1.0;
      if (col0 + c < p.N) p.stat_partial[((size_t)group * p.N + col0 + c) * 2 + w] = tot * factor;
    }
  }
}

template <int MA, int NP, bool W8, bool BWD, bool STATS, bool BITS, int NB = 2, bool POOL = false, bool ONE = false>
void launch_variant(hipStream_t st, const WideParams& p, dim3 grid, size_t lds) {
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&conv3_wide_kernel<MA, NP, W8, BWD, STATS, BITS, NB, POOL, ONE>), kLdsOfComputeUnit);
  hipLaunchKernelGGL((conv3_wide_kernel<MA, NP, W8, BWD, STATS, BITS, NB, POOL, ONE>), grid, dim3(kThreads), lds, st, p);
}

// without mask and sums: with pooling, on the narrow tile, with a single slice
template <int MA, int NP, bool W8, int NB>
void launch_plain(hipStream_t st, const WideParams& p, dim3 grid, size_t lds) {
  auto launch = [&](auto one) {
    constexpr bool ONE = decltype(one)::value;
    if (p.pool) launch_variant<MA, NP, W8, false, false, false, NB, true, ONE>(st, p, grid, lds);
    else launch_variant<MA, NP, W8, false, false, false, NB, false, ONE>(st, p, grid, lds);
  };
  if constexpr (NP > 0) {
    if (p.Cs == KC) return launch(std::true_type{});
  }
  launch(std::false_type{});
}

template <int MA, int NP, bool W8>
void launch_wide(hipStream_t st, const WideParams& p, dim3 grid, size_t lds, bool bwd, bool stats) {
  if (bwd) {
    if constexpr (MA == 2) {
      if (stats) return launch_variant<MA, NP, W8, true, true, true>(st, p, grid, lds);
    }
    if (p.mask_bits) return launch_variant<MA, NP, W8, true, false, true>(st, p, grid, lds);
    return launch_variant<MA, NP, W8, true, false, false>(st, p, grid, lds);
  }
  if constexpr (MA == 2) {
    if (stats) return launch_variant<MA, NP, W8, false, true, false>(st, p, grid, lds);
    return launch_plain<MA, NP, W8, 2>(st, p, grid, lds);
  }
  launch_variant<MA, NP, W8, false, false, false>(st, p, grid, lds);
}

}  // namespace

namespace {
// Unit geometry for units of `unit` positions: R rows of nimg images; false if the map does not tile that way.
bool unit_shape(int H, int W, int unit, int& R, int& nimg) {
  if (W < 4 || W > unit || unit % W != 0) return false;
  R = std::min(H, unit / W);
  if (H % R != 0 || unit % (R * W) != 0) return false;
  nimg = unit / (R * W);
  return (nimg == 1 || R == H) && nimg <= 255;
}
}  // namespace

// Whether conv3_wide_bf16 takes the layer with weights in operand order (ConvGeom::frag = 2), staged by loads that write LDS: maps 8, 16
// and 32 wide, whole blocks of 32 channels in and out, two slices of the reduction or more (a single one, 32 -> 64 on 16x16 with
// pooling, 1024 images: 23.0 us, and 20.3 in the variant whose weights stay in LDS).  pooled: forward with a max pooling behind;
// relu: after the product; share: as input gradient, a mask or another share to add.
bool conv3_wide_takes(const ConvGeom& g, int N, bool pooled, bool relu, bool share) {
  const int H = g.Hs, W = g.Ws;
  if (g.raw3 || g.ks != 3 || g.stride != 1 || g.pad != 1 || g.Hp != H || g.Wp != W || (W != 8 && W != 16 && W != 32)) return false;
  if (g.Cs % KC != 0 || g.Cs < 2 * KC || N % 32 != 0 || (long)g.rows * H * W * std::max(g.Cs, N) >= (1L << 31)) return false;
  int R, nimg;
  if (!unit_shape(H, W, 256, R, nimg) || nimg * (R + 2) * W > kDmaPatch) return false;
  if (N == 32 && share) return false;
  if (pooled && (!relu || W == 32 || H % 2 != 0 || R % 2 != 0 || (W == 8 && R % 8 != 0))) return false;
  const long units = nimg == 1 ? (long)g.rows * (H / R) : (g.rows + nimg - 1) / nimg;
  if (H > R && !reciprocal_below(H / R, units)) return false;
  return units * ((N + 63) / 64) >= 32;
}

bool conv3_wide_bf16(hipStream_t st, const bf16_t* src, const bf16_t* wgt, bf16_t* out, int M, int N,
                     const ConvGeom& g, const float* bias, const bf16_t* mask, bool relu, bool accumulate,
                     const bf16_t* addend, bf16_t* pool, uint8_t* pool_code, BnStatRequest* stats,
                     UnpoolRequest* unpool) {
  const bool dma = g.frag == 2;   // (conv3_wide_takes has said yes)
  const int H = g.Hs, W = g.Ws;
  if (g.raw3 || g.ks != 3 || g.stride != 1 || g.pad != 1 || g.Hp != H || g.Wp != W) return false;
  if (g.Cs % 32 != 0 || N % 8 != 0 || (long)g.rows * H * W != M) return false;
  if ((long)M * std::max(g.Cs, N) >= (1L << 31)) return false;   // 32-bit element offsets in the kernel
  int nb = N <= 32 ? 1 : 2;
  if (dma && nb == 1) stats = nullptr;   // (not taken: the narrow tile has no sums)
  // Units of 256 positions with two workgroups per compute unit where both fit LDS (one workgroup's loads,
  // stores and epilogue then run under the other's matrix instructions); units of 512 with one otherwise.
  // Two 256-register kernels also share a SIMD with the weight-gradient kernels of the side streams; a
  // 512-register wavefront has its SIMD to itself, and the two chains then merely take turns.
  const bool bwd = mask || addend || accumulate;
  if (bwd && (bias || relu)) return false;   // the input-gradient epilogue carries neither (32 registers it needs elsewhere)
  // pooling: the windows of 16- and 8-wide maps lie in lanes that can exchange them; the others stay with kernel D
  const bool pooling = pool && pool_code, plain = !bwd && !stats;
  // (after a ReLU, whose values compare as integers).
  if (pooling && (bwd || g.transposed || stats || !relu || (W != 16 && W != 8) || H % 2 != 0)) return false;
  if (nb == 1 && (bwd || stats)) return false;
  int ma = 0, R = 0, nimg = 0, npatch = 0;
  for (int cand : {2, 4}) {
    int r, n;
    if (!unit_shape(H, W, 128 * cand, r, n)) continue;
    if ((nb == 1 || pooling) && cand == 4) continue;
    if (pooling && (r % 2 != 0 || (W == 8 && r % 8 != 0))) continue;
    if (dma) {
      ma = 2; R = r; nimg = n;
      break;
    }
    const int np_ = n * (r + 2) * (W + 2);
    const size_t l = ((size_t)np_ + 9 * 64) * kRow * sizeof(bf16_t);   // patch + the nine taps' weights of a slice
    if (l + 2 * 64 * sizeof(float) > kLdsOfComputeUnit / (cand == 2 ? 2 : 1)) continue;
    ma = cand; R = r; nimg = n; npatch = np_;
    break;
  }
  if (!ma) return false;
  const int units = nimg == 1 ? g.rows * (H / R) : (g.rows + nimg - 1) / nimg;
  const uint32_t by_units = reciprocal_below(H / R, units);
  if (H > R && !by_units) return false;   // (few images of a great many rows: the other kernels divide)
  // Where 64 channels per workgroup leave a compute unit with one or none: 32, so that one's loads run under another's
  // instructions (1024 images, 128 -> 64 on 8x8, alone: 16.65 -> 15.9 us).
  if (plain && ma == 2 && (long)units * ((N + 63) / 64) <= 256) nb = 1;
  const int kTN = 32 * nb, tiles_n = (N + kTN - 1) / kTN;
  const size_t lds = (dma ? dma_lds(nb) : ((size_t)npatch + 9 * kTN) * kRow * sizeof(bf16_t)) + 2 * kTN * sizeof(float);
  if ((long)units * tiles_n < 32) return false;   // too little work to fill the chip this way: the generic kernels spread it better
  const bool w8 = W == 8 && R % (dma ? 4 : 8) == 0;
  const int need = (npatch * OC + kThreads - 1) / kThreads;   // patch pieces per thread
  WideParams p{};
  p.src = src; p.wgt = wgt; p.out = out; p.rows = g.rows; p.H = H; p.W = W; p.Cs = g.Cs; p.N = N;
  p.R = R; p.nimg = nimg; p.flip = g.transposed ? 1 : 0; p.zero = g.zero;
  p.bias = bias; p.mask = mask; p.addend = addend; p.relu = relu ? 1 : 0; p.accumulate = accumulate ? 1 : 0;
  p.mask_bits = (bwd && mask && N % kTN == 0) ? g.mask_bits : nullptr;
  // several units per workgroup (the next unit's patch and weights travel under the current one's taps) while
  // the grid still covers the chip a few times over
  int upw = 1;
  while (upw < 8 && (long)units * tiles_n / (upw * 2) >= (ma == 2 ? 2048 : 1024)) upw *= 2;
  // (a single slice: the weights are fetched once per workgroup, so no more of them than are resident)
  if (plain && ma == 2 && g.Cs == KC) {
    const long resident = nb == 1 ? 768 : 512;
    upw = (int)std::max(1L, ((long)units * tiles_n + resident - 1) / resident);
  }
  if (pooling) { p.pool = pool; p.pool_code = pool_code; }
  const bool unpooling = unpool && g.transposed && ma == 2 && plain && !pooling && (dma || g.Cs == KC);
  if (unpooling) { p.unpool = unpool->din; p.unpool_code = unpool->code; }
  // Batch-norm sums on the way out: no bias, no ReLU, and units and groups that do not cross from one worker to the next,
  // few enough groups for the statistics scratch.
  bool with_stats = false;
  p.gK = 1;
  p.ufirst[0] = 0; p.ufirst[1] = units;
  p.ifirst[0] = 0; p.ifirst[1] = g.rows;
  if (stats && stats->partial && stats->seg && ma == 2 && bwd == (stats->x != nullptr) && (!bwd || p.mask_bits) && !bias &&
      !relu && N % kTN == 0 && stats->seg->off[stats->seg->K] == g.rows) {
    const Segments& seg = *stats->seg;
    auto units_of = [&](int k) {
      const long rows = seg.off[k + 1] - seg.off[k];
      return nimg == 1 ? rows * (H / R) : (rows + nimg - 1) / nimg;
    };
    int u = upw;
    auto groups_at = [&](int per) {
      long n = 0;
      for (int k = 0; k < seg.K; ++k) n += (units_of(k) + per - 1) / per;
      return n;
    };
    while (groups_at(u) > (long)seg.K * kBnMaxSplits && u < 64) u *= 2;
    if (groups_at(u) <= (long)seg.K * kBnMaxSplits) {
      with_stats = true;
      upw = u;
      p.gK = seg.K;
      for (int k = 0; k < seg.K; ++k) p.ufirst[k + 1] = p.ufirst[k] + (int)units_of(k);
      for (int k = 0; k <= seg.K; ++k) p.ifirst[k] = seg.off[k];
      p.stat_partial = stats->partial;
      p.stat_x = stats->x;
      p.stat_norm = stats->stats;
    }
  }
  p.units = p.ufirst[p.gK]; p.upw = upw;
  auto reciprocal = [](int d) { return (uint32_t)(((1 << 22) + d - 1) / d); };   // (exact: positions and divisors below 2^11)
  p.by_patch = reciprocal((R + 2) * (W + 2)); p.by_row = reciprocal(W + 2); p.by_rows = reciprocal(R + 2); p.by_r = reciprocal(R);
  p.by_units = by_units;
  while ((1 << p.wlog) < W) ++p.wlog;
  p.gfirst[0] = 0;
  for (int k = 0; k < p.gK; ++k) p.gfirst[k + 1] = p.gfirst[k] + (p.ufirst[k + 1] - p.ufirst[k] + upw - 1) / upw;
  const int groups = p.groups = p.gfirst[p.gK];
  const dim3 grid(((groups + 7) / 8) * 8 * tiles_n);   // whole rounds of 8 groups: see the kernel's index mapping
  if (dma) {
    if (nb == 1) {
      if (w8) launch_plain<2, 0, true, 1>(st, p, grid, lds);
      else launch_plain<2, 0, false, 1>(st, p, grid, lds);
    } else {
      if (w8) launch_wide<2, 0, true>(st, p, grid, lds, bwd, with_stats);
      else launch_wide<2, 0, false>(st, p, grid, lds, bwd, with_stats);
    }
  } else if (nb == 1) {
    if (w8 && need <= 7) launch_plain<2, 7, true, 1>(st, p, grid, lds);
    else if (!w8 && need <= 6) launch_plain<2, 6, false, 1>(st, p, grid, lds);
    else return false;
  } else if (ma == 2) {
    if (w8 && need <= 7) launch_wide<2, 7, true>(st, p, grid, lds, bwd, with_stats);
    else if (!w8 && need <= 6) launch_wide<2, 6, false>(st, p, grid, lds, bwd, with_stats);
    else return false;
  } else {
    if (w8 && need <= 13) launch_wide<4, 13, true>(st, p, grid, lds, bwd, false);
    else if (!w8 && need <= 11) launch_wide<4, 11, false>(st, p, grid, lds, bwd, false);
    else if (!w8 && need <= 18) launch_wide<4, 18, false>(st, p, grid, lds, bwd, false);
    else return false;
  }
  if (unpooling) unpool->done = true;
  if (with_stats) {
    for (int k = 0; k <= p.gK; ++k) stats->table.first[k] = p.gfirst[k];
    stats->done = true;
  }
  return true;
}

}  // namespace omni
