// Forward convolutions in bf16 (fp32 accumulation) that meet only part of their input's rows or columns at a tap, or have one tap: 3x3 and
// 1x1 at stride 2, 1x1 at stride 1 (the inner F(.) of the gradient line of procedure Train, Algorithm 1).
//
//   out[m][co] = sum_{u,v,ci} src[n, h s + u - pad, w s + v - pad, ci] * wgt[co][u][v][ci]
//
// A workgroup takes tiles of 256 output positions x 128 channels, a wavefront 128 x 64 of them, in steps of one tap and 32 channels.
// A stride of 2 makes a patch of the input four times the outputs, too large to lie in LDS twice; instead every step gathers the 256
// rows of its tap, 64 bytes each, straight into LDS, where a row lies as the matrix instruction's operand wants it (pieces
// moved by xor), beside the tap's weights in operand order.  Three steps' buffers: the step after next is on its way while this
// one is multiplied, waited for by count, one barrier per step, across tiles as well.  The batch norm that follows gets its
// sums from the epilogue.
//
// 2048 images of the ResNet-18 shape, 3x3 and 1x1 together, us, from 64, 128 and 256 channels: 251, 190 and 149 in the general kernel
// and 53, 32 and 21 for the sums' pass -> 236, 160 and 155 with them (the step 11.11 -> 10.98 ms), 219, 157 and 152 with the results in whole
// lines.  The address unit is busy for 0.73 of the first: a gathered half line costs as much as a whole one.
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
constexpr int kTM = 256, kTN = 128;   // positions and channels per tile
constexpr int KC = 32;                // reduction channels per step
constexpr uint32_t kRows = kTM * 64;  // bytes of a step's gathered rows
constexpr uint32_t kStep = kRows + kTN * 64;
constexpr uint32_t kSums = 4 * 2 * 64 * sizeof(double);

struct GatherParams {
  const bf16_t* src;   // [rows][Hs][Ws][Cs]
  const bf16_t* wgt;   // operand order: blocks [N/32][ks*ks][Cs/16]
  bf16_t* out;         // [rows*Hp*Wp][N]
  int rows, Hs, Ws, Cs, N, Hp, Wp;
  int ks, stride, pad, relu;
  uint32_t by_image, by_row;   // reciprocals of Hp * Wp and of Wp
  const void* zero;
  const float* bias;
  // Group g takes tpg tiles of one entry: entry k owns the positions mfirst[k] .. mfirst[k+1]-1, in tiles tfirst[k] .. tfirst[k+1]-1 from
  // its first position on, and the groups gfirst[k] .. gfirst[k+1]-1.  One entry, or one per worker for the sums.
  int gK, groups, tpg;
  int32_t gfirst[OMNI_MAX_WORKERS + 1], tfirst[OMNI_MAX_WORKERS + 1], mfirst[OMNI_MAX_WORKERS + 1];
  double* stat_partial;   // STATS: [group][N][2] sums of the stored output and of its squares
};

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

template <bool STATS>
__global__ __launch_bounds__(kThreads, 2) void conv_gather_kernel(GatherParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smemG[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 31, h = lane >> 5;
  const int tiles_n = p.N / kTN;
  // (workgroup b runs on XCD b % 8: the channel tiles of a group, which gather the same rows, share one)
  const int on_xcd = blockIdx.x >> 3;
  const int tile_n = on_xcd % tiles_n;
  const int group = (on_xcd / tiles_n) * 8 + (blockIdx.x & 7);
  if (group >= p.groups) return;
  int gk = 0;
  if (STATS) gk = __popcll(__ballot(lane < p.gK && p.gfirst[lane] <= group)) - 1;
  const int mend = p.mfirst[gk + 1];
  const int tbeg = (group - p.gfirst[gk]) * p.tpg, tend = min(p.tfirst[gk + 1] - p.tfirst[gk], tbeg + p.tpg);
  const int m0 = p.mfirst[gk];
  const int col0 = tile_n * kTN;
  const int taps = p.ks * p.ks, nslice = p.Cs / KC, spt = taps * nslice, c16n = p.Cs >> 4;
  const uint32_t lds0 = lds_address(smemG);
  const bf16_t* const zp = static_cast<const bf16_t*>(p.zero);

  // ---- loads of the step that is next in turn: rows wave * 64 + 16 i + lane / 4, and the weights of channels 32 wave on
  int row_at[4];        // element of tap (0, 0) (before the tensor, perhaps), and its row and column
  int row_hw[4];
  const bf16_t* row_ptr[4];
  uint32_t row_in = 0;
  int ltile = tbeg, ltap = 0, lu = 0, lv = 0, lslice = 0;
  uint32_t lbuf = 0;
  const char* wsrc = nullptr;
  auto load_tile = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = wave * 64 + 16 * i + (lane >> 2);
      const int m = m0 + ltile * kTM + r;
      const int n = quotient(m, p.by_image, p.Hp * p.Wp), rem = m - n * (p.Hp * p.Wp);
      const int y = quotient(rem, p.by_row, p.Wp), hh = y * p.stride - p.pad, ww = (rem - y * p.Wp) * p.stride - p.pad;
      row_at[i] = ((n * p.Hs + hh) * p.Ws + ww) * p.Cs + ((lane & 3) ^ (r >> 2 & 3)) * 8;
      row_hw[i] = m < mend && ltile < tend ? (hh << 16) | (ww & 0xffff) : (int)0x80000000;
    }
  };
  auto load_tap = [&]() {
    row_in = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int hh = (row_hw[i] >> 16) + lu, ww = (int)(int16_t)row_hw[i] + lv;
      const bool in = hh >= 0 && hh < p.Hs && ww >= 0 && ww < p.Ws;
      row_ptr[i] = in ? p.src + (row_at[i] + (lu * p.Ws + lv) * p.Cs) : zp;
      row_in |= (in ? 1u : 0u) << i;
    }
    wsrc = reinterpret_cast<const char*>(p.wgt) + ((size_t)(((col0 >> 5) + wave) * taps + ltap) * c16n << 10);
  };
  auto load_step = [&]() {
    const uint32_t to = lds0 + lbuf;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      load_to_lds(row_ptr[i], to + (wave * 4 + i) * 1024);
      row_ptr[i] += (row_in >> i & 1u) * KC;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) load_to_lds(wsrc, lane * 16 + i * 1024, to + kRows + (wave * 2 + i) * 1024);
    wsrc += 2048;
    lbuf = lbuf == 2 * kStep ? 0 : lbuf + kStep;
    if (++lslice == nslice) {
      lslice = 0;
      if (++lv == p.ks) { lv = 0; ++lu; }
      if (++ltap == taps) {
        ltap = 0;
        lu = 0;
        ++ltile;
        load_tile();                                       // (past the last tile: rows that are not there, zeros)
      }
      load_tap();
    }
  };
  load_tile();
  load_tap();
  load_step();
  load_step();

  // ---- fragments: positions wp * 128 + a * 32 + j, channels wc * 64 + b * 32 ..
  const int wp = wave & 1, wc = wave >> 1;
  const uint32_t xlane = lds0 + wp * 8192 + j * 64 + ((h ^ (j >> 2 & 3)) * 16), wlane = lds0 + kRows + wc * 4096 + lane * 16;
  uint32_t buf = 0;
  int ready = 0;   // steps whose data is known to have arrived
  double stat_sum[2] = {0.0, 0.0};
  for (int tile = tbeg; tile < tend; ++tile) {
    v16f acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    for (int s = 0; s < spt; ++s) {
      // own loads of this step (six per step, the next one's under way), then everyone's; the barrier also ends the reading of the
      // buffer that is filled next
      if (ready > 0) {
        --ready;
        asm volatile("s_barrier" ::: "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(6)\n\ts_barrier" ::: "memory");
      }
      load_step();
      __builtin_amdgcn_sched_barrier(0);
      auto read = [](uint32_t at) {
        typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
        return as_bf16x8(*(lds_u32x4*)(uintptr_t)at);
      };
      const uint32_t xa = xlane + buf, xb = xa ^ 32, wa = wlane + buf;
      bf16x8 fa[2][4], fb[2][2];
#pragma unroll
      for (int b = 0; b < 2; ++b) fb[0][b] = read(wa + b * 2048);
#pragma unroll
      for (int a = 0; a < 4; ++a) fa[0][a] = read(xa + a * 2048);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (half == 0) {
#pragma unroll
          for (int b = 0; b < 2; ++b) fb[1][b] = read(wa + b * 2048 + 1024);
#pragma unroll
          for (int a = 0; a < 4; ++a) fa[1][a] = read(xb + a * 2048);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[half][b], fa[half][a], acc[a][b], 0, 0, 0);
        if (half == 0) {
#pragma unroll
          for (int i = 0; i < 6; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // ... and a read
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      buf = buf == 2 * kStep ? 0 : buf + kStep;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the next two steps, before results are stored
    ready = 2;

    // ---- epilogue, straight from registers, in whole lines (lines_device.h): a lane has eight channels at four positions of a block
    int mlane = wp * 128 + lines_base<2>(lane);
    asm volatile("" : "+v"(mlane));                       // (nothing formed from it before)
    const int c0 = wc * 64 + lines_channel<2>(lane), m_tile = m0 + tile * kTM, live = mend - m_tile;
    u32x4 kept[STATS ? 4 : 1][4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      if (!STATS && p.bias) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int o = 0; o < 4; ++o) {
            const v4f add = *reinterpret_cast<const v4f*>(p.bias + col0 + wc * 64 + b * 32 + o * 8 + h * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[a][b][4 * o + e] += add[e];
          }
      }
      if (!STATS && p.relu) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[a][b][v] = fmaxf(acc[a][b][v], 0.f);   // (zero for NaN, as v > 0 ? v : 0)
      }
      uint32_t w[2][8];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int d = 0; d < 8; ++d) w[b][d] = pack_bf16(acc[a][b][2 * d], acc[a][b][2 * d + 1]);
      u32x4(&stored)[4] = kept[STATS ? a : 0];
      lines_of<2>(w, stored);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at = a * 32 + lines_position<2>(r);
        if (mlane + at < live)
          *reinterpret_cast<u32x4*>(p.out + (size_t)(m_tile + at) * p.N + col0 + (uint32_t)(mlane * p.N + c0)) = stored[r];
      }
    }
    if constexpr (STATS) {
      __builtin_amdgcn_sched_barrier(0);                  // (conversions to double drawn up into the loop above would spill)
      double t[2][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) t[0][e] = t[1][e] = 0.0;
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (mlane + a * 32 + lines_position<2>(r) < live) bn_sums_add(t, kept[a][r]);
      lines_sums(t, lane, stat_sum);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // nothing may be on its way to LDS when the workgroup ends
  if (STATS) {
    // the sums of the two wavefronts that have a channel, in wavefront order
    double* red = reinterpret_cast<double*>(smemG + 3 * kStep);   // [4][2][64]
#pragma unroll
    for (int i = 0; i < 2; ++i) red[(wave * 2 + lines_sum(lane)) * 64 + lines_sum_channel(lane) + i] = stat_sum[i];
    __syncthreads();
    const int c = tid & 127, w = tid >> 7, of = c >> 6;
    p.stat_partial[((size_t)group * p.N + col0 + c) * 2 + w] = red[(of * 4 + w) * 64 + (c & 63)] + red[(of * 4 + 2 + w) * 64 + (c & 63)];
  }
}

template <bool STATS>
void launch(hipStream_t st, const GatherParams& p) {
  static LdsLimit limit;
  limit.raise(reinterpret_cast<const void*>(&conv_gather_kernel<STATS>), kLdsOfComputeUnit);
  const dim3 grid(((p.groups + 7) / 8) * 8 * (p.N / kTN));   // whole rounds of 8 groups
  hipLaunchKernelGGL(conv_gather_kernel<STATS>, grid, dim3(kThreads), 3 * kStep + (STATS ? kSums : 0), st, p);
}

}  // namespace

// Whole steps and channel tiles, at least a tile per compute unit, at stride 2 or with one tap.
bool conv_gather_takes(const ConvGeom& g, int N) {
  if (g.raw3 || g.transposed || (g.ks != 1 && g.ks != 3) || (g.stride != 2 && g.ks != 1) || g.stride > 2) return false;
  if (g.Cs % KC != 0 || N % kTN != 0 || g.Hs > 16384 || g.Ws > 16384) return false;
  const long M = (long)g.rows * g.Hp * g.Wp;
  if ((long)g.rows * g.Hs * g.Ws * g.Cs >= (1L << 31) - (1L << 24) || M * N >= (1L << 31)) return false;
  return (M + kTM - 1) / kTM * (N / kTN) >= 256;
}

void conv_gather_bf16(hipStream_t st, const bf16_t* src, const bf16_t* wgt, bf16_t* out, int N, const ConvGeom& g, const float* bias,
                      bool relu, BnStatRequest* stats) {
  GatherParams p{};
  p.src = src; p.wgt = wgt; p.out = out;
  p.rows = g.rows; p.Hs = g.Hs; p.Ws = g.Ws; p.Cs = g.Cs; p.N = N; p.Hp = g.Hp; p.Wp = g.Wp;
  p.ks = g.ks; p.stride = g.stride; p.pad = g.pad; p.relu = relu ? 1 : 0;
  const int hw = g.Hp * g.Wp, M = g.rows * hw;
  p.by_image = reciprocal_below(hw, (uint64_t)M + kTM);
  p.by_row = reciprocal_below(g.Wp, hw);
  p.zero = g.zero; p.bias = bias;
  const int tiles_n = N / kTN;
  auto tiles_of = [](int m) { return (m + kTM - 1) / kTM; };
  int tpg = 1;
  while (tpg < 8 && (long)tiles_of(M) * tiles_n / (tpg * 2) >= 1024) tpg *= 2;
  p.gK = 1;
  p.tfirst[1] = tiles_of(M);
  p.mfirst[1] = M;
  bool with_stats = false;
  if (stats && stats->partial && stats->seg && !stats->x && !bias && !relu && stats->seg->off[stats->seg->K] == g.rows) {
    const Segments& seg = *stats->seg;
    int u = tpg;
    auto groups_at = [&](int per) {
      long n = 0;
      for (int k = 0; k < seg.K; ++k) n += (tiles_of((seg.off[k + 1] - seg.off[k]) * hw) + per - 1) / per;
      return n;
    };
    while (groups_at(u) > (long)seg.K * kBnMaxSplits && u < 64) u *= 2;
    if (groups_at(u) <= (long)seg.K * kBnMaxSplits) {
      with_stats = true;
      tpg = u;
      p.gK = seg.K;
      for (int k = 0; k < seg.K; ++k) p.tfirst[k + 1] = p.tfirst[k] + tiles_of((seg.off[k + 1] - seg.off[k]) * hw);
      for (int k = 0; k <= seg.K; ++k) p.mfirst[k] = seg.off[k] * hw;
      p.stat_partial = stats->partial;
    }
  }
  p.tpg = tpg;
  for (int k = 0; k < p.gK; ++k) p.gfirst[k + 1] = p.gfirst[k] + (p.tfirst[k + 1] - p.tfirst[k] + tpg - 1) / tpg;
  p.groups = p.gfirst[p.gK];
  if (with_stats) launch<true>(st, p);
  else launch<false>(st, p);
  if (with_stats) {
    for (int k = 0; k <= p.gK; ++k) stats->table.first[k] = p.gfirst[k];
    stats->done = true;
  }
}

}  // namespace omni
