// Which output tile a workgroup of a matrix product takes.  Workgroup b runs on XCD b % 8, and every XCD has an L2 of its
// own, so the tiles of an XCD should share operands: it takes a rectangle of them.  (Dealt out in turn, with a power of
// two of row tiles, every XCD read all of the weights: 128 rows, 3072 -> 1024 in fp32 took 17.7 us, now 13.3.)
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace omni {

struct XcdTiles {
  int tiles_m, tiles_n;   // all tiles
  int cm, cn;             // an XCD's rectangle
  int lsm;                // 2^lsm XCDs along m, 8 >> lsm along n
  uint32_t by_cm;         // 2^32 / cm rounded up where that gives every quotient of the rectangle, otherwise 0
  int grid() const { return 8 * cm * cn; }
};

// The rectangle with the fewest tiles, then the one with the shortest sides (the operand panels it reads).
inline XcdTiles xcd_tiles(int tiles_m, int tiles_n) {
  XcdTiles best{};
  for (int lsm = 0; lsm <= 3; ++lsm) {
    const int sm = 1 << lsm, sn = 8 >> lsm;
    const int cm = (tiles_m + sm - 1) / sm, cn = (tiles_n + sn - 1) / sn;
    if (lsm == 0 || cm * cn < best.cm * best.cn || (cm * cn == best.cm * best.cn && cm + cn < best.cm + best.cn))
      best = XcdTiles{tiles_m, tiles_n, cm, cn, lsm, 0};
  }
  if (best.cm > 1 && (uint64_t)best.cm * best.cm * best.cn < 1ull << 32)
    best.by_cm = (uint32_t)(((1ull << 32) + best.cm - 1) / best.cm);
  return best;
}

// False: this workgroup has no tile.  (Row tiles fastest.  A run-time division takes 150 to 300 cycles, two of them stood
// in front of every product's first load.)
__device__ __forceinline__ bool xcd_tile(const XcdTiles& x, int b, int& tile_m, int& tile_n) {
  const int xcd = b & 7, local = b >> 3;
  const int ln = x.cm == 1 ? local : x.by_cm ? (int)__umulhi((uint32_t)local, x.by_cm) : local / x.cm, lm = local - ln * x.cm;
  const int xn = xcd >> x.lsm, xm = xcd - (xn << x.lsm);
  tile_m = xm * x.cm + lm;
  tile_n = xn * x.cn + ln;
  return tile_m < x.tiles_m && tile_n < x.tiles_n;
}

}  // namespace omni
