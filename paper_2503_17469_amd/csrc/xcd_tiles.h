// Which output tile a workgroup of a matrix product takes.  Workgroup b runs on XCD b % 8, and every XCD has an L2 of its
// own, so the tiles of an XCD should share operands: it takes a rectangle of them.  (Dealt out in turn, with a power of
// two of row tiles, every XCD read all of the weights: 128 rows, 3072 -> 1024 in fp32 took 17.7 us, now 13.3.)
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "quotient.h"

namespace omni {

struct XcdTiles {
  int tiles_m, tiles_n;   // all tiles
  int cm, cn;             // an XCD's rectangle
  int lsm;                // 2^lsm XCDs along m, 8 >> lsm along n
  uint32_t by_cm;         // reciprocal_below(cm)
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
  best.by_cm = reciprocal_below(best.cm, (uint64_t)best.cm * best.cn);
  return best;
}

// False: this workgroup has no tile.  (Row tiles fastest.)
__device__ __forceinline__ bool xcd_tile(const XcdTiles& x, int b, int& tile_m, int& tile_n) {
  const int xcd = b & 7, local = b >> 3;
  const int ln = quotient(local, x.by_cm, x.cm), lm = local - ln * x.cm;
  const int xn = xcd >> x.lsm, xm = xcd - (xn << x.lsm);
  tile_m = xm * x.cm + lm;
  tile_n = xn * x.cn + ln;
  return tile_m < x.tiles_m && tile_n < x.tiles_n;
}

}  // namespace omni
