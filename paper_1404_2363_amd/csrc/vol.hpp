// Launches of two D3Q15 steps (compiled in vol.hip).
#pragma once

#include "common.hpp"

namespace lbm {

using VolFn = void (*)(const RunArgs&, hipStream_t);

// Tiles built: 64 x 8 and 32 x 16 columns in FP32, 32 x 8 and 32 x 13 in FP64
// (a block's registers leave room for one per CU, of at most 12 waves in FP32
// and 8 in FP64).
constexpr int kVolTiles[2][2][2] = {{{64, 8}, {32, 16}}, {{32, 8}, {32, 13}}};

// The launch over tiles of bx x by columns, or null where it is not built.
VolFn vol_launch(int bx, int by, bool dbl);

// Planes per block and the relative time of a launch over such tiles, from
// the rounds of 256 blocks it takes (256^3 FP64: 32 x 8 411 us a step, 32 x 13
// 436; 101 x 90 x 77: 27.6 and 21.2).
struct VolCut {
  int32_t L;
  double cost;
};
VolCut vol_cut(int bx, int by, bool dbl, int64_t nx, int64_t ny, int64_t nz);

}  // namespace lbm
