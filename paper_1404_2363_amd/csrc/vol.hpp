// Launches of two D3Q15 steps (compiled in vol.hip).
#pragma once

#include "common.hpp"
#include "vol_cut.hpp"

namespace lbm {

using VolFn = void (*)(const RunArgs&, hipStream_t);

// The launch over tiles of at most bx x by columns, cut as a.cut says, or null
// where it is not built.
VolFn vol_launch(int bx, int by, bool dbl);

}  // namespace lbm
