// The multi-step launches over small tiles in FP64 (fused_launch.hpp).
#include "fused_launch.hpp"

namespace lbm {

// Eight steps of 32 x 32 tiles, or of half their height where those are at most
// one per CU: a launch then lasts as long as one block, and the 46 x 30 nodes of
// the half tile take its 1024 threads 1.35 passes instead of 2.07 (300^2, us a
// step: 64 x 8 tiles of four steps 2.24, 32 x 32 2.64, 32 x 16 1.85; with a D
// field 2.57, 3.36 and 2.16).
static void launch_32(const RunArgs& a, hipStream_t s) {
  if ((a.nx + 31) / 32 * ((a.ny + 15) / 16) <= 256) launch_fused<double, 32, 32, -2, 8>(a, s);
  else launch_fused<double, 32, 32, 1, 8>(a, s);
}

void launch_small_f64(int k, const RunArgs& a, hipStream_t s) {
  switch (k) {
    case 0: return launch_fused<double, 8, 64, -8, 8>(a, s);
    case 1: return launch_fused<double, 16, 64, -4, 8>(a, s);
    case 2: return launch_32(a, s);
    default: return launch_fused<double, 16, 32, -2, 4>(a, s);
  }
}

}  // namespace lbm
