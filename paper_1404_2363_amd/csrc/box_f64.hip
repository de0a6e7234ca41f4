// The multi-step launches of runs with walls on both axes in FP64 (fused_launch.hpp).
#include "fused_launch.hpp"

namespace lbm {

void launch_box_f64(int k, const RunArgs& a, hipStream_t s) {
  switch (k) {
    case 0: return launch_fused<double, 16, 32, -2, 4, true>(a, s);
    default: return launch_fused<double, 32, 16, 1, 4, true>(a, s);
  }
}

}  // namespace lbm
