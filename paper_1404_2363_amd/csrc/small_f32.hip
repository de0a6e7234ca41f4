// The multi-step launches over small tiles in FP32 (fused_launch.hpp).
#include "fused_launch.hpp"

namespace lbm {

void launch_small_f32(int k, const RunArgs& a, hipStream_t s) {
  switch (k) {
    case 0: return launch_fused<float, 8, 64, -8, 8>(a, s);
    case 1: return launch_fused<float, 16, 64, -4, 8>(a, s);
    case 2: return launch_fused<float, 32, 32, 1, 8>(a, s);
    default: return launch_fused<float, 16, 32, -2, 4>(a, s);
  }
}

}  // namespace lbm
