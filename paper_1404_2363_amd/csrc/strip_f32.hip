// The marching multi-step kernels (strip_d2q9.hpp) in FP32.
#include "strip_d2q9.hpp"

namespace lbm {

void launch_strip_f32(int T, const RunArgs& a, hipStream_t s) {
  switch (T) {
    case 2: return launch_strip_t<float, 2>(a, s);
    case 3: return launch_strip_t<float, 3>(a, s);
    case 4: return launch_strip_t<float, 4>(a, s);
    case 5: return launch_strip_t<float, 5>(a, s);
    default: return launch_strip_t<float, 6>(a, s);
  }
}

void launch_strip_batch_f32(int T, const StripBatch& v, hipStream_t s) {
  switch (T) {
    case 2: return launch_strip_batch_t<float, 2>(v, s);
    case 3: return launch_strip_batch_t<float, 3>(v, s);
    case 4: return launch_strip_batch_t<float, 4>(v, s);
    case 5: return launch_strip_batch_t<float, 5>(v, s);
    default: return launch_strip_batch_t<float, 6>(v, s);
  }
}

}  // namespace lbm
