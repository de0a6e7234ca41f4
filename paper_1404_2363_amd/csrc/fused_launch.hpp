// Launch of several D2Q9 steps over LDS tiles (fused_d2q9.hpp).
#pragma once

#include "fused_d2q9.hpp"

namespace lbm {

// D2Q9 in FP64 or FP32, periodic on both axes or with walls in y, streaming
// stores; tile BX x tile_height(BY, NY) nodes; the velocity kind is a template
// argument.  A shape whose LDS (nine planes of the tile widened by T - 1 nodes
// on every side) would exceed the 160 KiB of a CU is not built for that
// precision.
template <typename R, int BX, int BY, int NY, int T, bool WX = false>
void launch_fused(const RunArgs a, hipStream_t s) {
  constexpr int TY = tile_height(BY, NY);
  const int64_t ntx = (a.nx + BX - 1) / BX, nty = (a.ny + TY - 1) / TY;
  const dim3 g((unsigned)(ntx * nty)), b(BX, BY);
  if constexpr (WX) {  // walls on both axes (velocity constant or separable)
    if (a.u_kind == U_CONST) hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 0, true, false, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 1, true, false, true>), g, b, 0, s, a);
  } else if (a.node_par) {  // a D field (periodic, velocity constant or separable: fused_ok)
    if (a.u_kind == U_CONST) hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 0, false, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 1, false, true>), g, b, 0, s, a);
  } else if (a.bc[1] != LBM_CDE_PERIODIC) {  // walls in y (velocity constant or separable)
    if (a.u_kind == U_CONST) hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 0, true, false>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 1, true, false>), g, b, 0, s, a);
  } else if (a.u_kind == U_CONST) {
    hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 0, false, false>), g, b, 0, s, a);
  } else if (a.u_kind == U_SEPARABLE) {
    hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 1, false, false>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_fused_d2q9<R, BX, BY, NY, T, 2, false, false>), g, b, 0, s, a);
  }
}

// The launches over small tiles (small_f32.hip, small_f64.hip): grids whose
// tiles of the usual sizes would leave most of the 256 CUs without a block.
struct SmallTile {
  int bx, by, ny, T;
};
constexpr SmallTile kSmall[] = {{8, 64, -8, 8}, {16, 64, -4, 8}, {32, 32, 1, 8}, {16, 32, -2, 4}};
constexpr int kSmallCount = 4;
void launch_small_f32(int k, const RunArgs& a, hipStream_t s);
void launch_small_f64(int k, const RunArgs& a, hipStream_t s);

// The launches of runs with walls on both axes (box_f32.hip, box_f64.hip).
constexpr SmallTile kBox[] = {{16, 32, -2, 4}, {32, 16, 1, 4}};
constexpr int kBoxCount = 2;
void launch_box_f32(int k, const RunArgs& a, hipStream_t s);
void launch_box_f64(int k, const RunArgs& a, hipStream_t s);

}  // namespace lbm
