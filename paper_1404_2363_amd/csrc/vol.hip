// The two-step D3Q15 launches (fused_d3q15.hpp).
#include "fused_d3q15.hpp"
#include "vol.hpp"

namespace lbm {

template <typename R, int TX, int TY, int NTH>
static void launch(const RunArgs& args, hipStream_t s) {
  RunArgs a = args;
  const int32_t tx = a.cut[0], ty = a.cut[1], L = a.cut[2];
  const int64_t ntx = (a.nx + tx - 1) / tx, nty = (a.ny + ty - 1) / ty;
  a.tiles_x = make_fastdiv((uint32_t)ntx);
  a.tiles_y = make_fastdiv((uint32_t)nty);
  const dim3 g((unsigned)(ntx * nty * ((a.nz + L - 1) / L))), b(((tx + 2) * (ty + 2) + 63) / 64 * 64);
  const bool wxy = a.bc[0] != LBM_CDE_PERIODIC || a.bc[1] != LBM_CDE_PERIODIC, wz = a.bc[2] != LBM_CDE_PERIODIC;
#define LBM_VOL(UK, WXY, WZ) hipLaunchKernelGGL((k_fused_d3q15<R, TX, TY, NTH, UK, WXY, WZ>), g, b, 0, s, a)
  if (a.u_kind == U_CONST) {
    if (wxy && wz) LBM_VOL(0, true, true);
    else if (wxy) LBM_VOL(0, true, false);
    else if (wz) LBM_VOL(0, false, true);
    else LBM_VOL(0, false, false);
  } else {
    if (wxy && wz) LBM_VOL(1, true, true);
    else if (wxy) LBM_VOL(1, true, false);
    else if (wz) LBM_VOL(1, false, true);
    else LBM_VOL(1, false, false);
  }
#undef LBM_VOL
}

VolFn vol_launch(int bx, int by, bool dbl) {
  if (bx == 64 && by == 8 && !dbl) return launch<float, 64, 8, 704>;
  if (bx == 32 && by == 16 && !dbl) return launch<float, 32, 16, 640>;
  if (bx == 32 && by == 8 && dbl) return launch<double, 32, 8, 384>;
  if (bx == 32 && by == 13 && dbl) return launch<double, 32, 13, 512>;
  return nullptr;
}

}  // namespace lbm
