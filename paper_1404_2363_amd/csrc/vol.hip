// The two-step D3Q15 launches (fused_d3q15.hpp).
#include <algorithm>
#include <cmath>

#include "fused_d3q15.hpp"
#include "vol.hpp"

namespace lbm {

VolCut vol_cut(int bx, int by, bool dbl, int64_t nx, int64_t ny, int64_t nz) {
  // one block per CU (its registers); a plane costs the waves of its first
  // step and of its second, a chunk two planes more than it stores
  const int64_t tiles = ((nx + bx - 1) / bx) * ((ny + by - 1) / by);
  const double waves = (double)(((bx + 2) * (by + 2) + 63) / 64 + (bx * by + 63) / 64);
  VolCut best{(int32_t)nz, 1e300};
  for (int64_t nc = 1; nc <= std::min<int64_t>(nz, 64); ++nc) {
    const int64_t L = (nz + nc - 1) / nc, blocks = tiles * ((nz + L - 1) / L);
    const double r = (double)blocks / 256.0;
    const double c = (r <= 1.0 ? 1.0 : std::max(r, std::ceil(r) - 0.3)) * (double)(L + 2) * waves;
    if (c < best.cost) best = VolCut{(int32_t)L, c};
  }
  return best;
}

template <typename R, int TX, int TY, int NTH>
static void launch(const RunArgs& args, hipStream_t s) {
  RunArgs a = args;
  const int64_t ntx = (a.nx + TX - 1) / TX, nty = (a.ny + TY - 1) / TY;
  const int32_t L = vol_cut(TX, TY, sizeof(R) == 8, a.nx, a.ny, a.nz).L;
  a.tiles_x = make_fastdiv((uint32_t)ntx);
  a.tiles_y = make_fastdiv((uint32_t)nty);
  const dim3 g((unsigned)(ntx * nty * ((a.nz + L - 1) / L))), b(NTH);
  const bool wxy = a.bc[0] != LBM_CDE_PERIODIC || a.bc[1] != LBM_CDE_PERIODIC, wz = a.bc[2] != LBM_CDE_PERIODIC;
#define LBM_VOL(UK, WXY, WZ) hipLaunchKernelGGL((k_fused_d3q15<R, TX, TY, NTH, UK, WXY, WZ>), g, b, 0, s, a, L)
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
