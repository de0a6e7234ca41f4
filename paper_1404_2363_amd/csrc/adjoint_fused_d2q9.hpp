// Several adjoint steps per launch for D2Q9 runs periodic on both axes: the
// checkpoint segment's forward recomputation and its reverse sweep through
// LDS, as the multi-step forward kernel does (fused_d2q9.hpp).
//
// The reverse step at a node gathers mu_{t+1} from the push destinations
// y + e_i, so it too depends only on nodes within one node: a block owns a
// tile, the first of its T reverse steps gathers mu from memory over the tile
// widened by T - 1 nodes, the next ones from LDS over rings shrinking by one
// node per step, and the last stores mu_t of the tile itself.  Each node's
// step is adjoint_node with v of that step read from the segment's scratch,
// so mu is bitwise that of one-step launches.  The gradient contributions of
// the tile's own nodes (each computed once per step by the block that owns
// it) accumulate in registers in the one-step sequence's order and precision:
// FP32 runs add them to the segment's FP32 partial and, when the launch ends
// with the segment's first step, fold partial and last contribution into the
// FP64 gradient; FP64 runs add them to the FP64 gradient.  The segment's last
// step (first reverse step), which takes the injected dL/dphi, stays a
// one-step launch.
//
// What bounds it: vector instructions (512^2 FP32, four steps: a third of a
// launch's 13 us alone, two thirds when other launches fill its start and
// end).  A thread therefore keeps the same nodes for all T steps, with their
// coordinates, flux block, velocity and gradient sums in registers, and v of
// the next step is read while the current one computes.  Vector instructions
// per node and step, recomputed rings included: reverse 189, 223 with new
// coordinates and reads at every step and a 64 x 16 tile; recomputation 199 and
// 193 (the smaller tile has more of a ring).  Four steps of 2048^2: reverse
// 180 -> 151 us, recomputation 133 -> 131.
// mu, the sums and the recomputed states are stored plainly, since the next
// launch reads them from the caches; v, read back after the whole segment,
// bypasses them.  Four conditions at 512^2, 400 steps backward: FP32 9.3 ms
// before, 8.7 with the nodes kept, 7.5 with plain stores and the 58 x 16 tile
// (one condition 3.4, 3.0, 2.9), FP64 18.3 -> 13.1 ms.
#pragma once

#include <type_traits>

#include "adjoint_d2q9.hpp"
#include "fused_d2q9.hpp"

namespace lbm {

// Forward recomputation: T steps of the run from a.src, v of every step into
// vout (step s of the launch at vout + s * vstep bytes, planes [2][nx ny]),
// the end state into a.dst when store_end.
template <typename R, int TX, int TY, int NTH, int T, int UK, bool NP>
__global__ __launch_bounds__(NTH) void k_fused_v_d2q9(const RunArgs a, char* vout, int64_t vstep, int store_end) {
  // XCD-contiguous block order: neighbouring tiles, which share halo rows,
  // run on one XCD and its L2
  const uint32_t b = tile_of_block32(blockIdx.x, gridDim.x, a.tiles_x, 1);
  const uint32_t ntx = ((uint32_t)a.nx + TX - 1) / TX, tyi = b / ntx;
  fused_tile<R, TX, TY, NTH, T, UK, false, true, NP>(a, b - tyi * ntx, tyi, vout, vstep, store_end != 0);
}

// Reverse steps k_hi, k_hi - 1, ..., k_hi - T + 1 of a segment: mu_in =
// mu_{k_hi + 1}, v of step k_hi - s at v_hi - s * vstep bytes, mu_out =
// mu_{k_hi - T + 1}; grad (FP64 [3][N]) and part (FP32 [3][N]) as described
// above (fold: the launch ends with the segment's first step, FP32 only).
template <typename R, int TX, int TY, int NTH, int T, int UK, bool NP>
__global__ __launch_bounds__(NTH) void k_fused_adj_d2q9(const RunArgs a, const char* __restrict__ v_hi,
                                                       int64_t vstep, const R* __restrict__ mu_in,
                                                       R* __restrict__ mu_out, double* __restrict__ grad,
                                                       float* __restrict__ part, double inv_kappa, int fold) {
  constexpr bool F64 = sizeof(R) == 8;
  using Acc = typename std::conditional<F64, double, float>::type;
  constexpr int RG = T - 1, W0 = TX + 2 * RG, H0 = TY + 2 * RG, C0 = W0 * H0;
  constexpr int K0 = (C0 + NTH - 1) / NTH;
  constexpr uint32_t E = sizeof(R);
  __shared__ R lds[9 * C0];

  const int tid = threadIdx.x;
  if (tid >= NTH) __builtin_unreachable();
  const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny;
  // XCD-contiguous block order, as the forward recomputation
  const uint32_t b = tile_of_block32(blockIdx.x, gridDim.x, a.tiles_x, 1);
  const uint32_t ntx = ((uint32_t)nx + TX - 1) / TX, tyi = b / ntx, txi = b - tyi * ntx;
  const int32_t x0 = (int32_t)txi * TX - RG, y0 = (int32_t)tyi * TY - RG;
  const uint32_t N = (uint32_t)nx * (uint32_t)ny;
  const size_t pb = (size_t)a.plane * E;
  const Rel2<R> rc = const_rel2<R>(a);
  const char* np = (const char*)a.node_par;

  // Slot k of a thread is node tid + k NTH of the widened tile in every step
  // (slots past the tile repeat its last node and take part in no step): its
  // flux block, velocity and running gradient sums stay in registers.
  int depth[K0];      // distance from the widened tile's edge: step s takes depth >= s
  bool own[K0];       // a node of the tile itself, inside the grid
  uint32_t node[K0];
  R npar[NP ? K0 : 1][3], us[UK ? K0 : 1][2], v[K0][2], f[K0][9];
  Acc acc[K0][3];
  auto load_v = [&](int s, R(&out)[K0][2]) {
    const char* vx = v_hi - s * vstep;
    const char* vy = vx + (size_t)N * E;
    asm volatile("" : "+s"(vx));
    asm volatile("" : "+s"(vy));
#pragma unroll
    for (int k = 0; k < K0; ++k) {
      out[k][0] = gld<R>(vx, node[k] * E);
      out[k][1] = gld<R>(vy, node[k] * E);
    }
  };
  {
    const char* spl[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      spl[i] = (const char*)mu_in + i * pb;
      asm volatile("" : "+s"(spl[i]));
    }
    const uint32_t rlast = (uint32_t)(ny - 1) * (uint32_t)nx;  // offset of the last row
#pragma unroll
    for (int k = 0; k < K0; ++k) {
      const int j = tid + k * NTH, jc = K0 * NTH > C0 ? min(j, C0 - 1) : j;
      const int ly = jc / W0, lx = jc - ly * W0;
      depth[k] = j < C0 ? min(min(lx, W0 - 1 - lx), min(ly, H0 - 1 - ly)) : -1;
      own[k] = depth[k] >= RG && x0 + lx < nx && y0 + ly < ny;
      const int32_t x = wrap_once(x0 + lx, nx), y = wrap_once(y0 + ly, ny);
      const uint32_t xm = x == 0 ? nx - 1 : x - 1, xp = x + 1 == nx ? 0 : x + 1;
      const uint32_t r0 = __umul24((uint32_t)y, (uint32_t)nx), rm = y == 0 ? rlast : r0 - nx,
                     rp = y + 1 == ny ? 0u : r0 + nx;
      node[k] = r0 + x;
      // population (ex, ey) from its push destination (x + ex, y + ey)
      f[k][0] = gld<R>(spl[0], (r0 + x) * E);
      f[k][1] = gld<R>(spl[1], (r0 + xp) * E);
      f[k][2] = gld<R>(spl[2], (rp + x) * E);
      f[k][3] = gld<R>(spl[3], (r0 + xm) * E);
      f[k][4] = gld<R>(spl[4], (rm + x) * E);
      f[k][5] = gld<R>(spl[5], (rp + xp) * E);
      f[k][6] = gld<R>(spl[6], (rp + xm) * E);
      f[k][7] = gld<R>(spl[7], (rm + xm) * E);
      f[k][8] = gld<R>(spl[8], (rm + xp) * E);
      if constexpr (NP)
#pragma unroll
        for (int c = 0; c < 3; ++c) npar[k][c] = gld<R>(np + (size_t)c * N * E, node[k] * E);
      if constexpr (UK != 0) velocity2<R>(a, x, y, us[k][0], us[k][1]);
    }
    load_v(0, v);
#pragma unroll
    for (int k = 0; k < K0; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if constexpr (F64) acc[k][c] = gld<double>((const char*)grad + (size_t)c * N * 8, node[k] * 8u);
        else acc[k][c] = gld<float>((const char*)part + (size_t)c * N * 4, node[k] * 4u);
      }
  }
  // the reverse step of slot k from its gathered populations
  auto step = [&](int k, R(&m)[9], R(&gc)[3]) {
    const R ux = UK ? us[UK ? k : 0][0] : (R)a.u_const[0], uy = UK ? us[UK ? k : 0][1] : (R)a.u_const[1];
    if constexpr (NP) {
      const Rel2<R> rn = a.node_heat_const
                             ? make_rel2<R>(npar[k][0], npar[k][1], npar[k][2], (R)a.heat[0], (R)a.heat[1], a)
                             : node_rel2<R>(a, (int64_t)node[k]);
      adjoint_node<R>(f[k], v[k][0], v[k][1], ux, uy, rn, m, gc);
    } else {
      adjoint_node<R>(f[k], v[k][0], v[k][1], ux, uy, rc, m, gc);
    }
  };
  // population i of a slot from (lx + ex, ly + ey)
  auto gather = [&](int k) {
    const int j = tid + k * NTH;
#pragma unroll
    for (int i = 0; i < 9; ++i) f[k][i] = lds[i * C0 + j + kEy9[i] * W0 + kEx9[i]];
  };

  // steps 0 .. T-2: the first from memory over the widened tile, the next
  // ones from LDS, in place, over rings shrinking by one node; v of the next
  // step is on its way meanwhile
#pragma unroll
  for (int s = 0; s < T - 1; ++s) {
    R vn[K0][2];
    load_v(s + 1, vn);
    if (s > 0) {
#pragma unroll
      for (int k = 0; k < K0; ++k)
        if (depth[k] >= s) gather(k);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < K0; ++k) {
      if (depth[k] >= s) {
        R m[9], gc[3];
        step(k, m, gc);
        if (own[k]) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if constexpr (F64) acc[k][c] = acc[k][c] + inv_kappa * (double)gc[c];
            else acc[k][c] = acc[k][c] + (float)gc[c];
          }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) lds[i * C0 + tid + k * NTH] = m[i];
      }
      v[k][0] = vn[k][0];
      v[k][1] = vn[k][1];
    }
    __syncthreads();
  }

  // step T-1: mu and the gradient of the tile's own nodes to memory
  char* dpl[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    dpl[i] = (char*)mu_out + i * pb;
    asm volatile("" : "+s"(dpl[i]));
  }
#pragma unroll
  for (int k = 0; k < K0; ++k) {
    if (!own[k]) continue;
    R m[9], gc[3];
    gather(k);
    step(k, m, gc);
    const uint32_t n = node[k];
#pragma unroll
    for (int i = 0; i < 9; ++i) gst<R, false>(dpl[i], n * E, m[i]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const Acc s = acc[k][c];
      if constexpr (F64) {
        store_pop<double, false>(grad + c * N + n, s + inv_kappa * (double)gc[c]);
      } else if (fold) {
        store_pop<double, true>(grad + c * N + n, grad[c * N + n] + inv_kappa * ((double)s + (double)gc[c]));
      } else {
        store_pop<float, false>(part + c * N + n, s + (float)gc[c]);
      }
    }
  }
}

}  // namespace lbm
