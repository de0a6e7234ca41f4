// Two D3Q15 steps per launch: blocks that march along z.
//
// A block owns a tile of columns of nodes and walks the planes of its chunk.
// At plane p it pulls the stored state of the columns widened by one node on
// every side (one node per thread), does the first step and publishes the
// result in LDS; the threads of the block's own columns gather from there what
// the second step needs: the populations with e_z = -1 of plane p, used at
// once, those with e_z = 0, kept one plane, and those with e_z = +1, kept two
// planes in registers (Eq. 5: a population moves one node per step).  So the
// second step of plane p - 1 follows the first of plane p, and the state
// crosses HBM once per two steps.
//
// Every node's step has the pull, velocity and collision arithmetic of
// k_step_d3q15, so a launch here equals two one-step launches bitwise.  For
// constant or separable velocities; x and y periodic or mirrored (SPECULAR),
// z any kind: a bounced population of an x or y wall would come from the
// node's own plane instead of the neighbour plane that the registers hold.
//
// One step per launch moves 120 B per node (FP32) at 72 % of HBM's 8 TB/s, its
// access pattern's ceiling (365 us at 256^3, FP64 737 us); here a step moves
// half of that and the bound is the pace of one block per CU: barrier, second
// step, first step of the next plane.  Measured at 256^3: 196 us a step with
// 64 x 8 columns (FP64 396-411 with 32 x 8).  Narrower tiles re-read more halo
// lines (32 x 16: 208 us), smaller blocks two to a CU were slower (32 x 8, 384
// threads: 226 us), and so was a pull one plane ahead instead of two where
// registers allow both (64 x 8: 203 us, FP64 32 x 8: 439 us).  Plain stores: a
// tile's rows need not start on a cache line (100 x 90 x 77: 14.4 us a step
// against 16.9 with streaming stores; at 256^3 the two are equal).
#pragma once

#include "d3q15.hpp"

namespace lbm {

__device__ constexpr int kEx15[15] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1};
__device__ constexpr int kEy15[15] = {0, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 1, 1, -1, -1};
__device__ constexpr int kEz15[15] = {0, 0, 0, 0, 0, 1, -1, 1, 1, 1, 1, -1, -1, -1, -1};
// population with the x, y or z component reversed, and the opposite one
__device__ constexpr int kMx15[15] = {0, 2, 1, 3, 4, 5, 6, 8, 7, 10, 9, 12, 11, 14, 13};
__device__ constexpr int kMy15[15] = {0, 1, 2, 4, 3, 5, 6, 9, 10, 7, 8, 13, 14, 11, 12};
__device__ constexpr int kMz15[15] = {0, 1, 2, 3, 4, 6, 5, 11, 12, 13, 14, 7, 8, 9, 10};
__device__ constexpr int kOp15[15] = {0, 2, 1, 4, 3, 6, 5, 14, 13, 12, 11, 10, 9, 8, 7};
// the populations of a plane's register rings: e_z = +1, 0, -1
__device__ constexpr int kUp15[5] = {5, 7, 8, 9, 10};
__device__ constexpr int kMid15[5] = {0, 1, 2, 3, 4};
__device__ constexpr int kDown15[5] = {6, 11, 12, 13, 14};

// Barrier that orders LDS accesses only: loads and stores of the state stay
// in flight across it (a full one would wait for the next plane's pull).
LBM_FORCEINLINE void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// j / w for 0 <= j < 1024 and 1 <= w <= 66: the quotient is at least 1 / 132 off
// an integer, the reciprocal's error at most 1e-4 of it.
LBM_FORCEINLINE int row_of(int j, int w) { return (int)(((float)j + 0.5f) * __builtin_amdgcn_rcpf((float)w)); }

// A chunk of cut[2] planes of a tile of cut[0] x cut[1] columns: TX x TY, or
// fewer on grids that are narrower or have too few tiles (vol_cut); a block has
// a thread for every widened column, at most NTH.  WXY: a wall in x or y (every
// byte offset in the Q planes then fits 32 bits, else those in a plane z =
// const); WZ: walls in z.
template <typename R, int TX, int TY, int NTH, int UK, bool WXY, bool WZ>
__global__ __launch_bounds__(NTH) void k_fused_d3q15(const RunArgs a) {
  constexpr int W0 = TX + 2, C0 = W0 * (TY + 2);  // the LDS keeps the full tile's pitch
  const int32_t tx = a.cut[0], ty = a.cut[1], L = a.cut[2];
  // planes a pull is ahead of its use; with walls in the plane and across it
  // the registers of a second one would spill
  constexpr int PF = WXY && WZ ? 1 : 2;
  static_assert(NTH >= C0, "one node per thread");
  constexpr uint32_t E = sizeof(R);
  __shared__ R lds[15 * C0];
  const int tid = threadIdx.x;
  const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny, nz = (int32_t)a.nz;
  const uint32_t b = tile_of_block32(blockIdx.x, gridDim.x, a.tiles_x, 1);
  const uint32_t rest = fdiv(b, a.tiles_x), cz = fdiv(rest, a.tiles_y);
  const int32_t x0 = (int32_t)(b - rest * a.tiles_x.d) * tx, y0 = (int32_t)(rest - cz * a.tiles_y.d) * ty;
  const int32_t w0 = tx + 2, nown = tx * ty, nwide = w0 * (ty + 2);
  const int32_t z0 = __builtin_amdgcn_readfirstlane((int32_t)cz * L);
  const int32_t z1 = __builtin_amdgcn_readfirstlane(min(z0 + L, nz));
  const size_t pb = (size_t)a.plane * E, sz = (size_t)nx * (size_t)ny * E;
  const Rel3<R> rc = const_rel3<R>(a);
  const R phi_ref = (R)a.phi_ref;
  const bool px = a.bc[0] == LBM_CDE_PERIODIC, py = a.bc[1] == LBM_CDE_PERIODIC;
  const bool bz = WZ && a.bc[2] == LBM_CDE_BOUNCE_BACK;

  // the thread's node of the widened columns (first step).  Columns beyond a
  // wall or past the far edge of the last tile (+ its halo) are not needed;
  // they are clamped to valid addresses.
  const int jl = min(tid, nwide - 1), ly1 = row_of(jl, w0), lx1 = jl - ly1 * w0, j1 = ly1 * W0 + lx1;
  auto wrap = [](int32_t v, int32_t n, bool per) {
    return per ? (v < 0 ? v + n : (v >= n ? v - n : v)) : (v < 0 ? 0 : (v >= n ? n - 1 : v));
  };
  const int32_t xa = wrap(min(x0 + lx1 - 1, nx), nx, px), ya = wrap(min(y0 + ly1 - 1, ny), ny, py);
  // and of the block's own columns (second step)
  const int jo = min(tid, nown - 1), ly2 = row_of(jo, tx), lx2 = jo - ly2 * tx;
  const int32_t xb = min(x0 + lx2, nx - 1), yb = min(y0 + ly2, ny - 1);
  const bool wide = tid < nwide, mine = tid < nown, own = mine && x0 + lx2 < nx && y0 + ly2 < ny;

  // static byte offset of population i's pull within a plane of nodes, the
  // population plane included.  A mirror wall in x or y reverses that
  // component and keeps the coordinate (pull_index_d3q15).
  uint32_t off[15];
#pragma unroll
  for (int i = 0; i < 15; ++i) {
    int32_t sx = xa - kEx15[i], sy = ya - kEy15[i];
    const bool ox = sx < 0 || sx >= nx, oy = sy < 0 || sy >= ny;
    int pop = i;
    sx = wrap(sx, nx, px);
    sy = wrap(sy, ny, py);
    if constexpr (WXY) {
      const bool cx = ox && !px, cy = oy && !py;
      pop = cx && cy ? kMy15[kMx15[i]] : cx ? kMx15[i] : cy ? kMy15[i] : i;
    }
    off[i] = (WXY ? (uint32_t)pop * (uint32_t)pb : 0u) + ((uint32_t)sy * (uint32_t)nx + (uint32_t)sx) * E;
  }
  // where the second step finds population i of its node in LDS
  int at[15];
  const int j2 = (ly2 + 1) * W0 + lx2 + 1;
#pragma unroll
  for (int i = 0; i < 15; ++i) {
    int pop = i, dx = -kEx15[i], dy = -kEy15[i];
    if constexpr (WXY) {
      const bool cx = !px && (xb + dx < 0 || xb + dx >= nx), cy = !py && (yb + dy < 0 || yb + dy >= ny);
      pop = cx && cy ? kMy15[kMx15[i]] : cx ? kMx15[i] : cy ? kMy15[i] : i;
      dx = cx ? 0 : dx;
      dy = cy ? 0 : dy;
    }
    at[i] = pop * C0 + j2 + dy * W0 + dx;
  }
  // separable velocity: ((t_c[0] t_c[1+x]) t_c[1+nx+y]) t_c[1+nx+ny+z], the
  // first two products kept per thread, the plane's factor a scalar
  R va[3], vb[3];
  using CR = const __attribute__((address_space(4))) R;
  CR* vz[3];
  const int32_t ts = 1 + nx + ny + nz;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if constexpr (UK == 0) {
      va[c] = vb[c] = (R)a.u_const[c];
    } else {
      const R* t = (const R*)a.u_tab + c * ts;
      va[c] = (t[0] * t[1 + xa]) * t[1 + nx + ya];
      vb[c] = (t[0] * t[1 + xb]) * t[1 + nx + yb];
      vz[c] = (CR*)(uintptr_t)(t + 1 + nx + ny);
    }
  }
  auto collide = [&](R(&f)[15], const R(&v)[3], const R(&w)[3]) {
    if constexpr (UK == 0) collide_d3q15<R>(f, v[0], v[1], v[2], phi_ref, rc);
    else collide_d3q15<R>(f, v[0] * w[0], v[1] * w[1], v[2] * w[2], phi_ref, rc);
  };
  const char* src = (const char*)a.src;
  char* dst = (char*)a.dst;

  // the pull of plane z
  auto load = [&](R(&f)[15], int32_t z) {
    const int32_t zm = z == 0 ? (WZ ? 0 : nz - 1) : z - 1, zp = z + 1 == nz ? (WZ ? z : 0) : z + 1;
    if (WZ && (z == 0 || z == nz - 1)) {
      // z wall: the reversed population of the same node (bounce), or the
      // mirrored one pulled from the node's own plane
#pragma unroll
      for (int i = 0; i < 15; ++i) {
        const bool out = (z == 0 && kEz15[i] > 0) || (z == nz - 1 && kEz15[i] < 0);
        const int32_t zs = kEz15[i] > 0 ? (out ? z : zm) : kEz15[i] < 0 ? (out ? z : zp) : z;
        uint32_t o = off[i];
        int pop = 0;
        if constexpr (WXY) {
          // the offset holds its own (x, y rule) population plane
          if (out && bz) o = (uint32_t)kOp15[i] * (uint32_t)pb + ((uint32_t)ya * (uint32_t)nx + (uint32_t)xa) * E;
          else if (out) o = off[kMz15[i]];
        } else {
          pop = out ? (bz ? kOp15[i] : kMz15[i]) : i;
          if (out && bz) o = ((uint32_t)ya * (uint32_t)nx + (uint32_t)xa) * E;
        }
        f[i] = gld<R>(src + (size_t)zs * sz + (size_t)pop * pb, o);
      }
      return;
    }
    const size_t bz0 = (size_t)z * sz, bzm = (size_t)zm * sz, bzp = (size_t)zp * sz;
#pragma unroll
    for (int i = 0; i < 15; ++i) {
      const char* p = src + (kEz15[i] > 0 ? bzm : kEz15[i] < 0 ? bzp : bz0) + (WXY ? (size_t)0 : (size_t)i * pb);
      asm volatile("" : "+s"(p));
      f[i] = gld<R>(p, off[i]);
    }
  };

  int32_t p = WZ ? max(z0 - 1, 0) : z0 - 1;  // plane of the first step (not wrapped)
  const int32_t plast = WZ ? min(z1, nz - 1) : z1;
  // grid plane of plane q (one wrap; q >= 0 with walls)
  auto image = [&](int32_t q) {
    return __builtin_amdgcn_readfirstlane(WZ ? min(q, nz - 1) : (q < 0 ? q + nz : (q >= nz ? q - nz : q)));
  };
  // the pulls of this plane and the next, in flight PF planes ahead of use
  // (past the last plane it is pulled again and not used)
  R fa[15], fb[15];
  load(fa, image(p));
  if constexpr (PF == 2) load(fb, image(min(p + 1, plast)));
  R up1[5], up2[5], mid[5], top[5];  // level-1 values of earlier planes
#pragma unroll
  for (int k = 0; k < 5; ++k) up1[k] = up2[k] = mid[k] = top[k] = (R)0;
  const uint32_t so = ((uint32_t)yb * (uint32_t)nx + (uint32_t)xb) * E;
  // second step of plane q from the rings and the populations moving down
  auto second = [&](int32_t q, const R(&dn)[5], R(&f)[15]) {
    R g[15], w[3];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      g[kMid15[k]] = mid[k];
      g[kUp15[k]] = up2[k];
      g[kDown15[k]] = dn[k];
    }
    if constexpr (UK == 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) w[c] = vz[c][q];
    }
    collide(g, vb, w);
    // the next plane's pull has arrived before this plane's stores are issued
    // (after them, the in-order counter would make it wait for them as well)
#pragma unroll
    for (int i = 0; i < 15; ++i) asm volatile("" : "+v"(f[i]));
    char* d[15];
#pragma unroll
    for (int i = 0; i < 15; ++i) {
      d[i] = dst + (size_t)q * sz + (size_t)i * pb;
      asm volatile("" : "+s"(d[i]));
    }
    if (own) {
#pragma unroll
      for (int i = 0; i < 15; ++i) gst<R, false>(d[i], so, g[i]);
    }
  };
  auto plane = [&](R(&f)[15], R(&nf)[15]) {
    const int32_t z = image(p);
    if (wide) {
      R w[3];
      if constexpr (UK == 1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) w[c] = vz[c][z];
      }
      collide(f, va, w);
#pragma unroll
      for (int i = 0; i < 15; ++i) lds[i * C0 + j1] = f[i];
    }
    load(f, image(min(p + PF, plast)));
    lds_barrier();
    R dn[5], nu[5], nm[5];
    if (mine) {
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        dn[k] = lds[at[kDown15[k]]];
        nm[k] = lds[at[kMid15[k]]];
        nu[k] = lds[at[kUp15[k]]];
      }
      if (WZ && p == 0) {  // what plane 0 pulls from below its wall
#pragma unroll
        for (int k = 0; k < 5; ++k)
          up1[k] = bz ? lds[kOp15[kUp15[k]] * C0 + j2] : lds[at[kMz15[kUp15[k]]]];
      }
      if (WZ && p == nz - 1) {  // what the last plane pulls from above its wall
#pragma unroll
        for (int k = 0; k < 5; ++k)
          top[k] = bz ? lds[kOp15[kDown15[k]] * C0 + j2] : lds[at[kMz15[kDown15[k]]]];
      }
    }
    lds_barrier();
    if (mine) {
      if (p > z0) second(p - 1, dn, nf);
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        up2[k] = up1[k];
        up1[k] = nu[k];
        mid[k] = nm[k];
      }
    }
    ++p;
  };
  if constexpr (PF == 1) {
    while (p <= plast) plane(fa, fa);
  } else {
    while (p + 1 <= plast) {
      plane(fa, fb);
      plane(fb, fa);
    }
    if (p <= plast) plane(fa, fb);
  }
  if (WZ && z1 == nz && mine) second(nz - 1, top, fa);  // no plane above the last one
}

}  // namespace lbm
