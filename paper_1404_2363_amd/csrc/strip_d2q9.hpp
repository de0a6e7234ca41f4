// Several D2Q9 steps per launch by waves that march along y, with the state
// between the steps in registers.
//
// A wave has 64 columns, one per lane, and keeps the middle 64 - 2 (T - 1);
// the others are recomputed by its neighbours.
// It walks the rows of its chunk: at row p the first step of row p is pulled
// from memory, the second step of row p - 1 follows, and so on to the T-th
// step of row p - (T - 1), which is stored.  Step l + 1 of row q needs step l
// of rows q - 1, q and q + 1 (Eq. 5: a population moves one node per step):
// the populations moving up wait two rows in registers, those staying in
// their row one, and those moving down arrive with the row just computed;
// x neighbours are the neighbouring lanes (DPP wave shifts).  No LDS, no
// barrier: the waves of a launch run independently.
//
// Every node's step has the pull, velocity and collision arithmetic of the
// one-step kernel, so T steps here equal T one-step launches bitwise.  For
// runs periodic in x with an equilibrium linear in phi and phi u, a constant
// D and a constant or separable (unit z factors) velocity; y periodic or,
// with WY, bounded by walls.
//
// What bounds it, MI355X, 4096^2: the LDS tile kernel (fused_d2q9.hpp) issues
// 134 VALU instructions per node and step (addressing and the recomputed
// rings of a 64 x 24 tile on top of the collision's 93) and waits at two
// barriers per step; the march issues 99 for a node that it computes, 121 per
// node and step with the 64 / 54 columns and T - 1 rows per chunk that it
// recomputes.  A launch moves the state once whatever T is, which takes 280-290
// us in FP32 for T = 3 and 4 (4.2 TB/s: 9 + 9 row streams per wave), 310 for
// T = 5 and 348 for T = 6, where the VALU is the bound (1.9e8 wave instructions,
// 89 % of its issue rate; 1.32 GB, 1.09 times the state): T = 6 gives 58 us a step
// against 69-75 for the tile kernel on the same GPU (FP64: 98 against 152; at
// 2048^2 16.7 against 20.1, FP64 27 against 40).  T = 8 keeps 50 columns of 64
// and was 4-10 % slower.
// 64 channels of 32-128 rows in a batch x 400 sampled steps: 39.4 to 28.8 ms;
// 12 plate channels in FP64 x 200: 5.4 to 3.5 ms.
// Plain stores: the rows end inside a cache line that the neighbouring wave
// completes, and streaming stores (65 us a step) write it twice.
#pragma once

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "d2q9.hpp"
#include "fused_d2q9.hpp"

namespace lbm {

constexpr int kStripMax = 6;  // steps per launch built: 2 .. kStripMax

// Columns that a wave keeps.
constexpr int strip_width(int T) { return 64 - 2 * (T - 1); }

// The value of the lane to the left (lane l takes lane l - 1's) or right;
// the lane at the end of the wave takes 0 (its column is not kept).
template <int CTRL>
LBM_FORCEINLINE float wave_shift(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
LBM_FORCEINLINE double wave_shift(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <typename R>
LBM_FORCEINLINE R from_left(R v) { return wave_shift<0x138>(v); }   // wave_shr:1
template <typename R>
LBM_FORCEINLINE R from_right(R v) { return wave_shift<0x130>(v); }  // wave_shl:1

// What step l + 1 still needs of the rows step l has done, already shifted in
// x: populations 2, 5, 6 (moving up) of the last row but one (a) and the last
// row (b), populations 0, 1, 3 of the last row (c).
template <typename R>
struct StripRing {
  R a[3], b[3], c[3];
};

// T steps of rows [cy L, cy L + L) of strip sx of the run described by a, by
// one wave (all arguments uniform).  UK: velocity, 0 constant, 1 separable.
template <typename R, int T, int UK, bool WY>
LBM_FORCEINLINE void strip_march(const RunArgs& a, int32_t sx, int32_t cy, int32_t L) {
  static_assert(T >= 2, "one step per launch is k_step_d2q9");
  constexpr int RG = T - 1, VW = strip_width(T);
  constexpr uint32_t E = sizeof(R);
  const int lane = threadIdx.x;
  const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny;
  // the lane's column (periodic image) and its neighbours, as byte offsets
  const int32_t xs = sx * VW - RG + lane, x = wrap_once(xs, nx);
  const uint32_t xo = (uint32_t)x * E, xmo = (uint32_t)(x == 0 ? nx - 1 : x - 1) * E,
                 xpo = (uint32_t)(x + 1 == nx ? 0 : x + 1) * E;
  const bool own = lane >= RG && lane < RG + VW && xs < nx;
  const int32_t y0 = __builtin_amdgcn_readfirstlane(cy * L), y1 = __builtin_amdgcn_readfirstlane(min(y0 + L, ny));
  const size_t pb = (size_t)a.plane * E, pitch = (size_t)nx * E;
  const Rel2<R> rc = const_rel2<R>(a);
  const R phi_ref = (R)a.phi_ref;
  // separable velocity: component c at (x, y) is (t_c[0] t_c[1+x]) t_c[1+nx+y];
  // the first product stays in the lane, the row factors come as scalars
  using CR = const __attribute__((address_space(4))) R;
  const R* tab = (const R*)a.u_tab;
  const int32_t ts = 1 + nx + ny + 1;
  CR* rows0 = (CR*)(uintptr_t)(tab + 1 + nx);
  CR* rows1 = (CR*)(uintptr_t)(tab + ts + 1 + nx);
  R uc0, uc1;
  if constexpr (UK == 0) {
    uc0 = (R)a.u_const[0];
    uc1 = (R)a.u_const[1];
  } else {
    uc0 = tab[0] * tab[1 + x];
    uc1 = tab[ts] * tab[ts + 1 + x];
  }
  const char* src = (const char*)a.src;
  char* dst = (char*)a.dst;
  const int bcy = WY ? a.bc[1] : 0;
  const bool bounce = WY && bcy == LBM_CDE_BOUNCE_BACK, node = WY && bcy == LBM_CDE_NODE_MIRROR;

  // the pull of row r from memory.  Row bases are scalars (pinned by the
  // empty asm), so a load is base + the lane's 32-bit column offset.
  auto load = [&](R(&f)[9], int32_t r) {
    const int32_t rm = r == 0 ? (WY ? 0 : ny - 1) : r - 1, rp = r + 1 == ny ? (WY ? r : 0) : r + 1;
    int pop[9] = {0, 1, 2, 3, 4, 5, 6, 7, 8};
    int32_t ru = rm, rd = rp;  // source rows of the populations moving up and down
    uint32_t ol = xmo, orr = xpo, dl = xmo, dr = xpo;
    if constexpr (WY) {  // the wall rule of row_source_d2q9, without branches
      if (r == 0) {
        pop[2] = 4;
        pop[5] = bounce ? 7 : 8;
        pop[6] = bounce ? 8 : 7;
        ru = node ? 1 : 0;
        ol = bounce ? xo : xmo;
        orr = bounce ? xo : xpo;
      }
      if (r == ny - 1) {
        pop[4] = 2;
        pop[7] = bounce ? 5 : 6;
        pop[8] = bounce ? 6 : 5;
        rd = node ? ny - 2 : ny - 1;
        dl = bounce ? xo : xmo;
        dr = bounce ? xo : xpo;
      }
    }
    const size_t o0 = (size_t)r * pitch, ou = (size_t)ru * pitch, od = (size_t)rd * pitch;
    const size_t ro[9] = {o0, o0, ou, o0, od, ou, ou, od, od};
    const uint32_t co[9] = {xo, xmo, xo, xpo, xo, ol, orr, dr, dl};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const char* p = src + pop[i] * pb + ro[i];
      asm volatile("" : "+s"(p));
      f[i] = gld<R>(p, co[i]);
    }
  };

  R us[2][T];  // row factors of the velocity at row p - l
  StripRing<R> ring[T - 1];
#pragma unroll
  for (int l = 0; l < T; ++l) us[0][l] = us[1][l] = (R)0;
#pragma unroll
  for (int l = 0; l < T - 1; ++l)
#pragma unroll
    for (int k = 0; k < 3; ++k) ring[l].a[k] = ring[l].b[k] = ring[l].c[k] = (R)0;

  auto coll = [&](R(&f)[9], int l) {
    R ux, uy;
    if constexpr (UK == 0) {
      ux = uc0;
      uy = uc1;
    } else {
      ux = uc0 * us[0][l];
      uy = uc1 * us[1][l];
    }
    collide_d2q9<R, 1>(f, ux, uy, phi_ref, rc);
  };

  int32_t p = WY ? max(y0 - RG, 0) : y0 - RG;  // row of the first step (not wrapped)
  int32_t r = __builtin_amdgcn_readfirstlane(WY ? p : wrap_once(p, ny));  // its periodic image
  const int32_t plast = y1 - 1 + RG;
  R fn[9];  // the next row's pull, one row ahead
  load(fn, r);

  // One row of the march.  GUARD: near the chunk's ends and the walls, where
  // some steps have no row to do (step l does rows y0 - RG + l .. y1 - 1 +
  // RG - l, inside the walls) and the wall rules apply.
  auto row = [&](auto guard) {
    constexpr bool GUARD = decltype(guard)::value;
    auto active = [&](int l) {
      const int32_t q = p - l;
      return q >= y0 - RG + l && q <= y1 - 1 + RG - l && (!WY || (q >= 0 && q < ny));
    };
    R f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = fn[i];
    if constexpr (UK == 1) {
#pragma unroll
      for (int l = T - 1; l > 0; --l) {
        us[0][l] = us[0][l - 1];
        us[1][l] = us[1][l - 1];
      }
      us[0][0] = rows0[r];
      us[1][0] = rows1[r];
    }
    r = r + 1 == ny ? (WY ? r : 0) : r + 1;  // past the upper wall: the last row again, not used
    load(fn, r);
    __builtin_amdgcn_sched_barrier(0);
    if (!GUARD || active(0)) coll(f, 0);
#pragma unroll
    for (int l = 1; l < T; ++l) {
      StripRing<R>& k = ring[l - 1];
      const int32_t q = p - l;
      // f: step l - 1 of row q + 1
      R g[9] = {k.c[0], k.c[1], k.a[0], k.c[2], f[4], k.a[1], k.a[2], from_right(f[7]), from_left(f[8])};
      if constexpr (GUARD && WY) {
        if (node && q == 0) {  // on-node wall: the mirrored populations come from row 1
          g[2] = g[4];
          g[5] = g[8];
          g[6] = g[7];
        }
        if (q == ny - 1) {  // upper wall: row q itself (b), or row q - 1 (a) at an on-node wall
          g[4] = node ? k.a[0] : k.b[0];
          g[7] = node ? k.a[2] : (bounce ? from_right(k.b[1]) : k.b[2]);
          g[8] = node ? k.a[1] : (bounce ? from_left(k.b[2]) : k.b[1]);
        }
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) k.a[j] = k.b[j];
      k.b[0] = f[2];
      k.b[1] = from_left(f[5]);
      k.b[2] = from_right(f[6]);
      k.c[0] = f[0];
      k.c[1] = from_left(f[1]);
      k.c[2] = from_right(f[3]);
      if constexpr (GUARD && WY) {
        if (q + 1 == 0) {  // lower wall: what row 0 pulls from below comes from row 0
          k.a[0] = f[4];
          k.a[1] = bounce ? f[7] : g[8];
          k.a[2] = bounce ? f[8] : g[7];
        }
      }
      if (!GUARD || active(l)) coll(g, l);
#pragma unroll
      for (int i = 0; i < 9; ++i) f[i] = g[i];
    }
    // wait for the next row here, before this row's stores: after them, the
    // in-order counter would make the next row wait for the stores as well
#pragma unroll
    for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(fn[i]));
    char* d[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      d[i] = dst + (size_t)(p - RG) * pitch + i * pb;
      asm volatile("" : "+s"(d[i]));
    }
    if (own && (!GUARD || active(RG))) {
#pragma unroll
      for (int i = 0; i < 9; ++i) gst<R, false>(d[i], xo, f[i]);
    }
    ++p;
  };

  // rows in which every step has a full row to do, two at a time (the rings
  // then rotate without moves); one at a time before and after them
  const int32_t s0 = y0 + RG + (WY ? 1 : 0), s1 = WY ? min(plast, ny - 1) : plast;
  while (p < s0 && p <= plast) row(std::true_type{});
  while (p + 1 <= s1) {
    row(std::false_type{});
    row(std::false_type{});
  }
  while (p <= plast) row(std::true_type{});
}

// One run: block = one wave; strips of a chunk next to each other, XCD-contiguous
// (neighbouring strips share cache lines at their edges).
template <typename R, int T, int UK, bool WY>
__global__ __launch_bounds__(64) void k_strip_d2q9(const RunArgs a, int32_t L) {
  const uint32_t b = tile_of_block32(blockIdx.x, gridDim.x, a.tiles_x, 1);
  const uint32_t cy = fdiv(b, a.tiles_x);
  strip_march<R, T, UK, WY>(a, (int32_t)(b - cy * a.tiles_x.d), (int32_t)cy, L);
}

// T steps of every active run of a batch: block b takes wave unit t of a flat
// list of (run, chunk, strip), eight neighbouring strips to an XCD.  clock[0] +
// toff is the step before the launch, clock[2] ^ flip the buffer it reads.
template <typename R, int T, int UK, bool WY>
__global__ __launch_bounds__(64) void k_batch_strip_d2q9(const BatchRun* __restrict__ runs,
                                                        const uint32_t* __restrict__ tile_start, int nruns,
                                                        const int64_t* __restrict__ clock, int64_t toff, int flip,
                                                        int32_t L) {
  const uint32_t b = blockIdx.x, xcd = b & 7u, local = b >> 3;
  const uint32_t t = (local >> 3) * 64u + xcd * 8u + (local & 7u);
  const int na = batch_active_runs(runs, nruns, clock[0] + toff);
  if (na == 0 || t >= tile_start[na]) return;
  const int lo = __builtin_amdgcn_readfirstlane(batch_run_of(tile_start, na, t));
  RunArgs a = batch_run_args<R>(runs[lo], (int)(clock[2] & 1) ^ flip);
  constexpr int VW = strip_width(T);
  const uint32_t nsx = __builtin_amdgcn_readfirstlane((runs[lo].nx + VW - 1) / VW);
  const uint32_t u = t - __builtin_amdgcn_readfirstlane(tile_start[lo]);
  const uint32_t cy = __builtin_amdgcn_readfirstlane(u / nsx);
  strip_march<R, T, UK, WY>(a, (int32_t)(u - cy * nsx), (int32_t)cy, L);
}

// ---- launches (compiled per precision: strip_f32.hip, strip_f64.hip) ---------

// How a grid (or a batch) is cut: chunks of L rows, T steps per launch.
//
// Units (a strip's chunk, one wave each) go to the 1024 SIMDs; the last to
// finish sets the time.  A unit of h rows takes h + T - 1 rows' work; a row
// takes about (T + 2.5) times what one step of a row does (the 2.5: loads,
// stores, bookkeeping), two waves on a SIMD `two` times as long as one (they
// fill each other's gaps), and a launch has a fixed part.  Measured, one wave
// per SIMD, T = 6: 1.34 us a row in FP32 and 1.68 in FP64 (1024^2); two: 1.55
// and 1.84 times that (1024^2, 2048^2, 4096^2); a launch 3 us.
struct StripCut {
  int T;
  int32_t L;
  double cost;  // time per step, in units of one step of a row on one SIMD
};

// The cost of a launch with chunks of L rows; rows(f) calls f(height, strips) for
// every run, a chunk's ends cost `ends` times their T - 1 rows.
template <typename Rows>
double strip_cost(int T, int64_t L, bool dbl, double ends, Rows rows) {
  const double two = dbl ? 1.84 : 1.55, fixed = dbl ? 15.0 : 19.0, h = ends * (double)(T - 1);
  double all = 0.0, chunks = 0.0;
  int64_t least = L;
  rows([&](int64_t ny, int64_t strips) {
    const int64_t n = (ny + L - 1) / L;
    all += (double)strips * (double)ny;
    chunks += (double)(strips * n);
    least = std::min(least, (ny + n - 1) / n);
  });
  const double x = chunks / 1024.0, k = std::ceil(x);
  const double last = (all + chunks * h) / 1024.0 + (k - x) * ((double)least + h);
  return (last * (k >= 2.0 ? 0.5 * two : 1.0) * (T + 2.5) + fixed) / T;
}

// Between walls the rows at a chunk's ends, which test every step, take about
// three times as long in FP32 (1024^2, T = 4, 5, 6: 5.5, 5.6 and 5.8 us a step
// periodic, 7.2, 7.6 and 8.1 between walls).  The cost says so, and fewer steps
// per launch win on smaller grids; the chunks stay those of the periodic march,
// since longer ones leave SIMDs idle (870^2 T = 4 6.1 us a step, in chunks by that
// cost 6.3).
template <typename Rows>
StripCut strip_cut(int T, int64_t ny_max, bool dbl, bool walls, Rows rows) {
  StripCut best{T, 0, 1e300};
  double strips_all = 0.0;
  rows([&](int64_t, int64_t strips) { strips_all += (double)strips; });
  // whole columns and a few chunks of them, and the cuts that just fill the
  // SIMDs once and twice (three times: more row streams than the memory likes,
  // 61 us a step at 4096^2 FP32 against 58)
  for (int c = 1; c <= 6; ++c) {
    const int64_t nc = c <= 4 ? c : (int64_t)((c - 4) * 1024.0 / strips_all);
    if (nc < 1 || (nc > 1 && ny_max / nc < 2)) continue;
    const int64_t L = (ny_max + nc - 1) / nc;
    const double cost = strip_cost(T, L, dbl, 1.0, rows);
    if (cost < best.cost) best = StripCut{T, (int32_t)L, cost};
  }
  if (walls && !dbl) best.cost = strip_cost(T, best.L, dbl, 3.0, rows);
  return best;
}

// The cut of one run.
inline StripCut strip_cut_run(int T, int64_t nx, int64_t ny, bool dbl, bool walls) {
  return strip_cut(T, ny, dbl, walls, [&](auto f) { f(ny, (nx + strip_width(T) - 1) / strip_width(T)); });
}

template <typename R, int T>
void launch_strip_t(const RunArgs& args, hipStream_t s) {
  RunArgs a = args;
  const int64_t nsx = (a.nx + strip_width(T) - 1) / strip_width(T);
  const int32_t L = strip_cut_run(T, a.nx, a.ny, sizeof(R) == 8, a.bc[1] != LBM_CDE_PERIODIC).L;
  a.tiles_x = make_fastdiv((uint32_t)nsx);
  const dim3 g((unsigned)(nsx * ((a.ny + L - 1) / L))), b(64);
  const bool wy = a.bc[1] != LBM_CDE_PERIODIC, uc = a.u_kind == U_CONST;
  if (wy && uc) hipLaunchKernelGGL((k_strip_d2q9<R, T, 0, true>), g, b, 0, s, a, L);
  else if (wy) hipLaunchKernelGGL((k_strip_d2q9<R, T, 1, true>), g, b, 0, s, a, L);
  else if (uc) hipLaunchKernelGGL((k_strip_d2q9<R, T, 0, false>), g, b, 0, s, a, L);
  else hipLaunchKernelGGL((k_strip_d2q9<R, T, 1, false>), g, b, 0, s, a, L);
}

// A multi-step launch of a whole batch.
struct StripBatch {
  const BatchRun* runs;
  const uint32_t* tile_start;  // units (strips x chunks of L rows) of the runs
  int nruns;
  const int64_t* clock;
  int64_t toff;
  int flip;
  int32_t L;
  bool uconst, walls;
  unsigned grid;  // a multiple of 64
};

template <typename R, int T>
void launch_strip_batch_t(const StripBatch& v, hipStream_t s) {
  const dim3 g(v.grid), b(64);
#define LBM_STRIP_BATCH(UK, WY)                                                                                  \
  hipLaunchKernelGGL((k_batch_strip_d2q9<R, T, UK, WY>), g, b, 0, s, v.runs, v.tile_start, v.nruns, v.clock, v.toff, \
                     v.flip, v.L)
  if (v.walls && v.uconst) LBM_STRIP_BATCH(0, true);
  else if (v.walls) LBM_STRIP_BATCH(1, true);
  else if (v.uconst) LBM_STRIP_BATCH(0, false);
  else LBM_STRIP_BATCH(1, false);
#undef LBM_STRIP_BATCH
}

void launch_strip_f32(int T, const RunArgs& a, hipStream_t s);
void launch_strip_f64(int T, const RunArgs& a, hipStream_t s);
void launch_strip_batch_f32(int T, const StripBatch& v, hipStream_t s);
void launch_strip_batch_f64(int T, const StripBatch& v, hipStream_t s);

}  // namespace lbm
