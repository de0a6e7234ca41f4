// How a D3Q15 grid is cut for the launches of two steps (fused_d3q15.hpp): host
// arithmetic only.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <initializer_list>

namespace lbm {

// Tiles built: 64 x 8 and 32 x 16 columns in FP32, 32 x 8 and 32 x 13 in FP64
// (their registers leave room for at most 12 waves per CU in FP32 and 8 in FP64).
constexpr int kVolTiles[2][2][2] = {{{64, 8}, {32, 16}}, {{32, 8}, {32, 13}}};

struct VolCut {
  int32_t tx, ty, L;  // columns of a block, planes of its chunk
  double cost;        // us of a launch, from the fit below
};

// The cut of a launch over tiles of at most bx x by columns.
//
// A block holds a thread per column of its widened tile, so a tile wider than
// the grid, or one of few tiles, is cut down: with whole tiles and at most 64
// chunks 8^3 took 4.7 us a step and 8 x 8 x 4096 55 (one-step launches 3.4 and
// 27), in blocks of the grid's own columns 3.2 and 7.3.  The time of a launch,
// fitted to 6000 cuts of grids from 8^3 to 128^3 (the best cut by it is 1.5 %
// off the best one measured, 16 % at most): a fixed part, then per plane of a
// chunk a part of its own (two barriers and the latency of the pull), one per
// wave and one per cache line of the pull that the CU has to serve, for the k
// blocks that run on it at once.  Blocks share a CU as its LDS and registers
// allow; a started round of blocks costs most of a full one.
// States past the 256 MB memory-side cache wait longer for their planes and are
// bound by memory as well, of which the re-read halo takes a part: the constants
// of a fit of their own, to 3978 cuts of 28 grids up to 256^3 (the best cut by it
// is 0.8 % off the best one measured, 17 % at most; in FP32 a row cut inside a line
// counts a line more there than in cached grids).  Cut into even shares, they
// have no block that is mostly padding: 110 x 200 x 140 FP64 in 28 x 13 columns
// 82 us a step, 107 in 32 x 13; 150^3 93 in 30 columns and 109 in 32.
// 256^3: 64 x 8 197 us a step and 32 x 16 208, which re-reads more lines; FP64
// 32 x 8 407 and 32 x 13 433 (1.9 rounds of blocks); 101 x 90 x 77 FP64 32 x 13
// 19.4, 32 x 8 22.  Between z walls alone (wz) the FP64 kernel takes every
// register, and its planes of 6 waves come slower (128^3 67 us, 32 x 13 59).
inline VolCut vol_cut(int bx, int by, bool dbl, bool wz, int64_t nx, int64_t ny, int64_t nz) {
  const int64_t E = dbl ? 8 : 4, max_waves = dbl ? 8 : 12, lds = 15 * E * (bx + 2) * (by + 2);
  const double bytes = (double)nx * (double)ny * (double)nz * 30.0 * (double)E;
  const bool cached = bytes <= 256e6;
  const double fixed = dbl ? 3.2 : 3.0;
  const double plane = cached ? (dbl ? 1.1 : 1.0) : (dbl ? 0.53 : 0.87);
  const double wave = cached ? (dbl ? 0.19 : 0.07) : (dbl ? 0.34 : 0.07);
  const double line = cached ? (dbl ? 0.008 : 0.0085) : (dbl ? 0.037 : 0.0365);
  // whole tiles and even shares of the grid (along x, where rows then start inside
  // a line, if that saves a sixteenth of the columns: 400 x 30 x 30 FP32 9.4 us a
  // step in 31 columns, 9.0 in 32); of cached states halves and quarters too, which
  // give small grids more blocks
  const int64_t ex = (nx + bx - 1) / bx, ey = (ny + by - 1) / by;
  const int64_t share = 16 * (ex * bx - nx) > nx ? (nx + ex - 1) / ex : bx;
  VolCut best{bx, by, (int32_t)nz, 1e300};
  for (int64_t tx : {(int64_t)bx, (int64_t)bx / 2, (int64_t)bx / 4, (int64_t)8, share}) {
    if (!cached && tx != bx && tx != share) continue;
    tx = std::min(tx, nx);
    for (int64_t ty : {(int64_t)by, (int64_t)by / 2, (int64_t)by / 4, (ny + ey - 1) / ey, (ny + 2 * ey - 1) / (2 * ey)}) {
      if (!cached && ty != by && ty != (ny + ey - 1) / ey) continue;
      ty = std::min(ty, ny);
      const int64_t tiles = (nx + tx - 1) / tx * ((ny + ty - 1) / ty), w = ((tx + 2) * (ty + 2) + 63) / 64;
      const double lines = (double)((ty + 2) * ((tx * E + 127) / 128 + (tx * E % 128 == 0 || (!cached && !dbl) ? 2 : 1)));
      // blocks of more than a wave per SIMD take whole rows of the four SIMDs
      const double cap = (double)std::max<int64_t>(
          1, std::min<int64_t>(160 * 1024 / lds, max_waves / (w <= 4 ? w : (w + 3) / 4 * 4)));
      int64_t last_L = 0;
      for (int64_t blocks : {256, 512, 768, 1024, 1536, 2048}) {
        const int64_t nc = std::max<int64_t>(1, std::min<int64_t>(nz, blocks / tiles)), L = (nz + nc - 1) / nc;
        if (L == last_L) continue;
        last_L = L;
        const double n = (double)(tiles * ((nz + L - 1) / L)) / 256.0, q = n / cap;
        const double rounds = q <= 1.0 ? 1.0 : std::max(q + 0.15, std::ceil(q) - 0.3);
        double t = rounds * (double)(L + 2) * (plane + std::min(cap, std::ceil(n)) * (wave * (double)w + line * lines));
        if (!cached) {
          const double halo = 1.0 + (dbl ? 0.25 : 0.083) * (lines * 128.0 / (double)(tx * ty * E) - 1.0);
          t = std::max(t, bytes * halo * (double)(L + 3) / (double)L / (dbl ? 5.4e6 : 5.6e6) * (q > 1.0 ? rounds / q : 1.0));
        }
        t = (fixed + t) * (wz && dbl && by == 8 ? (cached ? 1.114 : 1.145) : 1.0);
        if (t < best.cost) best = VolCut{(int32_t)tx, (int32_t)ty, (int32_t)L, t};
      }
    }
  }
  return best;
}

// Whether a run starts with one step per launch all the same: without walls,
// grids of one row (the widened tile is three times its own columns: 200 x 1 x
// 200 4.4 us a step, two per launch 4.7, FP64 5.2 and 6.3) and those of long rows,
// which one-step blocks of 128 lanes fill, whose state the L2s hold (1000 x 10 x
// 10 4.4 and 6.2, FP64 5.9 and 7.8; 3000 x 8 x 8 FP64, 46 MB, 12.7 and 9.5), once
// there is more than launching to pay for.
inline bool vol_one_step(bool walls, bool dbl, int64_t nx, int64_t ny, int64_t nz) {
  const double nodes = (double)nx * (double)ny * (double)nz;
  return !walls && nodes > 4096.0 && (ny == 1 || (nx >= 400 && nodes * (dbl ? 240.0 : 120.0) <= 24e6));
}

}  // namespace lbm
