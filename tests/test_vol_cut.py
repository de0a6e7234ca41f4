"""The cut of D3Q15 grids for the launches of two steps (csrc/vol_cut.hpp, host
arithmetic): the tile that a run starts with against the measured times, and the
bounds that a launch relies on over grids of every proportion."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1404_2363_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "vol_cut.hpp"

int main() {
  long nx, ny, nz;
  int dbl, wz;
  while (std::scanf("%ld %ld %ld %d %d", &nx, &ny, &nz, &dbl, &wz) == 5) {
    lbm::VolCut c[2];
    for (int k = 0; k < 2; ++k) c[k] = lbm::vol_cut(lbm::kVolTiles[dbl][k][0], lbm::kVolTiles[dbl][k][1], dbl, wz, nx, ny, nz);
    std::printf("%d %d", c[1].cost < c[0].cost ? 1 : 0, (int)lbm::vol_one_step(wz, dbl, nx, ny, nz));
    for (int k = 0; k < 2; ++k) std::printf(" %d %d %d", c[k].tx, c[k].ty, c[k].L);
    std::printf("\n");
  }
}
"""
TILES = [[(64, 8), (32, 16)], [(32, 8), (32, 13)]]


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("vol_cut")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")],
                   check=True, capture_output=True, text=True)

    def run(grids, wz=0):
        text = "".join(f"{nx} {ny} {nz} {dbl} {wz}\n" for (nx, ny, nz), dbl in grids)
        out = subprocess.run([str(d / "t")], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        rows = [[int(v) for v in line.split()] for line in out.splitlines()]
        assert len(rows) == len(grids)
        return [(r[0], r[1], (tuple(r[2:5]), tuple(r[5:8]))) for r in rows]
    return run


def test_start_tile(cut):
    # (grid, fp64, tile): the faster of the two where they differ by more than 3 %
    pins = [((256, 256, 256), 0, (64, 8)), ((256, 256, 256), 1, (32, 8)), ((101, 90, 77), 1, (32, 13)),
            ((256, 256, 64), 0, (64, 8)), ((256, 256, 64), 1, (32, 8)), ((700, 300, 20), 0, (64, 8)),
            ((200, 200, 200), 0, (64, 8)), ((1, 20000, 1), 0, (32, 16))]
    for (first, one, _), (grid, dbl, tile) in zip(cut([(g, d) for g, d, _ in pins]), pins):
        assert TILES[dbl][first] == tile and not one, (grid, dbl)
    for grid in [(128, 128, 128), (256, 256, 256), (384, 384, 384)]:
        assert [TILES[d][r[0]] for d, r in zip((0, 1), cut([(grid, 0), (grid, 1)], wz=1))] == [(64, 8), (32, 13)], grid


def test_small_and_thin_grids_are_cut(cut):
    # blocks of the grid's own columns, enough of them for the 256 CUs where the planes allow it
    for grid in [(8, 8, 4096), (16, 16, 2000), (5, 7, 300), (3, 2, 5000), (8, 8, 8)]:
        for dbl in (0, 1):
            first, one, cuts = cut([(grid, dbl)])[0]
            tx, ty, L = cuts[first]
            assert not one and tx <= grid[0] and ty <= grid[1]
            blocks = -(-grid[0] // tx) * -(-grid[1] // ty) * -(-grid[2] // L)
            assert blocks >= min(256, grid[2]), (grid, dbl, cuts)
    one_step = {((20000, 1, 1), 0): 1, ((1, 1, 20000), 1): 1, ((200, 1, 200), 0): 1, ((1, 1, 1), 0): 0,
                ((1000, 10, 10), 0): 1, ((1000, 10, 10), 1): 1, ((3000, 8, 8), 0): 1, ((3000, 8, 8), 1): 0,
                ((300, 12, 40), 0): 0}
    assert [r[1] for r in cut(list(one_step))] == list(one_step.values())


def test_large_grids_have_even_shares(cut):
    # states past the memory-side cache whose last column of tiles would be mostly padding
    for grid, dbl, first, shape in [((110, 200, 140), 1, (32, 13), (28, 13)), ((110, 200, 140), 0, (64, 8), (55, 8)),
                                    ((150, 150, 150), 1, (32, 13), (30, 13)), ((66, 66, 600), 1, (32, 13), (22, 11)),
                                    ((192, 192, 192), 0, (64, 8), (64, 8)), ((256, 256, 256), 1, (32, 8), (32, 8))]:
        k, one, cuts = cut([(grid, dbl)])[0]
        assert TILES[dbl][k] == first and not one and cuts[k][:2] == shape, (grid, dbl, cuts)


def test_large_fp32_start_tile(cut):
    # where the two tiles lie close, and even shares of 64 columns save no line of the pull
    for grid in [(160, 160, 160), (220, 90, 200), (150, 150, 150), (90, 300, 100)]:
        assert TILES[0][cut([(grid, 0)])[0][0]] == (32, 16), grid
    for grid in [(192, 192, 192), (144, 144, 144), (300, 300, 90), (512, 256, 64)]:
        assert TILES[0][cut([(grid, 0)])[0][0]] == (64, 8), grid


def test_bounds(cut):
    import random
    rng = random.Random(5)
    size = lambda: int(round(2 ** rng.uniform(0, 11)))
    grids = [((size(), size(), size()), d) for _ in range(400) for d in (0, 1)]
    grids += [((1 << 29, 1, 1), 0), ((1, 1 << 29, 1), 1), ((1, 1, 1 << 29), 0)]
    for ((nx, ny, nz), dbl), (_, _, cuts) in zip(grids, cut(grids)):
        for (bx, by), (tx, ty, L) in zip(TILES[dbl], cuts):
            assert 1 <= tx <= min(bx, nx) and 1 <= ty <= min(by, ny) and 1 <= L <= nz
            assert -(-nx // tx) * -(-ny // ty) * -(-nz // L) < 2 ** 31
