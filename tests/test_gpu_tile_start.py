"""The tile that a D2Q9 run between the small tiles and the marching launch
starts with, on either side of each line of the rule (tiles on the fullest of
the 256 CUs times their rows), against one-step launches, bitwise.
"""
import dataclasses

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W
from state_views import populations

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,nx,ny,kind,block", [
    ("fp32", 513, 600, "periodic", (64, 12)), ("fp32", 700, 552, "periodic", (64, 12)),
    ("fp32", 700, 553, "periodic", (64, 8)), ("fp32", 705, 600, "dfield", (64, 8)),
    ("fp32", 760, 760, "dfield", (64, 8)),
    ("fp32", 512, 256, "walls", (16, 32)), ("fp32", 513, 256, "walls", (64, 8)), ("fp32", 513, 500, "walls", (64, 12)),
    ("fp32", 513, 700, "walls", (64, 8)),
    ("fp64", 520, 520, "periodic", (64, 12)), ("fp64", 640, 600, "periodic", (64, 12)),
    ("fp64", 641, 560, "periodic", (64, 1)), ("fp64", 520, 520, "dfield", (64, 12)),
    ("fp64", 700, 600, "dfield", (64, 4)), ("fp64", 513, 256, "walls", (64, 4)), ("fp64", 2000, 150, "walls", (64, 12)),
])
def test_start_tiles_equal_one_step(precision, nx, ny, kind, block):
    from paper_1404_2363_amd.solver import Solver
    wl = W.cellular(nx=nx, ny=ny, steps=1, n_hills=3, sigma=5.0)
    kw = {}
    if kind == "dfield":
        rng = W.rng_for(96, nx)
        wl = dataclasses.replace(wl, D=None, D_field=W.dfield_from(*(W.fourier_field(rng, nx, ny, kmax=2)
                                                                    for _ in range(3))))
        kw = {"heat": [1.0, 1.1]}
    elif kind == "walls":
        one = np.ones(1)
        prof = np.sin(np.pi * (np.arange(ny) + 0.5) / ny)
        wl = dataclasses.replace(wl, walls=("periodic", "bounce"), D=0.08 * np.eye(2), u_sep=W.SeparableU(
            np.array([0.05, 0.0]), [[np.ones(nx), prof, one], [np.ones(nx), np.zeros(ny), one]]))
    print(f"case start tile {nx}x{ny} {kind} {precision}", flush=True)
    out = []
    for one_step in (True, False):
        s = Solver(wl, precision, **kw)
        if one_step:
            s.set_variant(next(v for v in s.variants() if v["steps_per_launch"] == 1))
        else:
            assert s.variant()["block"] == block
        rec = []
        for n in (4, 9, 50):
            s.step(n)
            rec.append(populations(s.get_state().cpu().numpy(), 9, wl.nodes, precision)[0])
        out.append(rec)
        s.close()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
