"""The launch that a D2Q9 run of up to 512^2 nodes starts with (small tiles, one
per CU, eight or four steps) on either side of each line of the rule, against
one-step launches, bitwise: step counts with four-step and one-step remainders
and captured graphs.
"""
import dataclasses

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W
from state_views import populations

pytestmark = pytest.mark.gpu

SEQ = [8, 4, 7, 13, 32, 70]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,kind,tile,steps", [
    (22, 22, "periodic", (8, 8), 8), (128, 128, "periodic", (8, 8), 8), (129, 128, "periodic", (16, 16), 4),
    (256, 191, "periodic", (16, 16), 4), (256, 192, "periodic", (16, 16), 8), (250, 256, "periodic", (16, 16), 8),
    (257, 256, "periodic", (32, 32), 8), (512, 512, "periodic", (32, 32), 8),
    (100, 22, "dfield", (8, 8), 8), (200, 250, "dfield", (16, 16), 8), (300, 290, "dfield", (32, 32), 8),
    (90, 37, "walls", (16, 16), 4), (256, 256, "walls", (16, 16), 4),
])
def test_small_tiles_equal_one_step(nx, ny, kind, tile, steps, precision):
    from paper_1404_2363_amd.solver import Solver
    wl = W.cellular(nx=nx, ny=ny, steps=1, n_hills=3, sigma=5.0)
    kw = {}
    if kind == "dfield":
        rng = W.rng_for(94, nx)
        D = W.dfield_from(*(W.fourier_field(rng, nx, ny, kmax=2) for _ in range(3)))
        wl = dataclasses.replace(wl, D=None, D_field=D)
        kw = {"heat": [1.0, 1.1]}
    elif kind == "walls":
        one = np.ones(1)
        prof = np.sin(np.pi * (np.arange(ny) + 0.5) / ny)
        wl = dataclasses.replace(wl, walls=("periodic", "specular"), D=0.08 * np.eye(2), u_sep=W.SeparableU(
            np.array([0.05, 0.0]), [[np.ones(nx), prof, one], [np.ones(nx), np.zeros(ny), one]]))
    out = []
    for one_step in (True, False):
        s = Solver(wl, precision, **kw)
        if one_step:
            s.set_variant(next(v for v in s.variants() if v["steps_per_launch"] == 1))
        else:
            v = s.variant()
            block = {((8, 8), 8): (8, 64), ((16, 16), 8): (16, 64), ((32, 32), 8): (32, 32), ((16, 16), 4): (16, 32)}
            assert (v["block"], v["steps_per_launch"]) == (block[tile, steps], steps)
        rec = []
        for n in SEQ:
            s.step(n)
            rec.append(populations(s.get_state().cpu().numpy(), 9, wl.nodes, precision)[0])
        assert s.steps_done() == sum(SEQ)
        out.append(rec)
        s.close()
    print(f"case small tiles {nx}x{ny} {kind} {precision}", flush=True)
    for n, a, b in zip(SEQ, *out):
        np.testing.assert_array_equal(a, b, err_msg=f"after {n}")
