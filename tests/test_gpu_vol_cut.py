"""Two D3Q15 steps per launch in blocks cut to the grid: thin and small grids,
partial tiles of every kind and single rows against one-step launches, bitwise,
and the launch that large and thin runs start with."""
import dataclasses

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W
from state_views import populations

pytestmark = pytest.mark.gpu

P, S, B = "periodic", "specular", "bounce"


def _workload(shape, walls, velocity):
    nx, ny, nz = shape
    wl = W.sine3d(n=nx, ny=ny, nz=nz, steps=1, n_hills=3, sigma=3.0)
    wl.walls = walls
    if velocity == "const":
        wl = dataclasses.replace(wl, u_sep=None, u_const=np.array([0.03, -0.02, 0.01]), D=0.05 * np.eye(3))
    return wl


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape,walls,velocity", [
    ((8, 8, 300), (P, P, P), "separable"), ((8, 9, 8), (S, S, B), "separable"), ((17, 33, 40), (P, P, B), "const"),
    ((33, 5, 70), (S, P, S), "separable"), ((1, 1, 700), (P, P, P), "const"), ((1, 60, 9), (P, S, P), "separable"),
    ((300, 1, 5), (P, P, P), "const"), ((47, 47, 47), (P, P, P), "separable"), ((19, 26, 2), (S, S, S), "const"),
])
def test_cut_blocks_equal_one_step(shape, walls, velocity, precision):
    from paper_1404_2363_amd.solver import Solver
    wl = _workload(shape, walls, velocity)
    ref = Solver(wl, precision, stability_check=False)
    vs = ref.variants()
    two = [v for v in vs if v["steps_per_launch"] == 2]
    assert len(two) == 2
    want = []
    for v in [next(v for v in vs if v["steps_per_launch"] == 1)] + two:
        print(f"case cut blocks {shape} {walls} {velocity} u {precision} {v['block']}x{v['steps_per_launch']}", flush=True)
        s = Solver(wl, precision, stability_check=False)
        s.set_variant(v)
        for i, n in enumerate([2, 3, 32]):
            s.step(n)
            got = populations(s.get_state().cpu().numpy(), 15, wl.nodes, precision)[0]
            if v["steps_per_launch"] == 1:
                want.append(got)
            np.testing.assert_array_equal(got, want[i], err_msg=f"{v} after {n}")
        s.close()
    ref.close()


@pytest.mark.parametrize("precision,shape,block,steps", [
    ("fp32", (256, 256, 256), (64, 8), 2), ("fp64", (256, 256, 256), (32, 8), 2), ("fp64", (101, 90, 77), (32, 13), 2),
    ("fp32", (6000, 1, 1), (128, 1), 1), ("fp64", (80, 1, 80), (128, 1), 1),
])
def test_start(precision, shape, block, steps):
    from paper_1404_2363_amd.solver import Solver
    s = Solver(_workload(shape, (P, P, P), "separable"), precision)
    v = s.variant()
    s.close()
    assert (v["block"], v["steps_per_launch"]) == (block, steps)
