"""Two D3Q15 steps per launch against one-step launches, bitwise: grids around
one and two tiles (64 x 8 and 32 x 16 columns in FP32, 32 x 8 and 32 x 13 in
FP64), down to a single node, chunks of few planes, walls across and along the
marching direction, constant and separable velocities, odd step counts.
"""
import dataclasses

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W
from state_views import populations

pytestmark = pytest.mark.gpu

SEQ = [2, 1, 3, 32, 5]
P, S, B = "periodic", "specular", "bounce"


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape,walls,velocity", [
    ((1, 1, 1), (P, P, P), "const"), ((1, 1, 1), (S, S, B), "const"), ((3, 2, 1), (P, P, S), "const"),
    ((64, 8, 5), (P, P, P), "separable"), ((65, 9, 7), (P, P, B), "separable"), ((33, 17, 2), (S, P, P), "const"),
    ((32, 13, 40), (P, S, S), "separable"), ((130, 27, 11), (P, P, P), "separable"), ((31, 14, 3), (S, S, B), "const"),
    ((70, 33, 21), (S, S, S), "separable"), ((40, 16, 90), (P, S, P), "separable"),
])
def test_two_steps_equal_one_step(shape, walls, velocity, precision):
    from paper_1404_2363_amd.solver import Solver
    nx, ny, nz = shape
    wl = W.sine3d(n=nx, ny=ny, nz=nz, steps=1, n_hills=3, sigma=3.0)
    wl.walls = walls
    if velocity == "const":
        wl = dataclasses.replace(wl, u_sep=None, u_const=np.array([0.03, -0.02, 0.01]), D=0.05 * np.eye(3))
    kw = {"stability_check": False}
    ref = Solver(wl, precision, **kw)
    assert ref.variant()["steps_per_launch"] == 2
    two = [v for v in ref.variants() if v["steps_per_launch"] == 2]
    assert len(two) == 2
    ref.set_variant(next(v for v in ref.variants() if v["steps_per_launch"] == 1))
    want = []
    for n in SEQ:
        ref.step(n)
        want.append(populations(ref.get_state().cpu().numpy(), 15, wl.nodes, precision)[0])
    ref.close()
    print(f"case two steps {shape} {walls} {velocity} u {precision}", flush=True)
    for v in two:
        s = Solver(wl, precision, **kw)
        s.set_variant(v)
        for n, w in zip(SEQ, want):
            s.step(n)
            got = populations(s.get_state().cpu().numpy(), 15, wl.nodes, precision)[0]
            np.testing.assert_array_equal(got, w, err_msg=f"{v} after {n}")
        assert s.steps_done() == sum(SEQ)
        s.close()


def test_refused_with_bounced_columns_and_fields():
    from paper_1404_2363_amd.solver import Solver
    wl = W.sine3d(n=40, ny=16, nz=8, steps=1, n_hills=2, sigma=3.0)
    wl.walls = (P, B, P)
    s = Solver(wl, "fp32")
    assert all(v["steps_per_launch"] == 1 for v in s.variants())
    s.close()
    wl.walls = (P, P, P)
    wl.u_field, wl.u_sep = wl.u(), None
    s = Solver(wl, "fp32")
    assert all(v["steps_per_launch"] == 1 for v in s.variants())
    s.close()
