"""The multi-step launches of D2Q9 runs with walls on both axes against one-step
launches, bitwise: grids smaller than a tile, of one node more than whole tiles
and with single columns left over; constant and separable velocity; the launch
that such a run starts with.
"""
import dataclasses

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W
from state_views import populations

pytestmark = pytest.mark.gpu

SEQ = [4, 7, 50]


def _workload(nx, ny, walls, u):
    wl = W.cellular(nx=nx, ny=ny, steps=1, n_hills=2, sigma=3.0)
    kw = {"u_sep": None, "u_const": np.array([0.02, -0.01])}
    if u == "separable":
        one = np.ones(1)
        sx, sy = np.sin(np.pi * (np.arange(nx) + 0.5) / nx), np.sin(np.pi * (np.arange(ny) + 0.5) / ny)
        kw = {"u_sep": W.SeparableU(np.array([0.05, 0.03]), [[sx, sy, one], [sx, sy, one]])}
    D = np.array([[0.08, 0.02], [0.02, 0.05]])
    return dataclasses.replace(wl, walls=walls, D=D, **kw)


def _run(wl, precision, variant):
    from paper_1404_2363_amd.solver import Solver
    s = Solver(wl, precision)
    if variant:
        s.set_variant(variant)
    got, rec = s.variant(), []
    for n in SEQ:
        s.step(n)
        rec.append(populations(s.get_state().cpu().numpy(), 9, wl.nodes, precision)[0])
    s.close()
    return got, rec


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,walls,u", [
    (5, 3, ("bounce", "bounce"), "separable"), (16, 17, ("specular", "bounce"), "const"),
    (33, 22, ("bounce", "specular"), "separable"), (65, 38, ("specular", "specular"), "const"),
    (64, 33, ("specular", "specular"), "separable"), (130, 49, ("bounce", "bounce"), "separable"),
    (97, 64, ("bounce", "specular"), "const"), (129, 70, ("specular", "bounce"), "separable"),
])
def test_box_variants_equal_one_step(nx, ny, walls, u, precision):
    from paper_1404_2363_amd.solver import Solver
    wl = _workload(nx, ny, walls, u)
    s = Solver(wl, precision)
    variants = s.variants()
    s.close()
    multi = [v for v in variants if v["steps_per_launch"] > 1]
    assert len(multi) == 2
    print(f"case box {nx}x{ny} {walls} {u} {precision}: {len(multi)} variants", flush=True)
    _, want = _run(wl, precision, next(v for v in variants if v["steps_per_launch"] == 1))
    for v in multi:
        _, got = _run(wl, precision, v)
        for a, b in zip(want, got):
            np.testing.assert_array_equal(a, b, err_msg=str(v))


@pytest.mark.parametrize("precision,nx,ny,walls,block", [
    ("fp32", 30, 40, ("bounce", "periodic"), (256, 1)), ("fp32", 2, 1, ("bounce", "specular"), (16, 32)),
    ("fp32", 512, 768, ("bounce", "specular"), (16, 32)), ("fp64", 513, 768, ("bounce", "specular"), (32, 16)),
    ("fp32", 2000, 1000, ("specular", "bounce"), (32, 16)),
])
def test_box_start(precision, nx, ny, walls, block):
    wl = _workload(nx, ny, walls, "separable")
    print(f"case box start {nx}x{ny} {walls} {precision}", flush=True)
    got, rec = _run(wl, precision, None)
    assert got["block"] == block
    from paper_1404_2363_amd.solver import Solver
    s = Solver(wl, precision)
    one = next(v for v in s.variants() if v["steps_per_launch"] == 1)
    s.close()
    for a, b in zip(_run(wl, precision, one)[1], rec):
        np.testing.assert_array_equal(a, b)
