"""Gradients through the two tiles of the multi-step adjoint launches, on either
side of the line between them and at the smallest grids of each, against one
step per launch, bitwise: constant and separable velocity, segments with
eight-step, four-step and one-step remainders.
"""
import dataclasses

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,velocity,ckpt", [
    (30, 30, "const", 18), (31, 47, "separable", 12),                        # 16 x 16 tiles, eight steps
    (256, 256, "const", 18), (257, 256, "const", 11), (257, 256, "separable", 18),  # the line between the tiles
    (64, 22, "separable", 12), (65, 23, "const", 11), (176, 480, "const", 11),    # 58-wide tiles, four steps
    (29, 40, "const", 12),                                                    # neither: one step per launch
])
def test_adjoint_tiles_equal_one_step(nx, ny, velocity, ckpt, precision, monkeypatch):
    import torch
    from paper_1404_2363_amd.adjoint import RolloutSpec, misfit
    wl = W.cellular(nx=nx, ny=ny, steps=36, n_hills=3, sigma=4.0)
    if velocity == "const":
        wl = dataclasses.replace(wl, u_sep=None, u_const=np.array([0.03, -0.02]))
    rng = W.rng_for(95, nx)
    D0 = W.dfield_from(*(W.fourier_field(rng, nx, ny, kmax=2) for _ in range(3)))
    dev = "cuda:0"
    phi0 = torch.as_tensor(np.ascontiguousarray(wl.phi0()), dtype=torch.float64, device=dev)
    obs = torch.stack([0.9 * phi0 + 0.01 * k for k in range(2)])
    out = []
    for fused in ("0", "1"):
        monkeypatch.setenv("LBM_CDE_ADJ_FUSED", fused)
        print(f"case adjoint tiles {nx}x{ny} {velocity} {precision} multi-step={fused}", flush=True)
        D = torch.tensor(D0, dtype=torch.float64, device=dev, requires_grad=True)
        p0 = phi0.clone().requires_grad_(True)
        misfit(D, p0, obs, RolloutSpec(wl, 36, 18, ckpt, precision, (1.0, 1.1))).backward()
        out.append((D.grad.cpu().numpy(), p0.grad.cpu().numpy()))
    assert np.abs(out[0][0]).max() > 0
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])
