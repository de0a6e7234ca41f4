"""Gradients of FP64 grids of 12 to 15 rows, which take three steps per adjoint
launch: bitwise those of one step per launch, and faster."""
import dataclasses
import time

import numpy as np
import pytest

from paper_1404_2363_amd import workloads as W

pytestmark = pytest.mark.gpu


def _gradients(wl, steps, ckpt, D0, phi0, obs):
    import torch
    from paper_1404_2363_amd.adjoint import RolloutSpec, misfit
    D = torch.tensor(D0, dtype=torch.float64, device="cuda:0", requires_grad=True)
    p0 = phi0.clone().requires_grad_(True)
    J = misfit(D, p0, obs, RolloutSpec(wl, steps, steps // 2, ckpt, "fp64", (1.0, 1.1)))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    J.backward()
    torch.cuda.synchronize()
    return D.grad.cpu().numpy(), p0.grad.cpu().numpy(), time.perf_counter() - t0


def _case(nx, ny, velocity):
    import torch
    wl = W.cellular(nx=nx, ny=ny, steps=36, n_hills=3, sigma=4.0)
    if velocity == "const":
        wl = dataclasses.replace(wl, u_sep=None, u_const=np.array([0.03, -0.02]))
    rng = W.rng_for(98, nx)
    D0 = W.dfield_from(*(W.fourier_field(rng, nx, ny, kmax=2) for _ in range(3)))
    phi0 = torch.as_tensor(np.ascontiguousarray(wl.phi0()), dtype=torch.float64, device="cuda:0")
    return wl, D0, phi0, torch.stack([0.9 * phi0 + 0.01 * k for k in range(2)])


@pytest.mark.parametrize("nx,ny,velocity,ckpt", [
    (64, 12, "const", 18), (65, 13, "separable", 11), (121, 15, "const", 9), (200, 14, "separable", 18), (63, 13, "const", 18),
])
def test_low_grids_equal_one_step(nx, ny, velocity, ckpt, monkeypatch):
    case = _case(nx, ny, velocity)
    out = []
    for fused in ("0", "1"):
        monkeypatch.setenv("LBM_CDE_ADJ_FUSED", fused)
        print(f"case adjoint low {nx}x{ny} {velocity} multi-step={fused}", flush=True)
        out.append(_gradients(case[0], 36, ckpt, *case[1:]))
    assert np.abs(out[0][0]).max() > 0
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("nx,ny", [(200, 12), (2048, 14)])
def test_low_grids_are_faster_than_one_step(nx, ny, monkeypatch):
    case = _case(nx, ny, "const")
    best = {"0": 1e9, "1": 1e9}
    for _ in range(6):
        for fused in best:
            monkeypatch.setenv("LBM_CDE_ADJ_FUSED", fused)
            best[fused] = min(best[fused], _gradients(case[0], 200, 100, *case[1:])[2])
    print(f"case adjoint low {nx}x{ny}: {best['1'] * 1e6:.0f} us, one step {best['0'] * 1e6:.0f} us", flush=True)
    assert best["1"] < 0.97 * best["0"]
