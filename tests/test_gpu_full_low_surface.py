"""The fully nonlinear mode with a surface far below z = 0 (a basin part empty): the
distances between surface and bed, and between surface and image, lose nothing
against those of their heights.  W to 1e-11 of the FP64 oracle with its sweep
count in FP64, to 1e-5 in FP32 at 32 points a length of 2 pi and in proportion at
more (the rounding of the derivatives).
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


def _check(gpu, nx, h, depth, level):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    lx = 2 * math.pi
    gs = si.GridSpec(nx, 1, lx, 1.0)
    eta = si.narrowband_random(gs, 1, amp=0.05) + level
    phi = si.narrowband_random(gs, 2, amp=0.1)
    for precision, bar, tol in (("fp64", 1e-11, 1e-10), ("fp32", 1e-5 * nx / 32, 1e-6)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        e = torch.tensor(eta.reshape(1, 1, nx), dtype=dt, device=gpu)
        p = torch.tensor(phi.reshape(1, 1, nx), dtype=dt, device=gpu)
        s = Solver(nx, 1, lx, 1.0, depth, h_ref=h, device=gpu, mode="full", max_sweeps=200, precision=precision)
        W, st, info = s.vertical_velocity(e, p, tol=tol)
        o = OSolver(Grid(nx, 1, lx, 1.0), depth, h_ref=h, mode="full", max_sweeps=200)
        Wo, oi = o.vertical_velocity(e.double().cpu().numpy()[0], p.double().cpu().numpy()[0],
                                     tol=tol if precision == "fp64" else 1e-12)
        err = float(np.abs(W[0].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
        print(f"{precision} {nx} depth {h} level {level}: {err:.2e} sweeps {info[0][0]}/{oi.sweeps}", flush=True)
        assert err < bar and (precision == "fp32" or info[0][0] == oi.sweeps)


@pytest.mark.parametrize("nx", [64, 256])
@pytest.mark.parametrize("h,depth_min,level", [(9.0, 8.4, -8.0), (17.0, 16.0, -15.0), (17.0, 12.0, -10.0)])
def test_over_a_variable_bed(gpu, nx, h, depth_min, level):
    x = np.arange(nx) * 2 * math.pi / nx
    _check(gpu, nx, h, (h - (h - depth_min) * np.exp(np.cos(x - 2.0) - 1.0))[None, :], level)


@pytest.mark.parametrize("nx", [64, 256])
@pytest.mark.parametrize("h,level", [(2.0, -1.5), (5.0, -4.0), (9.0, -8.5), (17.0, -8.0), (17.0, -15.0), (17.0, 10.0)])
def test_over_a_flat_bed(gpu, nx, h, level):
    _check(gpu, nx, h, np.full((1, nx), h), level)
