"""The fully nonlinear mode over beds that rise far above the reference depth:
mounts in water deep against the wave length, and a reference depth given far
below the bed.  The distance between surface and bed is then far from the flat
geometry's everywhere.  W to 1e-11 of the FP64 oracle with its sweep count in
FP64; in FP32 to 1e-5 at the 32 points a length of 2 pi of the other tests of the
mode, eight times that at the 256 here (the rounding of the derivatives grows as
the largest wave number; a flat bed without image is off by 1e-5 here as well).
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,depth_min,depth_max", [(12.0, 1.0, 12.0), (16.0, 1.0, 16.0), (30.0, 2.0, 30.0), (40.0, 2.0, 40.0),
                                                   (45.0, 3.0, 45.0), (60.0, 0.7, 1.0), (1500.0, 2.0, 3.0)])
def test_w_matches_oracle(gpu, h, depth_min, depth_max):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    nx, lx = 256, 2 * math.pi
    gs = si.GridSpec(nx, 1, lx, 1.0)
    x = np.arange(nx) * lx / nx
    depth = (depth_max - (depth_max - depth_min) * np.exp(np.cos(x - 2.0) - 1.0))[None, :]
    eta = si.narrowband_random(gs, 1, amp=0.05)
    phi = si.narrowband_random(gs, 2, amp=0.1)
    for precision, bar, tol in (("fp64", 1e-11, 1e-10), ("fp32", 8e-5, 1e-6)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        e = torch.tensor(eta.reshape(1, 1, nx), dtype=dt, device=gpu)
        p = torch.tensor(phi.reshape(1, 1, nx), dtype=dt, device=gpu)
        s = Solver(nx, 1, lx, 1.0, depth, h_ref=h, device=gpu, mode="full", max_sweeps=200, precision=precision)
        W, st, info = s.vertical_velocity(e, p, tol=tol)
        o = OSolver(Grid(nx, 1, lx, 1.0), depth, h_ref=h, mode="full", max_sweeps=200)
        Wo, oi = o.vertical_velocity(e.double().cpu().numpy()[0], p.double().cpu().numpy()[0],
                                     tol=tol if precision == "fp64" else 1e-12)
        err = float(np.abs(W[0].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
        print(f"{precision} depth {depth_min} under {h}: {err:.2e} sweeps {info[0][0]}/{oi.sweeps}", flush=True)
        assert err < bar and (precision == "fp32" or info[0][0] == oi.sweeps)
