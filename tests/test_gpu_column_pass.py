"""The column pass where its shapes change: bands wider and narrower than a
quarter (several kept modes per owner at 1024 and 2048 rows, most of a column's
modes kept at the others), columns split into classes (1024, 2048 rows), and
member counts that change the wavefronts per workgroup, in SA mode (sums over
the orders) and in the Anderson-mixed iteration (inner products formed by the
sweep's owners; same sweep count).  Bars as everywhere: W to 1e-11 in FP64,
1e-5 in FP32, against the FP64 oracle.
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,dealias,batch", [
    (16, 16, 0.9, 1), (32, 128, 0.9, 3), (16, 256, 0.3, 1), (16, 512, 0.9, 1), (16, 1024, 0.9, 2),
    (16, 1024, 0.3, 1), (16, 2048, 0.9, 1), (16, 2048, 0.3, 1), (16, 1024, 0.5, 70), (16, 64, 0.5, 1030)])
def test_w_over_bands_and_members(gpu, nx, ny, dealias, batch):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    lx, ly = 2 * math.pi, 2 * math.pi * ny / 16
    gs = si.GridSpec(nx, ny, lx, ly)
    rng = np.random.Generator(np.random.PCG64(nx + ny))
    eta = si.narrowband_random(gs, nx + 7 * ny, amp=0.02)
    phi = si.narrowband_random(gs, nx + 7 * ny + 1, amp=0.1)
    depth = 1.5 - 0.2 * np.exp(-((np.arange(ny) * ly / ny - ly / 2) ** 2)[:, None] / 4.0) * np.ones((1, nx))
    scale = rng.uniform(0.5, 1.0, size=batch)  # members differ in height
    for precision, bar in (("fp64", 1e-11), ("fp32", 1e-5)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        e = torch.tensor(scale[:, None, None] * eta, dtype=dt, device=gpu)
        p = torch.tensor(scale[:, None, None] * phi, dtype=dt, device=gpu)
        for mode, accel in (("sa", None), ("iter", "anderson")):
            tol = 1e-12 if precision == "fp64" else 1e-6
            s = Solver(nx, ny, lx, ly, depth, batch=batch, device=gpu, mode=mode, accel=accel, max_sweeps=200,
                       dealias=dealias, precision=precision)
            W, st, info = s.vertical_velocity(e, p, tol=tol)
            o = OSolver(Grid(nx, ny, lx, ly, dealias=dealias), depth, mode=mode, accel=accel, max_sweeps=200)
            for b in sorted({0, batch - 1}):
                Wo, oi = o.vertical_velocity(e[b].double().cpu().numpy(), p[b].double().cpu().numpy(), tol=1e-12)
                err = float(np.abs(W[b].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
                print(f"{precision} {mode} {nx}x{ny} band {dealias} member {b} of {batch}: {err:.2e}", flush=True)
                assert err < bar
                if mode == "iter" and precision == "fp64":
                    assert info[b][0] == oi.sweeps
