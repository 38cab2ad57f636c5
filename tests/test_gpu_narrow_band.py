"""Narrow kept bands: a column pass has far more threads than kept modes (down
to one mode a column), and a thread without a mode reads and writes nothing
beyond the workgroup's areas.  Iteration with and without mixing (whose
products come order by order) and the plain method, random waves of the kept
modes over a bed: W to 1e-11 in FP64 and 1e-5 in FP32 of the FP64 oracle, the
same sweep count in FP64.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _waves(nx, ny, lx, ly, dealias, seed, amp):
    rng = np.random.Generator(np.random.PCG64(seed))
    X, Y = np.meshgrid(np.arange(nx) * lx / nx, np.arange(ny) * ly / ny)
    mx, my = (math.ceil(dealias * n / 2 - 1e-9) - 1 for n in (nx, ny))
    f = np.zeros((ny, nx))
    for m in range(min(mx, 3) + 1):
        for l in range(-min(my, 2), min(my, 2) + 1):
            if m or l > 0:
                f += rng.normal() * np.cos(2 * np.pi * (m * X / lx + l * Y / ly) + rng.uniform(0, 2 * np.pi))
    return amp * f / np.abs(f).max()


@pytest.mark.parametrize("nx,ny,dealias,batch", [(128, 16, 0.1, 1), (128, 32, 0.05, 3), (64, 64, 0.1, 1), (128, 64, 0.05, 70),
                                                 (64, 512, 0.05, 1), (64, 1024, 0.05, 1), (64, 2048, 0.05, 2)])
def test_w_matches_oracle(gpu, nx, ny, dealias, batch):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    lx, ly = 4 * math.pi, 4 * math.pi * max(1, ny // 128)
    eta, phi = (_waves(nx, ny, lx, ly, dealias, nx + ny + s, a) for s, a in ((0, 0.05), (1, 0.1)))
    depth = 1.5 - 0.3 * _waves(nx, ny, lx, ly, dealias, nx + ny + 2, 1.0) ** 2
    for precision, bar in (("fp64", 1e-11), ("fp32", 1e-5)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        e, p = (torch.tensor(np.broadcast_to(a, (batch, ny, nx)).copy(), dtype=dt, device=gpu) for a in (eta, phi))
        for mode, accel in (("iter", None), ("iter", "anderson"), ("sa", None)):
            s = Solver(nx, ny, lx, ly, depth, batch=batch, device=gpu, mode=mode, accel=accel, max_sweeps=200,
                       dealias=dealias, precision=precision)
            W, st, info = s.vertical_velocity(e, p, tol=1e-12 if precision == "fp64" else 1e-6)
            o = OSolver(Grid(nx, ny, lx, ly, dealias=dealias), depth, mode=mode, accel=accel, max_sweeps=200)
            Wo, oi = o.vertical_velocity(e[0].double().cpu().numpy(), p[0].double().cpu().numpy(), tol=1e-12)
            for b in sorted({0, batch - 1}):
                err = float(np.abs(W[b].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
                print(f"{precision} {mode} {accel} {nx}x{ny} band {dealias} member {b}: {err:.2e}", flush=True)
                assert err < bar
                if mode == "iter" and precision == "fp64":
                    assert info[b][0] == oi.sweeps
