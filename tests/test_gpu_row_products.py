"""Row passes whose product chains are cut into pieces (few rows over all
members) beside uncut ones, at every expansion order: the SA orders by forward
scatter and the iteration's sweeps, with and without a variable bed, 1D and
2D, one member and enough of them to leave the chains whole.  W to 1e-11
(FP64) and 1e-5 (FP32) of the FP64 oracle, iterations with its sweep count.
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,batch,bed", [(64, 1, 1, True), (64, 32, 1, True), (128, 16, 2, False),
                                             (1024, 16, 40, True), (2048, 16, 1, False), (16, 16, 200, True)])
@pytest.mark.parametrize("order", [1, 2, 3, 6, 7])
def test_w_at_every_order(gpu, nx, ny, batch, bed, order):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import SBIError, Solver
    lx, ly = 2 * math.pi * nx / 16, 2 * math.pi * max(ny, 16) / 16
    gs = si.GridSpec(nx, ny, lx, ly)
    eta = si.narrowband_random(gs, nx + ny, amp=0.04)
    phi = si.narrowband_random(gs, nx + ny + 1, amp=0.2)
    x = np.arange(nx) * lx / nx
    depth = 1.5 - (0.3 * np.exp(-((x - lx / 3) ** 2) / (0.02 * lx * lx)) if bed else 0.0) * np.ones((ny, nx))
    for precision, bar in (("fp64", 1e-11), ("fp32", 1e-5)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        e = torch.tensor(np.broadcast_to(eta, (batch, ny, nx)).copy(), dtype=dt, device=gpu)
        p = torch.tensor(np.broadcast_to(phi, (batch, ny, nx)).copy(), dtype=dt, device=gpu)
        for mode, accel in (("sa", None), ("iter", None), ("iter", "anderson")):
            s = Solver(nx, ny, lx, ly, depth, batch=batch, device=gpu, mode=mode, accel=accel, max_sweeps=200,
                       order=order, precision=precision)
            tol = 1e-12 if precision == "fp64" else 1e-6
            o = OSolver(Grid(nx, ny, lx, ly), depth, mode=mode, accel=accel, max_sweeps=200, order=order)
            Wo, oi = o.vertical_velocity(e[0].double().cpu().numpy(), p[0].double().cpu().numpy(), tol=1e-12)
            if oi.status != 0 and precision == "fp32":
                continue  # it stops at its own, looser tolerance before the FP64 iteration's end
            if oi.status < 0:
                # order 2 over this bed expands: the same end on both sides
                with pytest.raises(SBIError) as err:
                    s.vertical_velocity(e, p, tol=tol)
                assert err.value.code == oi.status
                continue
            W, st, info = s.vertical_velocity(e, p, tol=tol)
            if oi.status > 0:
                assert st == oi.status and info[0][0] == oi.sweeps
                continue
            for b in sorted({0, batch - 1}):
                err = float(np.abs(W[b].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
                print(f"{precision} {mode} {accel} {nx}x{ny} order {order} member {b}: {err:.2e}", flush=True)
                assert err < bar
                if mode == "iter" and precision == "fp64":
                    assert info[b][0] == oi.sweeps
