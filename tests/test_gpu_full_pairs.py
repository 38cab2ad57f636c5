"""The fully nonlinear mode's pair passes at the sizes where their tiles and
lanes change (below one tile, one and two tiles, a source block shorter than
the lanes' shares) and for geometries that leave the logarithm's series for
the library function: a bed that rises to a quarter of the depth, and deep
water without image.  W to 1e-11 (FP64) and 1e-5 (FP32) of the FP64 oracle with
its sweep count, two members of different beds in one context.  Many members
or points in all take blocks of two tiles a side, from one such block up: the same bounds.
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("h,rise", [(1.0, 0.0), (1.0, 0.75), (400.0, 0.0)])
def test_w_matches_oracle(gpu, nx, h, rise):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    lx = 2 * math.pi * max(1, nx // 32)
    gs = si.GridSpec(nx, 1, lx, 1.0)
    x = np.arange(nx) * lx / nx
    depth = np.stack([h - rise * np.exp(-((x - 0.4 * lx) / (0.15 * lx)) ** 2),
                      h - 0.5 * rise * np.exp(-((x - 0.6 * lx) / (0.2 * lx)) ** 2)])[:, None, :]
    eta = np.stack([si.narrowband_random(gs, nx + b, amp=0.1) for b in range(2)])
    phi = np.stack([si.narrowband_random(gs, nx + 10 + b, amp=0.15) for b in range(2)])
    for precision, bar in (("fp64", 1e-11), ("fp32", 1e-5)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        e = torch.tensor(eta.reshape(2, 1, nx), dtype=dt, device=gpu)
        p = torch.tensor(phi.reshape(2, 1, nx), dtype=dt, device=gpu)
        s = Solver(nx, 1, lx, 1.0, depth, h_ref=h, batch=2, device=gpu, mode="full", max_sweeps=200, precision=precision)
        W, st, info = s.vertical_velocity(e, p, tol=1e-12 if precision == "fp64" else 1e-6)
        for b in range(2):
            o = OSolver(Grid(nx, 1, lx, 1.0), depth[b], h_ref=h, mode="full", max_sweeps=200)
            Wo, oi = o.vertical_velocity(e[b].double().cpu().numpy(), p[b].double().cpu().numpy(), tol=1e-12)
            err = float(np.abs(W[b].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
            print(f"{precision} {nx} depth {h} rise {rise} member {b}: {err:.2e} sweeps {info[b][0]}/{oi.sweeps}", flush=True)
            if precision == "fp64":
                assert err < bar and info[b][0] == oi.sweeps
            else:
                assert err < bar


@pytest.mark.parametrize("nx,batch", [(128, 130), (256, 66), (1024, 17)])
def test_two_tile_blocks(gpu, nx, batch):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    lx = 2 * math.pi * (nx // 32)
    gs = si.GridSpec(nx, 1, lx, 1.0)
    eta = np.stack([si.narrowband_random(gs, nx + b, amp=0.1) for b in range(batch)])
    phi = np.stack([si.narrowband_random(gs, nx + 500 + b, amp=0.15) for b in range(batch)])
    e = torch.tensor(eta.reshape(batch, 1, nx), device=gpu)
    p = torch.tensor(phi.reshape(batch, 1, nx), device=gpu)
    s = Solver(nx, 1, lx, 1.0, np.ones((batch, 1, nx)), h_ref=1.0, batch=batch, device=gpu, mode="full", max_sweeps=200)
    W, st, info = s.vertical_velocity(e, p, tol=1e-12)
    for b in (0, batch - 1):
        o = OSolver(Grid(nx, 1, lx, 1.0), np.ones((1, nx)), h_ref=1.0, mode="full", max_sweeps=200)
        Wo, oi = o.vertical_velocity(e[b].cpu().numpy(), p[b].cpu().numpy(), tol=1e-12)
        err = float(np.abs(W[b].cpu().numpy() - Wo).max() / np.abs(Wo).max())
        print(f"{nx} member {b}: {err:.2e} sweeps {info[b][0]}/{oi.sweeps}", flush=True)
        assert err < 1e-11 and info[b][0] == oi.sweeps
