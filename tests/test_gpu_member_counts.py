"""What a member computes does not depend on how many others its context holds:
the same bits alone and among many, where launches take other shapes with the
member count (wavefronts of a column pass, of the one-dimensional column pass,
product chains cut).  Plain method and mixed iteration, with one member against
the FP64 oracle as everywhere (1e-11, FP32 1e-5).
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,dealias,counts", [
    (16, 2048, 0.5, (5, 150)), (16, 2048, 0.9, (40,)), (16, 1024, 0.9, (70, 200)), (32, 1024, 0.5, (40,)),
    (32, 64, 0.5, (3, 300, 1500)), (64, 16, 0.5, (700,)), (16, 512, 0.7, (130,)),
    (2048, 1, 0.5, (5, 60, 400)), (256, 1, 0.8, (3, 150, 1200))])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_alone_and_among_many(gpu, nx, ny, dealias, counts, precision):
    import torch
    from oracle import Grid, Solver as OSolver
    from paper_2310_19840_amd import Solver
    lx, ly = 2 * math.pi * nx / 16, 2 * math.pi * max(1, ny / 16)
    gs = si.GridSpec(nx, ny, lx, ly if ny > 1 else 1.0)
    f64 = precision == "fp64"
    dt = torch.float64 if f64 else torch.float32
    x, y = np.arange(nx) * lx / nx, np.arange(ny) * ly / ny
    depth = 1.5 - 0.2 * np.exp(-((x - lx / 3) / (0.2 * lx)) ** 2)[None, :] * np.exp(-((y - y.mean()) / (0.3 * ly)) ** 2)[:, None]
    eta = [si.narrowband_random(gs, nx + ny + b, amp=0.02).reshape(ny, nx) for b in range(3)]
    phi = [si.narrowband_random(gs, nx + ny + b + 9, amp=0.1).reshape(ny, nx) for b in range(3)]
    for mode, accel in (("sa", None), ("iter", "anderson")):
        def solve(members):
            e, p = (torch.tensor(np.stack([f[b] for b in members]), dtype=dt, device=gpu) for f in (eta, phi))
            s = Solver(nx, ny, lx, ly if ny > 1 else 1.0, depth, batch=len(members), device=gpu, mode=mode, accel=accel,
                       max_sweeps=200, dealias=dealias, precision=precision)
            W, _, info = s.vertical_velocity(e, p, tol=1e-12 if f64 else 1e-6)
            W = W.reshape(len(members), ny, nx)
            s.step(e, p, 0.05, 1, tol=1e-10 if f64 else 1e-5)
            return W, e, p, [i[0] for i in info]
        alone = [solve([b]) for b in range(3)]
        for m in counts:
            members = [b % 3 for b in range(m)]
            many = solve(members)
            for i in (0, 1, 2, m - 1):
                for a, b in zip(alone[members[i]][:3], many[:3]):
                    assert torch.equal(a[0], b[i]), (mode, m, i)
                assert alone[members[i]][3][0] == many[3][i]
        o = OSolver(Grid(nx, ny, lx, ly if ny > 1 else 1.0, dealias=dealias), depth, mode=mode, accel=accel, max_sweeps=200)
        e0, p0 = (torch.tensor(f[0], dtype=dt).double().numpy() for f in (eta, phi))
        Wo, oi = o.vertical_velocity(e0, p0, tol=1e-12)
        err = float(np.abs(alone[0][0][0].double().cpu().numpy() - Wo).max() / np.abs(Wo).max())
        print(f"{precision} {mode} {nx}x{ny} band {dealias}: {err:.2e}", flush=True)
        assert err < (1e-11 if f64 else 1e-5)
        assert not f64 or mode == "sa" or alone[0][3][0] == oi.sweeps
