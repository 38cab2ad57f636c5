"""One-dimensional solves and steps in one kernel against the separate passes
(which a profiled context keeps): every transform length it takes, both
precisions, the plain method and the iteration with and without mixing, one
member and several, orders from the smallest up, a band below the half, beds
and flat, the tank's pressures, zones and filter.  Both sides evaluate the
same sums in another order: 1e-11 (FP64, iterated to 1e-12 with the same
sweeps) and 2e-5 (FP32) of the largest value.  A non-finite member ends both
with the same code and leaves the state alone.
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


def _case(nx, batch, bed):
    lx = 2 * math.pi * nx / 16
    gs = si.GridSpec(nx, 1, lx, 1.0)
    x = np.arange(nx) * lx / nx
    depth = np.stack([1.5 - (0.2 + 0.05 * b) * np.exp(-((x - lx / 3) ** 2) / (0.02 * lx * lx)) * bed for b in range(batch)])
    eta = np.stack([si.narrowband_random(gs, nx + b, amp=0.04) for b in range(batch)])
    phi = np.stack([si.narrowband_random(gs, nx + 9 + b, amp=0.2) for b in range(batch)])
    return lx, depth.reshape(batch, 1, nx), eta.reshape(batch, 1, nx), phi.reshape(batch, 1, nx)


@pytest.mark.parametrize("nx", [16, 32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("batch,order,bed,dealias", [(1, 7, 1, 0.5), (3, 6, 1, 0.5), (2, 7, 0, 0.3), (1, 3, 1, 0.45),
                                                     (1, 2, 0, 0.5), (1, 1, 1, 0.5)])
def test_matches_separate_passes(gpu, nx, batch, order, bed, dealias):
    import torch
    from paper_2310_19840_amd import Solver
    lx, depth, eta, phi = _case(nx, batch, bed)
    for precision, bar in (("fp64", 1e-11), ("fp32", 2e-5)):
        dt = torch.float64 if precision == "fp64" else torch.float32
        tol = 1e-12 if precision == "fp64" else 1e-6
        for mode, accel in (("sa", None), ("iter", None), ("iter", "anderson")):
            out = []
            for separate in (False, True):
                s = Solver(nx, 1, lx, 1.0, depth, h_ref=1.5, batch=batch, device=gpu, mode=mode, accel=accel, order=order,
                           precision=precision, dealias=dealias, max_sweeps=200,
                           filter_beta=(9.0, 8.0) if order == 6 else None)
                if separate:
                    s.profile()
                e, p = (torch.tensor(a, dtype=dt, device=gpu) for a in (eta, phi))
                W, st, info = s.vertical_velocity(e, p, tol=tol)
                if order == 7:
                    s.set_wavemaker([(0.02, 1.0, 0.95, 0.3)], x0=0.8 * lx, width=0.1 * lx)
                if order >= 6:
                    s.set_relaxation(0.03, 1.0, 0.95, 0.1 * lx, 0.15 * lx, 2.0)
                st2, d = s.step(e, p, 0.05, 3, tol=tol, t=0.4)
                out.append((W, e, p, st, st2, [i[0] for i in info], d["sweeps_total"], d["solves"], d["t"]))
            for a, b in zip(out[0][:3], out[1][:3]):
                err = float(((a - b).abs().max() / b.abs().max()).double())
                print(f"{precision} {mode} {accel} {nx} order {order}: {err:.2e}", flush=True)
                assert err < bar
            assert out[0][7:] == out[1][7:]
            if precision == "fp64":
                assert out[0][3:7] == out[1][3:7]


@pytest.mark.parametrize("nx", [64, 1024])
@pytest.mark.parametrize("mode", ["sa", "iter"])
def test_nonfinite_member(gpu, nx, mode):
    import torch
    from paper_2310_19840_amd import SBIError, Solver
    lx, depth, eta, phi = _case(nx, 3, 1)
    eta[1, 0, 5] = np.nan
    for separate in (False, True):
        s = Solver(nx, 1, lx, 1.0, depth, h_ref=1.5, batch=3, device=gpu, mode=mode)
        if separate:
            s.profile()
        e, p = (torch.tensor(a, device=gpu) for a in (eta, phi))
        keep = e.clone(), p.clone()
        for call in (lambda: s.vertical_velocity(e, p), lambda: s.step(e, p, 0.05, 2)):
            with pytest.raises(SBIError) as err:
                call()
            assert err.value.code == -5
        assert torch.equal(e.nan_to_num(), keep[0].nan_to_num()) and torch.equal(p, keep[1])


@pytest.mark.parametrize("amp", [0.12, 0.2, 0.3, 0.6])
def test_first_failure_is_reported(gpu, amp):
    # member 1 is non-finite at once; member 0, at the steeper amplitudes, fails some steps later with another code
    import torch
    from paper_2310_19840_amd import SBIError, Solver
    lx, depth, eta, phi = _case(128, 2, 1)
    eta[0] *= amp / 0.04
    phi[0] *= amp / 0.04
    eta[1, 0, 7] = np.inf
    codes = []
    for separate in (False, True):
        s = Solver(128, 1, lx, 1.0, depth, h_ref=1.5, batch=2, device=gpu, mode="iter", max_sweeps=100)
        if separate:
            s.profile()
        with pytest.raises(SBIError) as err:
            s.step(*(torch.tensor(a, device=gpu) for a in (eta, phi)), 0.1, 7, tol=1e-10)
        codes.append(err.value.code)
    assert codes[0] == codes[1]
