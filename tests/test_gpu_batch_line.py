"""Ensembles with one-dimensional members, whose steps run in one kernel: states
and statistics equal a context of the member's own bit for bit, over several
calls, calls longer than a captured part (4 steps) and longer than a context's
launch (8), captured and not, beside groups that take the separate passes.
Such groups have no sweep budget.  A member that fails ends the call with its
code; the others' states are those of their own runs.
"""
import math

import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


def _member(nx, seed, amp=0.04, **opts):
    lx = 2 * math.pi * nx / 16
    gs = si.GridSpec(nx, 1, lx, 1.0)
    x = np.arange(nx) * lx / nx
    depth = 1.5 - (0.1 + 0.02 * seed) * np.exp(-((x - lx / 3) ** 2) / (0.02 * lx * lx))
    m = dict(nx=nx, ny=1, lx=lx, ly=1.0, depth=depth[None, :], max_sweeps=200, **opts)
    return m, si.narrowband_random(gs, nx + seed, amp=amp).reshape(1, nx), si.narrowband_random(gs, nx + seed + 50, amp=3 * amp).reshape(1, nx)


def _tensors(mems, gpu):
    import torch
    out = [[torch.tensor(f, dtype=torch.float32 if m.get("precision") == "fp32" else torch.float64, device=gpu) for m, f in
            ((m, (e, p)[i]) for m, e, p in mems)] for i in range(2)]
    return out


def _solver(m, gpu):
    from paper_2310_19840_amd import Solver
    opts = {k: v for k, v in m.items() if k not in ("nx", "ny", "lx", "ly", "depth")}
    return Solver(m["nx"], 1, m["lx"], 1.0, m["depth"], device=gpu, **opts)


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("mode,accel,precision", [("sa", None, "fp64"), ("iter", None, "fp64"), ("iter", "anderson", "fp64"),
                                                  ("iter", "anderson", "fp32")])
def test_members_equal_single_contexts(gpu, mode, accel, precision, graph):
    import torch
    from paper_2310_19840_amd import Batch
    o = dict(mode=mode, accel=accel, precision=precision)
    mems = [_member(nx, s, **o) for s, nx in enumerate((16, 64, 64, 256, 64, 1024, 16, 128, 1024))]
    e, p = _tensors(mems, gpu)
    e1, p1 = _tensors(mems, gpu)
    b = Batch([m for m, _, _ in mems], device=gpu, graph=graph)
    tol = 1e-10 if precision == "fp64" else 1e-5
    single = [_solver(m, gpu) for m, _, _ in mems]
    for n in (9, 1, 0, 4, 9):
        st, info = b.step(e, p, 0.05, n, tol=tol)
        assert st == 0
        for i, s in enumerate(single):
            _, d = s.step(e1[i], p1[i], 0.05, n, tol=tol)
            assert torch.equal(e[i], e1[i]) and torch.equal(p[i], p1[i]), (n, i)
            assert [info[i][k] for k in ("solves", "sweeps_total", "sweeps_max")] == [d[k] for k in ("solves", "sweeps_total", "sweeps_max")]
    budgets, redos = b.budgets()
    assert budgets == [200] * len(b.groups()) and redos == 0


def test_beside_separate_passes(gpu):
    import torch
    from paper_2310_19840_amd import Batch
    o = dict(mode="iter", accel="anderson")
    mems = [_member(64, 0, **o), _member(2048, 1, **o), _member(64, 2, dealias=0.8, **o), _member(256, 3, **o)]
    e, p = _tensors(mems, gpu)
    e1, p1 = _tensors(mems, gpu)
    b = Batch([m for m, _, _ in mems], device=gpu)
    for n in (2, 5, 5):
        b.step(e, p, 0.05, n, tol=1e-10)
        for i, (m, _, _) in enumerate(mems):
            _solver(m, gpu).step(e1[i], p1[i], 0.05, n, tol=1e-10)
            assert torch.equal(e[i], e1[i]) and torch.equal(p[i], p1[i]), (n, i)
    budgets, _ = b.budgets()
    assert budgets[0] == budgets[3] == 200 and max(budgets[1:3]) < 200


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("mode", ["sa", "iter"])
@pytest.mark.parametrize("bad", ["nan", "steep"])
def test_failing_member(gpu, mode, bad, graph):
    import torch
    from paper_2310_19840_amd import Batch, SBIError
    mems = [_member(128, s, mode=mode) for s in range(3)]
    if bad == "nan":
        mems[1][1][0, 5] = np.nan
    else:
        mems[1] = _member(128, 1, amp=5.0, mode=mode)
    e, p = _tensors(mems, gpu)
    e1, p1 = _tensors(mems, gpu)
    b = Batch([m for m, _, _ in mems], device=gpu, graph=graph)
    with pytest.raises(SBIError) as err:
        b.step(e, p, 0.05, 6, tol=1e-10)
    assert err.value.code == -5 if bad == "nan" or mode == "sa" else err.value.code in (-5, -6)
    for i in (0, 2):
        _solver(mems[i][0], gpu).step(e1[i], p1[i], 0.05, 6, tol=1e-10)
        assert torch.equal(e[i], e1[i]) and torch.equal(p[i], p1[i]), i
    # the next call of the same ensemble with every member sound again
    e[1], p[1] = e[0].clone(), p[0].clone()
    assert b.step(e, p, 0.05, 2, tol=1e-10)[0] == 0


def test_autotune_leaves_one_kernel_groups_alone(gpu):
    from paper_2310_19840_amd import Batch
    o = dict(mode="iter", accel="anderson")
    line = [_member(64, 0, **o)[0], _member(256, 1, **o)[0]]
    for mems, alone in ((line[:1], True), (line, True), (line + [_member(2048, 2, **o)[0]], False)):
        plans = Batch(mems, device=gpu, autotune=True).plans()
        for q in plans[:len(plans) if alone else 2]:
            assert (q["row_variant"], q["row_rows"], q["col_split"]) == (0, 0, 0)
