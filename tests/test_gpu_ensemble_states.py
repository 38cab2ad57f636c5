"""The states of an ensemble's members come from and go to wherever the caller
keeps them: tensors of their own, pieces of one buffer at odd offsets (whose
neighbours stay untouched), more members than one launch copies, one tensor
given for two members of the same bed.  Bitwise the same states each way, call
after call, captured and not.
"""
import numpy as np
import pytest

import sbi_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("precision,mode", [("fp32", "sa"), ("fp64", "iter")])
def test_states_wherever_they_lie(gpu, precision, mode, graph):
    import torch
    from paper_2310_19840_amd import Batch
    dt = torch.float32 if precision == "fp32" else torch.float64
    mems, eta, phi = [], [], []
    for k in range(133):
        nx, ny = (16, 16) if k < 130 else (64, 32)
        gs = si.GridSpec(nx, ny, 2 * np.pi * nx / 16, 2 * np.pi * ny / 16)
        mems.append(dict(nx=nx, ny=ny, lx=gs.lx, ly=gs.ly, precision=precision, mode=mode,
                         depth=1.5 - 0.1 * np.cos(gs.x() * (1 + k % 3) * 16 / nx)[None, :] * np.ones((ny, 1))))
        eta.append(torch.tensor(si.narrowband_random(gs, k, amp=0.03).reshape(ny, nx), dtype=dt, device=gpu))
        phi.append(torch.tensor(si.narrowband_random(gs, 500 + k, amp=0.1).reshape(ny, nx), dtype=dt, device=gpu))
    mems[2] = dict(mems[2], depth=mems[1]["depth"])

    def pieces(fields):
        n = sum(f.numel() + 1 for f in fields) + 1
        flat = torch.full((n,), 7.0, dtype=dt, device=gpu)
        out, o = [], 1
        for f in fields:
            out.append(flat[o:o + f.numel()].view(f.shape))
            out[-1].copy_(f)
            o += f.numel() + 1
        return flat, out

    b = Batch(mems, device=gpu, graph=graph)
    e1, p1 = [f.clone() for f in eta], [f.clone() for f in phi]
    (fe, e2), (fp, p2) = pieces(eta), pieces(phi)
    for call in range(3):
        b.step(e1, p1, 0.05, 1, tol=1e-9)
        b.step(e2, p2, 0.05, 1, tol=1e-9)
        for x, y in zip(e1 + p1, e2 + p2):
            assert torch.equal(x, y), call
    assert not torch.equal(e1[0], eta[0])
    for flat, fields in ((fe, e2), (fp, p2)):
        gaps = np.cumsum([0] + [f.numel() + 1 for f in fields])
        assert (flat[torch.tensor(gaps, device=gpu)] == 7.0).all()

    # members 1 and 2 share their tensors (and bed): the same as member 1 alone
    e3, p3 = [f.clone() for f in eta], [f.clone() for f in phi]
    e4, p4 = [f.clone() for f in eta], [f.clone() for f in phi]
    e4[2], p4[2] = e4[1], p4[1]
    b.step(e3, p3, 0.05, 1, tol=1e-9)
    b.step(e4, p4, 0.05, 1, tol=1e-9)
    for k in range(133):
        if k != 2:
            assert torch.equal(e3[k], e4[k]) and torch.equal(p3[k], p4[k]), k
