"""The loss of a segment on borrowed particles is summed in the caller's
order, whatever order the segment runs in: with the fixed-point mass
assignment and fixed centres (forces that do not depend on the order) it is
the same bit for bit with and without the sorted copy, and from run to run."""
import pytest

from tests import common as T
from tests.test_gpu_adjoint import _workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind,ckpt", [("single", 5), ("nested", 2)])
def test_loss_is_reproducible(sbx, prec, kind, ckpt):
    import torch
    pt = torch.float64 if prec == sbx.SBX_FP64 else torch.float32
    n = 20000
    w = _workload(kind, n=n, seed=6)
    losses, states = [], []
    for sort in (0, 4, 4):
        ctx = sbx.Context(prec=prec, G=w.G)
        ctx.sbx_build_grids([T.sbx_hier(h) for h in w.hier])
        ctx.sbx_set_deterministic_deposit(1)
        ctx.sbx_set_sort_interval(sort)
        st = [torch.tensor(w.x.T.copy(), dtype=pt, device="cuda"), torch.tensor(w.v.T.copy(), dtype=pt, device="cuda"),
              torch.tensor(w.m, dtype=pt, device="cuda"), torch.tensor(w.comp, device="cuda"),
              torch.tensor(w.gal, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")]
        gm, gx, gv = (torch.empty(s, dtype=torch.float64, device="cuda") for s in ((n,), (n, 3), (n, 3)))
        torch.cuda.synchronize()
        ctx.sbx_bind_device_particles(n, *(t.data_ptr() for t in st))
        losses.append(ctx.sbx_adjoint_segment_device(w.dt, w.steps, ckpt, 1, 0, gm.data_ptr(), gx.data_ptr(),
                                                     gv.data_ptr()))
        ctx.close()
        states.append([t.cpu() for t in st])
    assert losses[0] == losses[1] == losses[2]
    for s in states[1:]:
        assert all(bool((a == b).all()) for a, b in zip(states[0], s))
