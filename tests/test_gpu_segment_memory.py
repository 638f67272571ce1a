"""What a segment holds: a call whose earlier cycles' records fit beside the
last interval's gives them back, so that ckpt_every bounds what the context
keeps; the gradients are those of a call that keeps one interval of all cycles
(bars as in test_gpu_adjoint; the two differ by the order of the cell sums)."""
import time

import pytest

from tests import common as T
from tests.test_gpu_adjoint import _maxrel, _workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("ckpt", [1, 3])
def test_records_are_given_back(sbx, prec, ckpt):
    import torch

    def free_memory():
        time.sleep(0.2)  # the driver counts freed memory a little later
        return torch.cuda.mem_get_info()[0]

    w = _workload("single", n=3000, seed=4)
    N, steps = 128, 20
    record = N ** 3 * (8 if prec == sbx.SBX_FP64 else 4)
    out, held = [], []
    for every in (ckpt, steps):
        ctx = sbx.Context(prec=prec, G=w.G)
        ctx.sbx_build_grids([sbx.make_hierarchy([(N, w.hier[0].levels[0].R, 1.0)])])
        ctx.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
        ctx.sbx_adjoint_segment(1e-3, 1, 1, 1, 0)  # the adjoint grids and their plan
        free = free_memory()
        out.append(ctx.sbx_adjoint_segment(1e-3, steps, every, 1, 0))
        held.append(free - free_memory())
        out.append(ctx.sbx_adjoint_segment(1e-3, steps, every, 1, 0))  # and again, in the kept buffer
        ctx.close()
    assert held[0] < (ckpt + 2) * record + (16 << 20)
    assert held[1] > (steps - 2) * record  # what the caller asked to hold
    f64 = prec == sbx.SBX_FP64
    for (la, *ga), (lb, *gb) in (out[::2], out[1::2]):
        assert la == pytest.approx(lb, rel=1e-12 if f64 else 1e-6)
        for a, b, tol in zip(ga, gb, (1e-5, 1e-4, 1e-5)):
            assert _maxrel(a, b) < (1e-9 if f64 else 10 * tol)  # FP32: some cells differ after 40 cycles


@pytest.mark.parametrize("prec", [0, 1])
def test_few_records_stay_and_go_with_the_particles(sbx, prec):
    """Up to 128 MiB of further records stay with the context, for segments
    that need as many or fewer, until the particles are replaced."""
    import torch
    w = _workload("single", n=3000, seed=5)
    ctx = sbx.Context(prec=prec, G=w.G)
    ctx.sbx_build_grids([sbx.make_hierarchy([(64, w.hier[0].levels[0].R, 1.0)])])
    ctx.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
    ctx.sbx_adjoint_segment(1e-3, 1, 1, 1, 0)
    time.sleep(0.2)
    free, held = torch.cuda.mem_get_info()[0], []
    for steps, every in ((20, 1), (20, 1), (7, 2), (20, 1)):
        ctx.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal) if steps == 7 else None
        ctx.sbx_adjoint_segment(1e-3, steps, every, 1, 0)
        time.sleep(0.2)
        held.append(free - torch.cuda.mem_get_info()[0])
    record = 64 ** 3 * (8 if prec == sbx.SBX_FP64 else 4)
    assert 15 * record < held[0] < 26 * record + (16 << 20)
    assert held[1] == held[0] == held[3] and held[2] < held[0]
    ctx.close()
