"""What a segment holds: the work buffer that ckpt_every sizes, and records of
earlier cycles within the limit of sbx_set_segment_keep (2^30 bytes at first);
the gradients are those of a call that keeps one interval of all cycles (bars
as in test_gpu_adjoint; the two differ by the order of the cell sums)."""
import time

import pytest

from tests import common as T
from tests.test_gpu_adjoint import _maxrel, _workload

pytestmark = pytest.mark.gpu
MB = 1 << 20


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


def _free_memory():
    import torch
    time.sleep(0.2)  # the driver counts freed memory a little later
    return torch.cuda.mem_get_info()[0]


def _ctx(sbx, prec, N, w):
    ctx = sbx.Context(prec=prec, G=w.G)
    ctx.sbx_build_grids([sbx.make_hierarchy([(N, w.hier[0].levels[0].R, 1.0)])])
    ctx.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
    ctx.sbx_adjoint_segment(1e-3, 1, 1, 1, 0)  # the adjoint grids and their plan
    return ctx


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("ckpt", [1, 3])
@pytest.mark.parametrize("records", [0, 4, 20])
def test_limit_holds(sbx, prec, ckpt, records):
    w = _workload("single", n=3000, seed=4)
    N, steps = 128, 20
    f64 = prec == sbx.SBX_FP64
    record = N ** 3 * (8 if f64 else 4) + 3000 * (25 if f64 else 13) + (8 << 10)
    ctx = _ctx(sbx, prec, N, w)
    ctx.sbx_set_segment_keep(records * record)
    free = _free_memory()
    out = [ctx.sbx_adjoint_segment(1e-3, steps, ckpt, 1, 0)]
    held = free - _free_memory()
    more = min(records // ckpt * ckpt, steps - ckpt)  # whole intervals beside the last
    assert more * (record - (8 << 10)) <= held + 4 * MB  # (a one-cycle work buffer was there)
    assert held <= (ckpt + more) * record + steps * 3000 * 49 + 16 * MB
    out.append(ctx.sbx_adjoint_segment(1e-3, steps, ckpt, 1, 0))  # again, in the buffers there are
    assert abs(free - _free_memory() - held) <= 4 * MB
    ctx.sbx_set_segment_keep(0)
    assert free - _free_memory() <= ckpt * record + steps * 3000 * 49 + 16 * MB
    ctx.close()
    ref = _ctx(sbx, prec, N, w)
    for la, *ga in out:
        lb, *gb = ref.sbx_adjoint_segment(1e-3, steps, steps, 1, 0)
        assert la == pytest.approx(lb, rel=1e-12 if f64 else 1e-6)
        for a, b, tol in zip(ga, gb, (1e-5, 1e-4, 1e-5)):
            assert _maxrel(a, b) < (1e-9 if f64 else 10 * tol)  # FP32: some cells differ after 40 cycles
    ref.close()


def test_records_go_with_the_particles(sbx):
    w = _workload("single", n=3000, seed=5)
    ctx = _ctx(sbx, sbx.SBX_FP32, 128, w)
    free = _free_memory()
    ctx.sbx_adjoint_segment(1e-3, 20, 1, 1, 0)
    assert free - _free_memory() > 150 * MB
    ctx.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
    assert free - _free_memory() < 16 * MB
    with pytest.raises(sbx.SbxError):
        ctx.sbx_set_segment_keep(-1)
    ctx.close()
