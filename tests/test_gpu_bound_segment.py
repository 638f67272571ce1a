"""Differentiable segments on borrowed storage, which run as a cell-sorted
copy: gradients and final state in the caller's order against the oracle, with
and without the sort, rebinding the same and another number of particles, and
particles that leave the grid.

Bars as in test_gpu_adjoint: FP64 gradients within 1e-9 of their largest
magnitude, FP32 within 1e-5 (m, v) and 1e-4 (x); final positions within
1e-13 (FP64) and 1e-6 (FP32: one rounding of |x| < 3 per cycle, five
cycles)."""
import numpy as np
import pytest

from oracle import pm_oracle as O
from tests import common as T
from tests.test_gpu_adjoint import _maxrel, _workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind,ckpt,sort", [("single", 2, 4), ("single", 5, 4), ("nested", 1, 4),
                                            ("nested", 2, 0)])
def test_bound_segment(sbx, prec, kind, ckpt, sort):
    import torch
    pt = torch.float64 if prec == sbx.SBX_FP64 else torch.float32
    ctx = None
    for n, seed in ((3000, 1), (3000, 2), (517, 3)):
        w = _workload(kind, n=n, seed=seed)
        w.x[:3] = [[2.2, 0.1, 0.0], [0.0, -2.2, 0.0], [40.0, 0.0, 0.0]]
        w.v[:2] = [[9.0, 0.0, 0.0], [0.0, -9.0, 0.0]]  # off the single grid on the way
        x, v, m = T.oracle_inputs(w, prec)
        if ctx is None:
            ctx = sbx.Context(prec=prec, G=w.G)
            ctx.sbx_build_grids([T.sbx_hier(h) for h in w.hier])
            ctx.sbx_set_sort_interval(sort)
        st = [torch.tensor(x.T.copy(), dtype=pt, device="cuda"), torch.tensor(v.T.copy(), dtype=pt, device="cuda"),
              torch.tensor(m, dtype=pt, device="cuda"), torch.tensor(w.comp, device="cuda"),
              torch.tensor(w.gal, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")]
        kept = [t.clone() for t in st[2:5]]
        gm, gx, gv = (torch.empty(s, dtype=torch.float64, device="cuda") for s in ((n,), (n, 3), (n, 3)))
        torch.cuda.synchronize()
        ctx.sbx_bind_device_particles(n, *(t.data_ptr() for t in st))
        L = ctx.sbx_adjoint_segment_device(w.dt, w.steps, ckpt, 1, 0, gm.data_ptr(), gx.data_ptr(), gv.data_ptr())
        sysm = T.oracle_system(w)
        Lr, gmr, gxr, gvr = O.segment_loss_and_grads(sysm, x, v, m, w.comp, w.gal, w.dt, w.steps, 1, 0)
        f64 = prec == sbx.SBX_FP64
        assert L == pytest.approx(Lr, rel=1e-12 if f64 else 1e-6)
        for a, b, tol in ((gm, gmr, 1e-5), (gv, gvr, 1e-5), (gx, gxr, 1e-4)):
            assert _maxrel(a.cpu().numpy(), b) < (1e-9 if f64 else tol)
        xr, vr, lr = x, v, np.zeros(n, bool)
        for _ in range(w.steps):
            xr, vr, lr, _ = sysm.step(xr, vr, m, w.gal, lr, w.dt)
        assert lr.any()
        assert np.array_equal(st[5].cpu().numpy().astype(bool), lr)
        assert np.abs(st[0].cpu().numpy().T - xr).max() < (1e-13 if f64 else 1e-6) * 50  # |x| up to 40
        assert all(bool((a == b).all()) for a, b in zip(st[2:5], kept))
        # the context steps on from the borrowed storage
        ctx.sbx_step(w.dt, 1)
        xg, _, _ = ctx.sbx_get_particles()
        assert np.array_equal(st[0].double().cpu().numpy().T, xg)
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_records_beyond_the_kept_ones(sbx, prec):
    """A segment whose records do not all fit in 4 GiB (128^3 cells on three
    levels, 7 x 2^21 values a record): intervals kept from the forward and
    intervals recomputed, several of each, against one that keeps every cycle
    of one interval.  The two run the same cycles and differ by the order of
    the cell sums: the bars of the segment."""
    w = _workload("nested", n=4000, seed=5)
    steps = 80 if prec == sbx.SBX_FP32 else 44  # 58.7 or 117.4 MB a record: 73 or 36 cycles fit
    out = []
    for ckpt in (8, steps):
        ctx = sbx.Context(prec=prec, G=w.G)
        ctx.sbx_build_grids([sbx.make_hierarchy([(128, l.R, l.q) for l in w.hier[0].levels])])
        ctx.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
        out.append((ctx.sbx_adjoint_segment(1e-3, steps, ckpt, 1, 0), ctx.sbx_get_particles()))
        ctx.close()
    (la, gma, gxa, gva), sa = out[0]
    (lb, gmb, gxb, gvb), sb = out[1]
    f64 = prec == sbx.SBX_FP64
    assert la == pytest.approx(lb, rel=1e-12 if f64 else 1e-6)
    for a, b, tol in ((gma, gmb, 1e-5), (gva, gvb, 1e-5), (gxa, gxb, 1e-4)):
        assert _maxrel(a, b) < (1e-9 if f64 else 10 * tol)  # FP32: some cells differ after 80 cycles
    assert np.abs(sa[0] - sb[0]).max() < (1e-12 if f64 else 1e-5)
