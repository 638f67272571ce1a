"""Steps are stream-ordered: the first reorder after a load, which takes its
own route, returns while earlier work of the stream still runs, and a step
that holds it can be captured; the states against a context that steps
eagerly on a stream of its own.

Positions within 1e-12 (FP64, eight steps) and 1e-5 (FP32, one step: an ulp
below 32 is 1.9e-6 and dt^2 is 1e-4), for |x| < 20; the two differ by the
order of the cell and centre-of-mass sums)."""
import numpy as np
import pytest

from tests import common as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


def _ctx(sbx, w, prec, stream=None):
    c = sbx.Context(prec=prec, G=w.G, stream=stream)
    c.sbx_build_grids([T.sbx_hier(h) for h in w.hier])
    c.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
    c.sbx_step(w.dt, 0)  # dt reaches the device
    return c


@pytest.mark.parametrize("prec", [0, 1])
def test_first_reorder_does_not_wait(sbx, prec):
    import torch
    w = T.small_galaxy(scale=0.002, N=32, q=1.0)
    warm = _ctx(sbx, w, prec)
    warm.sbx_step(w.dt, 1)
    warm.sbx_sync()
    s = torch.cuda.Stream()
    c = _ctx(sbx, w, prec, s.cuda_stream)
    a = torch.randn(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(s):
        for _ in range(60):  # some 0.4 s
            torch.mm(a, a, out=b)
        done.record()
    c.sbx_step(w.dt, 1)
    assert not done.query()
    c.sbx_sync()
    x, v, _ = c.sbx_get_particles()
    xr, vr, _ = warm.sbx_get_particles()
    tol = 1e-12 if prec == sbx.SBX_FP64 else 1e-5
    assert np.abs(x - xr).max() <= tol
    c.close()
    warm.close()


def test_captured_steps_hold_the_first_reorder(sbx):
    import torch
    w = T.small_galaxy(scale=0.002, N=32, q=1.0)
    ref = _ctx(sbx, w, sbx.SBX_FP64)
    ref.sbx_set_sort_interval(1)
    s = torch.cuda.Stream()
    c = _ctx(sbx, w, sbx.SBX_FP64, s.cuda_stream)
    c.sbx_set_sort_interval(1)
    ref.sbx_step(w.dt, 0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.sbx_step(w.dt, 2)  # two reorders: the live set ends where it was
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        ref.sbx_step(w.dt, 2)
        x, _, lost = c.sbx_get_particles()
        xr, _, lr = ref.sbx_get_particles()
        assert np.array_equal(lost, lr)
        assert np.abs(x - xr).max() <= 1e-12
    c.sbx_step(w.dt, 2)  # and on without the graph
    ref.sbx_step(w.dt, 2)
    assert np.abs(c.sbx_get_particles()[0] - ref.sbx_get_particles()[0]).max() <= 1e-12
    c.close()
    ref.close()
