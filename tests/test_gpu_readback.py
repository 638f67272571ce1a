"""Device and host read-back of a reordered context in the caller's order, on
both sides of the particle counts where the staged form takes over (2^19 in
FP32, 3 * 2^20 in FP64) and with outputs left out.  The particles have not
moved (a step of no length, lost ones off the grid), so every value is exact:
bit equality."""
import numpy as np
import pytest

from tests import common as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


@pytest.mark.parametrize("prec,n", [(0, 1), (0, 259), (0, 2 ** 19 - 1), (0, 2 ** 19), (0, 2 ** 19 + 77),
                                    (1, 1), (1, 2 ** 19), (1, 3 * 2 ** 20 - 1), (1, 3 * 2 ** 20 + 5)])
def test_readback_in_callers_order(sbx, prec, n):
    import torch
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 981, n]))
    x = T.rounded(rng.uniform(-1.05, 1.05, (n, 3)), prec)  # grid of half-extent 1: some are lost
    v = T.rounded(rng.normal(size=(n, 3)), prec)
    ctx = sbx.Context(prec=prec)
    ctx.sbx_build_grids([sbx.make_hierarchy([(16, 1.0, 1.0)])])
    ctx.sbx_load_particles(x, v, np.full(n, 1.0 / n), np.zeros(n, np.int8), np.zeros(n, np.int8))
    ctx.sbx_step(0.0, 1)
    xh, vh, lh = ctx.sbx_get_particles()
    assert np.array_equal(xh, x) and np.array_equal(vh, v)
    cell = np.floor(x * 6.0 + 8.0 + 0.5)   # gamma = (16 - 4) / 2
    assert np.array_equal(lh, ((cell < 2) | (cell > 13)).any(axis=1))
    new = lambda *s: torch.full(s, -7.0, dtype=torch.float64, device="cuda")
    for wx, wv, wl in ((1, 1, 1), (1, 0, 0), (0, 1, 1), (0, 0, 1)):
        xd, vd = new(n, 3), new(n, 3)
        ld = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        ctx.sbx_get_particles_device(xd.data_ptr() if wx else None, vd.data_ptr() if wv else None,
                                     ld.data_ptr() if wl else None)
        same = lambda t, a, w, blank: bool(np.array_equal(t.cpu().numpy(), a) if w else (t == blank).all())
        assert same(xd, xh, wx, -7.0) and same(vd, vh, wv, -7.0) and same(ld, lh.astype(np.uint8), wl, 9)
    ctx.sbx_step(0.0, 1)  # the staging left the live set alone
    assert np.array_equal(ctx.sbx_get_particles()[0], x)
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [1, 300, 40001])
def test_forces_in_callers_order(sbx, prec, n):
    """Accelerations and potentials of a reordered context against the same
    context before the reorder: the same particles at the same rows, to the
    rounding of the cell sums (as the float and fixed-point assignments
    agree: 1e-10 FP64, 1e-4 FP32 of the rms); lost particles zero."""
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 986, n]))
    x = rng.uniform(-1.05, 1.05, (n, 3))
    x[0] = 0.1
    ctx = sbx.Context(prec=prec)
    ctx.sbx_build_grids([sbx.make_hierarchy([(16, 1.0, 1.0)])])
    ctx.sbx_load_particles(x, np.zeros_like(x), np.full(n, 1.0 / n), np.zeros(n, np.int8), np.zeros(n, np.int8))
    a0, p0 = ctx.sbx_compute_forces()
    ctx.sbx_step(0.0, 1)
    a1, p1 = ctx.sbx_compute_forces()
    lost = ctx.sbx_get_particles()[2]
    tol = 1e-10 if prec == sbx.SBX_FP64 else 1e-4
    scale = max(np.sqrt(np.mean(a0 * a0)), np.abs(p0).max() * 1e-3)
    assert np.abs(a1 - a0).max() <= tol * scale and np.abs(p1 - p0).max() <= tol * np.abs(p0).max()
    assert not a1[lost].any() and not p1[lost].any() and (p1[~lost] < 0).all()
    ctx.close()


@pytest.mark.parametrize("prec,n", [(0, 2 ** 25), (0, 2 ** 25 + 1), (1, 2 ** 20 + 1)])
def test_first_reorder_keeps_every_particle(sbx, prec, n):
    """The first reorder of particles in no order (through records up to 2^25
    particles in FP32, by gathering above) and the ones after it: every value,
    component, galaxy and flag still with its particle."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(1736 + n)
    x = (torch.rand((n, 3), generator=g, device="cuda") * 2.1 - 1.05).double()
    v = torch.rand((n, 3), generator=g, device="cuda").double()
    m = torch.rand(n, generator=g, device="cuda").double() / n
    comp = torch.randint(0, 8, (n,), generator=g, device="cuda", dtype=torch.int8)
    gal = torch.zeros(n, device="cuda", dtype=torch.int8)
    ctx = sbx.Context(prec=prec)
    ctx.sbx_build_grids([sbx.make_hierarchy([(32, 1.0, 1.0)])])
    torch.cuda.synchronize()
    ctx.sbx_load_particles_device(n, x.data_ptr(), v.data_ptr(), m.data_ptr(), comp.data_ptr(), gal.data_ptr())
    ctx.sbx_set_sort_interval(1)
    xo, vo, lo = torch.empty_like(x), torch.empty_like(v), torch.empty(n, device="cuda", dtype=torch.uint8)
    cell = torch.floor(x * 14.0 + 16.5)
    lost = ((cell < 2) | (cell > 29)).any(1)
    for _ in range(2):
        ctx.sbx_step(0.0, 1, 1)
        ctx.sbx_get_particles_device(xo.data_ptr(), vo.data_ptr(), lo.data_ptr())
        assert bool((xo == x).all()) and bool((vo == v).all()) and bool((lo.bool() == lost).all())
    d = ctx.sbx_diag_log()[-1]
    live = ~lost
    for c in range(8):
        sel = live & (comp == c)
        assert d["n_live"][c] == int(sel.sum())
        ek = float((0.5 * m * (v * v).sum(1))[sel].sum())
        assert d["ekin"][c] == pytest.approx(ek, rel=1e-6)  # v_sync of a step of no length is v
    ctx.close()
