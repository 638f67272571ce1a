"""The radial order of the disc diagnostics where it can go wrong: particles
crowded into one radial bucket (more than 768: the radix sort), buckets of
768 and 769, equal radii (ties in the caller's order), the centre itself,
radii beyond the bucketed octaves, one particle; in the caller's order and
reordered, against the oracle.

Bars as in test_gpu_disc (sums in another order): 1e-10 relative, and for
the dispersions 1e-10 of the rms speed; counts exact."""
import numpy as np
import pytest

import synth
from oracle import pm_oracle as O
from tests import common as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


def _cloud(kind, n, rng):
    ph = rng.uniform(0, 2 * np.pi, n)
    R = {"exp": lambda: rng.exponential(0.6, n), "ring": lambda: 2.0 + 1e-7 * rng.normal(size=n),
         "wide": lambda: 10.0 ** rng.uniform(-9, 0.4, n), "edge": lambda: np.full(n, 1.5),
         "one": lambda: np.full(n, 0.7), "centre": lambda: rng.exponential(0.6, n)}[kind]()
    R = np.minimum(R, 3.0)
    x = np.stack([R * np.cos(ph), R * np.sin(ph), 0.2 * rng.normal(size=n).clip(-3, 3)], 1)
    if kind == "centre":
        x[::3, :2] = 0.0
    if kind == "edge":  # equal radii exactly: multiples of the quarter turn
        q = rng.integers(0, 4, n)
        x[:, 0], x[:, 1] = 1.5 * (q == 0) - 1.5 * (q == 2), 1.5 * (q == 1) - 1.5 * (q == 3)
    return x


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kind,n", [("exp", 20000), ("ring", 5000), ("wide", 3001), ("edge", 768),
                                    ("edge", 769), ("edge", 1025), ("one", 1), ("centre", 4000)])
def test_radial_order(sbx, prec, kind, n):
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 982, n]))
    x = np.concatenate([_cloud(kind, n, rng), rng.uniform(-2, 2, (777, 3))])
    keep = rng.permutation(n + 777)
    comp = np.concatenate([np.zeros(n, np.int8), np.ones(777, np.int8)])[keep]
    x = x[keep]
    v = rng.normal(size=x.shape)
    m = rng.uniform(0.5, 1.5, n + 777) / n
    w = synth.Workload("order", x, v, m, comp, np.zeros(n + 777, np.int8),
                       [synth.HierSpec([synth.LevelSpec(16, 4.0, 1.0)])], 0.01, 1)
    ctx = T.make_ctx(w, prec)
    xr, vr, mr = T.oracle_inputs(w, prec)
    lost = np.zeros(n + 777, bool)
    nb = min(17, n)
    for _ in range(2):  # the caller's order, then cell order
        got = ctx.sbx_disc_analysis(nb, (0.5, 2.5), 12, 0.5)
        ref = O.disc_analysis(xr, vr, mr, comp, w.gal, lost, (0, 0, 0), nb, (0.5, 2.5), 12, 0.5)
        assert got["n_disc"] == n and got["n_annulus"] == ref["n_annulus"]
        for k in ("bin_r", "bin_vc", "bin_rms_z"):
            assert np.allclose(got[k], ref[k], rtol=1e-10, atol=1e-12), k
        if kind != "edge":  # bins of one radius: the interpolation between them is undefined
            assert got["e_heat"] == pytest.approx(ref["e_heat"], rel=1e-10)
        for k in ("sig_R", "sig_phi", "sig_z"):
            assert got[k] == pytest.approx(ref[k], rel=1e-10, abs=1e-7), k
        assert np.abs(got["rho_z"] - ref["rho_z"]).max() <= 1e-10 * max(ref["rho_z"].max(), 1e-300)
        for mm in (0, 3, 16):
            a = ctx.sbx_disc_modes(9, 3.5, mm)
            b = O.disc_modes(xr, mr, comp, w.gal, lost, (0, 0, 0), 9, 3.5, mm)
            assert np.abs(a - b).max() <= 1e-10 * np.abs(b[:, 0]).max()
        ctx.sbx_step(0.0, 1)
    ctx.close()


def test_work_buffer_grows_between_calls(sbx):
    """Calls of growing and shrinking needs on one context: each prepares its
    disc anew, in a new work buffer where the old one was too small (which may
    lie where the old one did)."""
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 983]))
    n = 30000
    x = _cloud("exp", n, rng)
    v, m, comp = rng.normal(size=x.shape), np.full(n, 1.0 / n), np.zeros(n, np.int8)
    w = synth.Workload("grow", x, v, m, comp, comp, [synth.HierSpec([synth.LevelSpec(16, 4.0, 1.0)])], 0.01, 1)
    ctx = T.make_ctx(w, sbx.SBX_FP64)
    ctx.sbx_step(0.0, 1)
    lost = np.zeros(n, bool)
    for nr, mm, nb in ((3, 1, 3), (64, 4, 100), (2000, 16, 2000), (10, 2, 10)):
        a = ctx.sbx_disc_modes(nr, 3.5, mm)
        b = O.disc_modes(x, m, comp, w.gal, lost, (0, 0, 0), nr, 3.5, mm)
        assert np.abs(a - b).max() <= 1e-10 * np.abs(b[:, 0]).max()
        got = ctx.sbx_disc_analysis(nb, (0.5, 2.5), 12, 0.5)
        ref = O.disc_analysis(x, v, m, comp, w.gal, lost, (0, 0, 0), nb, (0.5, 2.5), 12, 0.5)
        assert np.allclose(got["bin_r"], ref["bin_r"], rtol=1e-10)
        assert got["e_heat"] == pytest.approx(ref["e_heat"], rel=1e-10)
    ctx.close()
