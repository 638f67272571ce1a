"""The disc selection where the last wavefront of the reordered particles is
not full and holds consecutive numbers from a multiple of 64 (a single one, in
the smallest case), the other numbers of those 64 lying in other wavefronts:
such particles share their words of the selection with them.  Against the
oracle, in the caller's order and reordered, with bars as in test_gpu_disc
(sums in another order): 1e-10 relative; counts exact."""
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


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,first,tail", [(65, 0, 1), (129, 64, 1), (129, 0, 1), (1025, 512, 1), (4097, 0, 1),
                                          (98, 0, 34), (66, 0, 2), (127, 0, 63), (160, 64, 32), (161, 128, 33)])
def test_tail_wavefront(sbx, prec, n, first, tail):
    """`tail` = n mod 64 particles from number `first` on lie one by one in the
    last cells of the order (cells are ordered by z, then y, then x; the cell
    length is 2/3), all others below them, and all within the grid's R = 4."""
    assert tail == n % 64
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 986, n, first]))
    x = np.stack([rng.uniform(-2, 2, n), rng.uniform(-2, 2, n), rng.uniform(-2, 0.8, n)], 1)
    k = np.arange(tail)
    x[first:first + tail] = np.stack([2 / 3 * (k % 8 - 4), 2 / 3 * (k // 8 - 4), np.full(tail, 1.35)], 1) + 0.05
    v = rng.normal(size=x.shape)
    m = rng.uniform(0.5, 1.5, n) / n
    comp = np.zeros(n, np.int8)
    w = synth.Workload("tail", x, v, m, comp, comp, [synth.HierSpec([synth.LevelSpec(16, 4.0, 1.0)])], 0.01, 1)
    ctx = T.make_ctx(w, prec)
    xr, vr, mr = T.oracle_inputs(w, prec)
    lost = np.zeros(n, bool)
    for _ in range(2):  # the caller's order, then cell order
        got = ctx.sbx_disc_analysis(5, (0.5, 2.5), 12, 3.0)
        ref = O.disc_analysis(xr, vr, mr, comp, comp, lost, (0, 0, 0), 5, (0.5, 2.5), 12, 3.0)
        assert got["n_disc"] == n and got["n_annulus"] == ref["n_annulus"]
        for q in ("bin_r", "bin_vc", "bin_rms_z"):
            assert np.allclose(got[q], ref[q], rtol=1e-10, atol=1e-12), q
        assert got["e_heat"] == pytest.approx(ref["e_heat"], rel=1e-10)
        a = ctx.sbx_disc_modes(9, 4.5, 3)
        b = O.disc_modes(xr, mr, comp, comp, lost, (0, 0, 0), 9, 4.5, 3)
        assert np.abs(a - b).max() <= 1e-10 * np.abs(b[:, 0]).max()
        ctx.sbx_step(0.0, 1)
    ctx.close()
