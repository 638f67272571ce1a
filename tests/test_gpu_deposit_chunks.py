"""Cell masses where the mass assignment changes its particles per block
(256 up to 2^18 particles, 512 up to 2^19, ...) and at ragged last chunks,
against the oracle's fixed-point and float64 assignments.

Bars: the fixed-point form is bit-exact; the float form's cell masses are
sums of K terms of one sign, so each is within K eps of the oracle's, K at
most the cell's mass over the smallest particle mass."""
import dataclasses

import numpy as np
import pytest

from tests import common as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def workload():
    w = T.small_galaxy(scale=0.062, N=32, centring="fixed", q=1.0)
    assert w.n > 2 ** 19
    return w


@pytest.mark.parametrize("prec", [0, 1])  # SBX_FP32, SBX_FP64
@pytest.mark.parametrize("n", [1, 255, 257, 2 ** 18, 2 ** 18 + 1, 2 ** 19 + 3])
def test_cell_masses_at_chunk_edges(workload, prec, n):
    pick = np.random.default_rng(n).permutation(workload.n)[:n]
    w = dataclasses.replace(workload, x=workload.x[pick], v=workload.v[pick], m=workload.m[pick],
                            comp=workload.comp[pick], gal=workload.gal[pick])
    x, v, m = T.oracle_inputs(w, prec)
    sysm = T.oracle_system(w)
    lost = sysm.lost_now(x)
    cen = sysm.centres(x, m, w.gal, lost)
    refs = {}
    for fixed in (0, 1):
        sysm.fixed_deposit = bool(fixed)
        r = sysm.potentials(x, m, w.gal, lost, cen)[0]["M"]
        r = [T.rounded(a, prec) if fixed else a for a in r]
        refs[fixed] = [r[0], r[2], r[1] + r[2], r[4], r[3] + r[4]]
    ctx = T.make_ctx(w, prec)
    eps = 2.0 ** -52 if prec == 1 else 2.0 ** -23
    for fixed in (1, 0):
        ctx.sbx_set_deterministic_deposit(fixed)
        ctx.sbx_step(0.0, 1)  # positions kept; the particles in cell order
        for k, r in enumerate(refs[fixed]):
            g = ctx.sbx_get_grid(0, k, 0).transpose(2, 1, 0)
            if fixed:
                assert bool(np.array_equal(g, r)), k
            else:
                count = r / m[m > 0].min()
                ok = bool(np.all(np.abs(g - r) <= (count + 2) * eps * r))
                assert ok, k
    ctx.close()
