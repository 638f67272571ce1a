"""Solves of 8^3 and 16^3 grids, a block per solve in one launch: batches up
to the limits of one launch and past them, in place, on buffers where one
solve's field lies on another's masses (which take the five passes), without
allocation, and pinned to five passes, against the oracle's convolution;
contexts on such grids against its forces.

Bars as in test_gpu_parity: 1e-11 (FP64) and 3e-6 (FP32) of max|Phi|; forces
within 1e-9 of the rms force."""
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


def _grids(N, b, prec):
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 984, N, b]))
    return T.rounded(rng.uniform(0.0, 1.0, (b, N, N, N)) ** 3, prec)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("N", [8, 16])
@pytest.mark.parametrize("b", [1, 5, 40, 64])
@pytest.mark.parametrize("how", ["apart", "in place", "shifted", "noalloc", "five"])
def test_small_solves(sbx, prec, N, b, how):
    import torch
    dt = torch.float64 if prec == sbx.SBX_FP64 else torch.float32
    M = _grids(N, b, prec)
    if how == "five":
        sbx.sbx_set_fft_form(5)
    try:
        p = sbx.Poisson(N, 2.0, 0.5, G=0.7, prec=prec, stream=torch.cuda.current_stream().cuda_stream)
        buf = torch.zeros((b + 1, N, N, N), dtype=dt, device="cuda")
        rho = buf[:b]
        rho.copy_(torch.tensor(M, dtype=dt))
        phi = {"in place": rho, "shifted": buf[1:]}.get(how, torch.empty_like(rho))
        torch.cuda.synchronize()
        solve = p.sbx_poisson_solve_noalloc if how == "noalloc" else p.sbx_poisson_solve
        solve(b, rho.data_ptr(), phi.data_ptr())
        torch.cuda.synchronize()
    finally:
        sbx.sbx_set_fft_form(0)
    got = phi.double().cpu().numpy()
    p.close()
    Hh, _ = O.green_hat(O.Level(N, 2.0, 0.5))
    tol = 1e-11 if prec == sbx.SBX_FP64 else 3e-6
    for m, g in zip(M, got):
        ref = O.solve_fft(m.transpose(2, 1, 0), Hh, G=0.7).transpose(2, 1, 0)
        assert np.abs(g - ref).max() <= tol * np.abs(ref).max()
        if how == "shifted" and b > 40:
            break  # the second launch of 40 reads what the first one wrote, as ever


@pytest.mark.parametrize("levels", [1, 3])
def test_context_on_16_cells(sbx, levels):
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 985]))
    n = 3000
    x = rng.normal(size=(n, 3)) * 0.5
    lv = [synth.LevelSpec(16, 3.0, 1.0)] if levels == 1 else \
        [synth.LevelSpec(16, 0.6, 1.0), synth.LevelSpec(16, 1.5, 1.0), synth.LevelSpec(16, 3.0, 1.0)]
    w = synth.Workload("n16", x, np.zeros_like(x), np.full(n, 1.0 / n), np.zeros(n, np.int8),
                       np.zeros(n, np.int8), [synth.HierSpec(lv)], 0.01, 1)
    sysm = T.oracle_system(w)
    ref = sysm.accel(x, w.m, w.gal, sysm.lost_now(x))
    ctx = T.make_ctx(w, sbx.SBX_FP64)
    acc, _ = ctx.sbx_compute_forces()
    assert T.rel_err_vec(acc, ref).max() < 1e-9
    ctx.close()
