"""64 small solves on buffers where one solve's field lies on the next one's
masses: the first launch takes 40 of them (five passes, which read every mass
before they write a field), and each of those 40 results against the oracle's
convolution; the masses of the others were written by that launch.

Bars as in test_gpu_parity: 1e-11 (FP64) and 3e-6 (FP32) of max|Phi|."""
import numpy as np
import pytest

from oracle import pm_oracle as O
from tests import common as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("N", [8, 16])
def test_first_launch_of_shifted_solves(sbx, prec, N):
    import torch
    dt = torch.float64 if prec == sbx.SBX_FP64 else torch.float32
    b, first = 64, 40
    rng = np.random.default_rng(np.random.SeedSequence([1210, 1736, 988, N]))
    M = T.rounded(rng.uniform(0.0, 1.0, (b, N, N, N)) ** 3, prec)
    p = sbx.Poisson(N, 2.0, 0.5, G=0.7, prec=prec, stream=torch.cuda.current_stream().cuda_stream)
    buf = torch.zeros((b + 1, N, N, N), dtype=dt, device="cuda")
    buf[:b].copy_(torch.tensor(M, dtype=dt))
    torch.cuda.synchronize()
    p.sbx_poisson_solve(b, buf[:b].data_ptr(), buf[1:].data_ptr())
    torch.cuda.synchronize()
    got = buf[1:].double().cpu().numpy()
    p.close()
    Hh, _ = O.green_hat(O.Level(N, 2.0, 0.5))
    tol = 1e-11 if prec == sbx.SBX_FP64 else 3e-6
    for k in range(first):
        ref = O.solve_fft(M[k].transpose(2, 1, 0), Hh, G=0.7).transpose(2, 1, 0)
        assert np.abs(got[k] - ref).max() <= tol * np.abs(ref).max(), k
