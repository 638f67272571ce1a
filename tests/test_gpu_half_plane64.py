"""The forward plane pass at N = 64 in half-plane blocks (256 threads per
plane, as two blocks): both parities of kx, column 0 with the mirrored
spectrum of its own, one solve and an odd number of them, against the
oracle's FFT convolution (Eqs. 3-5)."""
import numpy as np
import pytest

from oracle import pm_oracle as O
from tests import common as T
from tests.test_gpu_parity import _solve_gpu, sbx, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("count", [1, 3])
def test_half_plane_forward_matches_oracle(sbx, torch, prec, count):  # noqa: F811
    N, R, q = 64, 1.5, 0.5
    rng = np.random.default_rng(640 + 2 * count + prec)
    Ms = []
    for b in range(count):
        M = np.zeros((N, N, N))
        cells = rng.integers(0, N, size=(N * N // (2 + b), 3))
        np.add.at(M, tuple(cells.T), rng.uniform(0.1, 1.0, cells.shape[0]))
        M[0, 0, 0] += 3.0  # the first row pair, column and plane,
        M[N - 1, N - 1, N - 1] += 2.0  # and the last
        Ms.append(T.rounded(M, prec))
    sbx.sbx_set_fft_form(3)
    sbx.sbx_set_plane_threads(256)
    try:
        got = _solve_gpu(sbx, torch, N, R, q, Ms, prec, G=0.7)
    finally:
        sbx.sbx_set_fft_form(0)
        sbx.sbx_set_plane_threads(0)
    Hh, _ = O.green_hat(O.Level(N, R, q))
    # the bounds of the other plane-form tests: 64 bits, and ~25 float32 ulps
    tol = 1e-11 if prec == sbx.SBX_FP64 else 3e-6
    for M, g in zip(Ms, got):
        ref = O.solve_fft(M, Hh, G=0.7)
        assert np.max(np.abs(g - ref)) <= tol * np.max(np.abs(ref))
