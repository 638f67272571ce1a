"""Host outputs change only when the results arrive: while the stream still
has earlier work to do, the arrays that a waiting call was given are as the
caller left them (a call that fails then leaves them so)."""
import threading
import time

import numpy as np
import pytest

from tests import common as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sbx():
    from paper_1210_1736_amd import sbx as m
    return m


@pytest.mark.parametrize("what", ["forces", "particles"])
def test_outputs_untouched_while_the_call_waits(sbx, what):
    import torch
    w = T.small_galaxy(scale=0.002, N=32, q=1.0)
    s = torch.cuda.Stream()
    c = sbx.Context(prec=sbx.SBX_FP64, G=w.G, stream=s.cuda_stream)
    c.sbx_build_grids([T.sbx_hier(h) for h in w.hier])
    c.sbx_load_particles(w.x, w.v, w.m, w.comp, w.gal)
    n, lib = c.n, sbx.lib()
    acc, pot = c.sbx_compute_forces()
    x, v, _ = c.sbx_get_particles()
    a, b = np.full((n, 3), 0.1), np.full(n if what == "forces" else 3 * n, 0.1)
    pa, pb = a.ctypes.data, b.ctypes.data
    mat = torch.randn(8192, 8192, device="cuda")
    out = torch.empty_like(mat)
    torch.mm(mat, mat, out=out)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(s):
        for _ in range(80):  # some 0.5 s
            torch.mm(mat, mat, out=out)
        done.record()
    rc = []
    call = (lambda: rc.append(lib.sbx_compute_forces(c._h, pa, pb))) if what == "forces" else \
        (lambda: rc.append(lib.sbx_get_particles(c._h, pa, pb, None)))
    t = threading.Thread(target=call)
    t.start()
    time.sleep(0.15)
    still, waiting = bool((a == 0.1).all() and (b == 0.1).all()), not done.query()
    t.join()
    assert waiting and still
    assert rc == [sbx.SBX_OK]
    if what == "forces":
        assert T.rel_err_vec(a, acc).max() < 1e-9 and np.abs(b - pot).max() < 1e-9 * np.abs(pot).max()
    else:
        assert np.array_equal(a, x) and np.array_equal(b.reshape(n, 3), v)
    c.close()
