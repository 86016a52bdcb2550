"""A step-size estimate whose launch gives up (a wait inside it ran out): no
iteration is made with the unfinished estimate.  With L scaled up the step
of an estimate that made no step (1) is far above 1/L_f, and a main phase run
with it would go on to its iteration cap (200000 steps, seconds); the solve
itself takes milliseconds.
"""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.reference import exact_mv_factor
from tests.gpu_util import banner
from tests.test_gpu_loop import _case, loop_wait

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


@pytest.mark.parametrize("n,T,path", [(300, 500, "syrk"), (700, 300, "gemv")])
def test_estimate_gives_up(npga, n, T, path):
    banner(f"unfinished estimate n={n} T={T} {path}")
    L, mu_d, mu, Lo, gamma, r = _case(npga, n, T, "f32")
    L, Lo, gamma = L * 1024.0, Lo * 1024.0, gamma * 1024.0 ** 2
    took = {}
    for us in (-1, 0):
        with loop_wait(us):
            npga.solve(L, mu_d, r, gamma=gamma, path=path, max_iter=5)  # (the kernels' first launches)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            x, info = npga.solve(L, mu_d, r, gamma=gamma, path=path)
            torch.cuda.synchronize()
            took[us] = time.perf_counter() - t0
        assert info["status"] == 0
        xh = x.cpu().numpy().astype(np.float64)
        assert np.abs(xh - exact_mv_factor(Lo, gamma, mu, r)["x"]).max() <= 1e-5
        assert info["time_ms"] <= 1e3 * took[us]
    assert took[0] <= 4.0 * took[-1] + 0.1, took
