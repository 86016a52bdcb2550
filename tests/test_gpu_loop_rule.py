"""Where a solve's phases run as one launch: up to the sizes at which a step of
it takes no longer than one by launches (2048 assets on Sigma; on L 8192
columns up to 256 assets, 4096 up to 512, 1024 up to 1024).  Which way ran
shows in the gradient launches sampled; both give the same minimiser.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import banner
from tests.test_gpu_loop import _case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


@pytest.mark.parametrize("n,T,dtype,path,one", [
    (256, 8192, "f32", "gemv", True), (256, 8193, "f32", "gemv", False), (60, 8193, "bf16", "gemv", False),
    (257, 4096, "f32", "gemv", True), (512, 4097, "f32", "gemv", False), (400, 4100, "bf16", "gemv", False),
    (513, 1024, "bf16", "gemv", True), (513, 1025, "bf16", "gemv", False), (1024, 1025, "f32", "gemv", False),
    (1025, 1024, "f32", "gemv", False),
    (2048, 2100, "f32", "syrk", True), (2049, 2100, "f32", "syrk", False),
])
def test_one_launch_or_not(npga, n, T, dtype, path, one):
    banner(f"rule of the one-launch phases n={n} T={T} {dtype} {path}")
    L, mu_d, mu, Lo, gamma, r = _case(npga, n, T, dtype)
    x, info = npga.solve(L, mu_d, r, gamma=gamma, path=path)
    assert info["status"] == 0 and info["iters"] >= 15
    assert (info["sweep_samples"] == 0) == one
    # the other path's minimiser
    other = "gemv" if path == "syrk" or dtype == "bf16" else "syrk"
    y, _ = npga.solve(L, mu_d, r, gamma=gamma, path=other)
    assert np.abs(x.cpu().numpy() - y.cpu().numpy()).max() <= 1e-5
