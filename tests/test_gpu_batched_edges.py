"""Batched products and tails at the edges of their tiles: 32-period tiles and
16-asset steps of the U product split over the assets, 64-row tiles, 32 / 64
target widths and stage ranges of the covariance form's product.

Gradient bar: (n + T + 8) u32 B as for the tiled products (a split sum has
no more roundings than one chain).  Solve bar: the single solves'.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import gen
from oracle import quantize as oq
from oracle.frontier import frontier
from tests.gpu_util import U32, banner, spec_with, to_dev
from tests.test_gpu_batched import _frontier_case, _rows_on_simplex
from tests.test_gpu_solve import _check_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,T,m", [(1, 1, 1), (5, 31, 2), (16, 32, 31), (17, 33, 32), (127, 64, 33), (129, 65, 64),
                                   (600, 4096, 128), (600, 4097, 128), (8192, 40, 3)])
def test_gradient_edges(npga, n, T, m, dtype):
    banner(f"batched gradient edges n={n} T={T} m={m} {dtype}")
    rng = np.random.default_rng(n + T + m)
    Rt = (0.02 * rng.standard_normal((T, n))).astype(np.float32)
    X = _rows_on_simplex(m, n, 7 + m)
    Ld, Lt = to_dev(Rt), Rt.astype(np.float64)
    if dtype == "bf16":
        Ld = npga.to_bf16(Ld)
        Lt = oq.round_to_bf16(Rt).reshape(Rt.shape)
    G, f = npga.gradient_batched(Ld, to_dev(X))
    L, Xd = Lt.T, X.astype(np.float64).T
    U = L.T @ Xd
    B = 2 * (np.abs(L) @ (np.abs(L).T @ np.abs(Xd)))
    assert np.all(np.abs(G.cpu().numpy().T - 2 * (L @ U)) <= (n + T + 8) * U32 * B)
    np.testing.assert_allclose(np.asarray(f), (U * U).sum(axis=0), rtol=1e-5)


@pytest.mark.parametrize("n,T,m", [(15, 60, 1), (63, 200, 32), (65, 200, 33), (129, 400, 64), (191, 500, 65),
                                   (257, 600, 128), (1030, 1200, 3)])
def test_covariance_form_edges(npga, n, T, m):
    banner(f"covariance form edges n={n} T={T} m={m}")
    L, mu, L_o, mu_o, rs = _frontier_case(n, T, m, 500 + n, 0.0, "f32", npga)
    X, infos = npga.solve_batched(L, mu, rs, path="syrk")
    pick = sorted({0, m // 2, m - 1})
    ref = frontier(L_o, 0.0, mu_o, [rs[j] for j in pick])
    Xh = X.cpu().numpy()
    for k, j in enumerate(pick):
        assert infos[j]["status"] == 0 and infos[j]["refined"] == 1, (j, infos[j])
        _check_parity(Xh[j], infos[j], L_o, mu_o, rs[j], 0.0, ref[k], f"target {j}")


@pytest.mark.parametrize("n,T,m", [(15, 7, 1), (31, 16, 15), (33, 17, 16), (255, 15, 17), (257, 100, 33), (1500, 701, 24),
                                   (40, 2048, 32), (40, 2049, 32), (1000, 512, 128)])
def test_gradient_small_tiles(npga, n, T, m):
    """The bfloat16 U product by 16 x 16 tiles (up to 64 tiles of 32 x 32):
    32-asset steps of eight wavefronts; the last but one shape is the first
    past the bound.  The bar of test_gradient_edges."""
    test_gradient_edges(npga, n, T, m, "bf16")
