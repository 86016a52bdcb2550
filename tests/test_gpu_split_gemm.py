"""The three-plane bfloat16 products (Sigma = L L^T and Y = L S) at the edges
of their tiling: 128-row panels, 16-period stages padded to 64, 256-period
float64 flushes, left-over tiles split over the contraction.

Bound.  An entry is a sum of T products; each 256-period chunk is accumulated
in float32 over 16 stages of six plane products, every one a chain of 16
terms: at most 16 * 6 + 16 roundings reach a term, each within 2 u (u = 2^-24;
a truncating adder).  The three dropped plane products weigh 3 u, the stored
float32 u.  So |C - C_ref| <= 2 (112 + 3) u |A||B| + u |C_ref|.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import U32, banner, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


def _data(rows, T, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((T, rows)) * np.exp(2.0 * rng.standard_normal((T, rows)))).astype(np.float32)


@pytest.mark.parametrize("n,T", [
    (1, 1), (3, 15), (127, 16), (128, 17), (129, 63), (128, 256), (130, 257), (255, 320),
    (501, 2003),    # ten tiles, all of them split
    (2900, 640),    # 276 tiles: 256 whole, 20 split
    (4000, 2048),   # 528 tiles: 512 whole, 16 split
])
def test_syrk_split_edges(npga, n, T):
    banner(f"syrk split edges n={n} T={T}")
    Lt = _data(n, T, 31 * n + T)
    S = npga.syrk(to_dev(Lt), method="split").cpu().numpy().astype(np.float64)
    L = Lt.astype(np.float64)
    ref = L.T @ L
    bound = 2 * (112 + 3) * U32 * (np.abs(L).T @ np.abs(L)) + U32 * np.abs(ref)
    assert np.all(np.abs(S - ref) <= bound)
    assert np.array_equal(S, S.T)


@pytest.mark.parametrize("n,T,k", [(40, 33, 5), (130, 77, 37), (128, 1100, 64), (300, 2051, 129)])
def test_sketch_product_edges(npga, n, T, k):
    """ell = k keeps every eigenvector, so L_eff L_eff^T = Y Y^T whatever the
    eigenvectors' signs: V is orthogonal to float32 rounding, and L_eff = Y V
    is a float32 product of k terms on top of Y's own error."""
    banner(f"sketch product n={n} T={T} k={k}")
    Lt = _data(n, T, 7 * n + T)
    S = (np.random.default_rng(k).standard_normal((k, T)) / np.sqrt(k)).astype(np.float32)
    Leff, _, _ = npga.sketch_str(to_dev(Lt), to_dev(S), k)
    Le = Leff.cpu().numpy().astype(np.float64)
    L, Sd = Lt.astype(np.float64), S.astype(np.float64)
    Y = Sd @ L
    eY = 2 * (112 + 3) * U32 * (np.abs(Sd) @ np.abs(L)) + U32 * np.abs(Y)
    # ||L_eff L_eff^T - Y Y^T||_F <= 2 ||Y|| (||dY|| + (k + 2) u sqrt(k) ||Y||)
    nY = np.linalg.norm(Y)
    bar = 2 * nY * (np.linalg.norm(eY) + (k + 2) * np.sqrt(k) * U32 * nY)
    assert np.linalg.norm(Le.T @ Le - Y.T @ Y) <= bar
