"""A tile configuration that a caller names governs both batched products, also
where the built-in choice (-1) takes other kernels for small ones (the U
product split over the assets, the bfloat16 G product as one sum): the results
are those of that configuration's sums, which differ in their last bits from
the built-in choice's.  All are within the gradient bar (n + T + 8) u32 B.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import quantize as oq
from tests.gpu_util import U32, banner, to_dev
from tests.test_gpu_batched import _rows_on_simplex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


def _configs(npga, n, T, m, dtype):
    rng = np.random.default_rng(n + T + m)
    Rt = (0.02 * rng.standard_normal((T, n))).astype(np.float32)
    X = _rows_on_simplex(m, n, 7 + m)
    Ld, Lt = to_dev(Rt), Rt.astype(np.float64)
    if dtype == "bf16":
        Ld = npga.to_bf16(Ld)
        Lt = oq.round_to_bf16(Rt).reshape(Rt.shape)
    L, Xd = Lt.T, X.astype(np.float64).T
    ref = 2 * (L @ (L.T @ Xd))
    bar = (n + T + 8) * U32 * 2 * (np.abs(L) @ (np.abs(L).T @ np.abs(Xd)))
    G = {c: npga.gradient_batched(Ld, to_dev(X), config=c)[0] for c in range(-1, 12)}
    for g in G.values():
        assert np.all(np.abs(g.cpu().numpy().T - ref) <= bar)
    return G


def _ranges(T, splits):
    """Ranges of the G product: whole 32-period steps."""
    chunk = -(-(-(-T // splits)) // 32) * 32
    return -(-T // chunk)


@pytest.mark.parametrize("n,T,m", [(1500, 701, 24), (300, 1100, 100)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_named_configuration_governs(npga, n, T, m, dtype):
    banner(f"batch configurations n={n} T={T} m={m} {dtype}")
    G = _configs(npga, n, T, m, dtype)
    assert not any(torch.equal(G[-1], G[c]) for c in range(12))
    # configurations 0, 1 and 11 differ in their ranges: 16, 32 and 64 asked for
    for (c, s), (d, u) in (((0, 16), (1, 32)), ((1, 32), (11, 64)), ((0, 16), (11, 64))):
        assert torch.equal(G[c], G[d]) == (_ranges(T, s) == _ranges(T, u)), (c, d)
