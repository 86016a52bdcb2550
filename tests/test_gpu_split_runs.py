"""The three-plane product leaves float32 at least every 256 periods, whatever
the number of periods: rows of ones against rows of integers whose products
and 256-period sums float32 holds exactly, and longer runs' sums do not.

b: 2^24 at period p, 1 at two periods and -2^24 at one, all at least 256
periods after p.  The exact sum is 2; a float32 sum that still holds the
first when a 1 arrives rounds 2^24 + 1 to 2^24 and ends at 0.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import banner, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


# stages of 16 periods: 28 = 16 + 12, 24 = 16 + 8, 20 = 16 + 4, 44 = 32 + 12,
# and whole groups; p in each part of a group (the sums of a tile's four
# blocks leave float32 at different stages)
@pytest.mark.parametrize("T,p", [(448, 0), (448, 70), (448, 130), (384, 5), (320, 0), (704, 256), (704, 330),
                                 (512, 0), (512, 250), (768, 300), (433, 3)])
def test_runs_of_256_periods(npga, T, p):
    banner(f"float32 runs T={T} p={p}")
    n = 128
    L = np.zeros((T, n), dtype=np.float32)
    L[:, 0::2] = 1.0                     # rows of ones, among every block's rows and columns
    big = 2.0 ** 24
    L[p, 1::2] = big
    q = p + 256
    step = (T - 1 - q) // 2              # the three later periods, as far apart as T allows
    for t, v in ((q, 1.0), (q + step, 1.0), (q + 2 * step, -big)):
        L[t, 1::2] += np.float32(v)
    exact = L.astype(np.float64)[:, 1::2].sum(axis=0)
    assert np.all(exact == 2.0) and step >= 1
    S = npga.syrk(to_dev(L), method="split").cpu().numpy()
    assert np.all(S[0::2, 1::2] == 2.0) and np.all(S[1::2, 0::2] == 2.0)
