"""The factor path's phases as one launch: the gradient's sum over the columns
of L leaves float32 after two columns and is exchanged with more than float32
precision, as the launches' sum, which adds whole workgroups' columns in
float64, keeps what single columns contribute.

Three columns of powers of two: a = K e0, c = e0, b = K e0 - 2 K e1, all
others zero.  At x = 1/n they add K^2/n, 1/n and -K^2/n to (L L^T x)_0, with K
= 2^12; a float32 sum of the first two loses the second (a tie, rounded to
even).  With the step 1/8 given and one iteration, x_0 and x_2 then differ by
1/8 g_0 = 1/(4 n): every product, g and x before its rounding to float32 are
exact, so the bar is that rounding, 2 * 2^-24 / n, four times over.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import banner, to_dev
from tests.test_gpu_loop import loop_wait

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


# (n, T, columns a, c, b): of one wavefront, held or streamed; of one
# workgroup's piece and another's (entries per thread 1, 2, 4)
CASES = [
    (256, 60, 0, 8, 16),                            # one workgroup
    (256, 100, 0, 16, 32), (256, 100, 0, 16, 4),    # 2 workgroups
    (512, 96, 0, 16, 32), (512, 96, 0, 16, 4),
    (512, 1600, 1344, 1568, 4),                     # 28 workgroups, streamed columns
    (1024, 64, 0, 32, 4),                           # 4 workgroups
    (1024, 1000, 0, 176, 352), (1024, 1000, 352, 528, 4),
]


@pytest.mark.parametrize("us", [50000, -1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,T,a,c,b", CASES)
def test_small_column_survives(npga, n, T, a, c, b, dtype, us):
    banner(f"column sums n={n} T={T} {a} {c} {b} {dtype} wait {us}")
    K = 4096.0
    L = np.zeros((T, n), dtype=np.float32)
    L[a, 0] = K
    L[c, 0] = 1.0
    L[b, 0] = K
    L[b, 1] = -2.0 * K
    Ld = to_dev(L)
    if dtype == "bf16":
        Ld = npga.to_bf16(Ld)
    mu = to_dev(np.zeros(n))
    with loop_wait(us):
        x, info = npga.solve(Ld, mu, -1.0, path="gemv", alpha=0.125, max_iter=1, refine=False)
    assert info["status"] == 3 and info["iters"] == 1
    xh = x.cpu().numpy().astype(np.float64)
    assert xh[1] == 0.0 and np.all(xh[3:] == xh[2])
    assert abs((xh[2] - xh[0]) - 0.25 / n) <= 8 * 2.0 ** -24 / n
