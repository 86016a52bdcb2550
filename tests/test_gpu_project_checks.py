"""The checks of npga_project, made in the projection's own launch: a
non-finite mu is reported before an unreachable return, wherever it stands,
and the largest reachable return (the largest mu, also when all are negative)
is accepted and one step above it is not."""
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


@pytest.mark.parametrize("n", [1, 64, 255, 257, 2049, 8192])
def test_checks(npga, n):
    banner(f"projection checks n={n}")
    rng = np.random.default_rng(n)
    mu = -1e-3 - rng.random(n)
    v = rng.standard_normal(n)
    top = float(mu.max())
    npga.project(to_dev(v), to_dev(mu), top)
    with pytest.raises(npga.NpgaError) as e:
        npga.project(to_dev(v), to_dev(mu), float(np.nextafter(top, 0.0)))
    assert e.value.code == 2
    for at, bad in ((n - 1, np.nan), (0, np.inf), (n // 2, -np.inf)):
        m = mu.copy()
        m[at] = bad
        with pytest.raises(npga.NpgaError) as e:
            npga.project(to_dev(v), to_dev(m), 1.0)
        assert e.value.code not in (0, 2)
