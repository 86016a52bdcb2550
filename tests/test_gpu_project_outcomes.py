"""npga_project's outcome is read from host memory that its launch writes: each
call's own, after calls with other outcomes and at other sizes.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.projection import proj_F
from tests.gpu_util import banner, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


def test_outcomes_in_turn(npga):
    banner("projection outcomes in turn")
    for k, n in enumerate((500, 3, 8192, 64, 257)):
        rng = np.random.default_rng(n)
        mu, v = rng.normal(5e-4, 4e-4, n), (1.0 + rng.standard_normal(n)) / n
        bad = mu.copy()
        bad[n // 2] = np.nan
        for r in (float(np.quantile(mu, 0.2)), float(np.quantile(mu, 0.95))):
            x, nu, tau = npga.project(to_dev(v), to_dev(mu), r)
            xo = proj_F(v, mu, r)[0]
            assert np.abs(x.cpu().numpy() - xo).max() <= 1e-9
            with pytest.raises(npga.NpgaError) as e:
                npga.project(to_dev(v), to_dev(mu), 2.0 * float(np.abs(mu).max()))
            assert e.value.code == 2
            with pytest.raises(npga.NpgaError) as e:
                npga.project(to_dev(v), to_dev(bad), r)
            assert e.value.code == 5
            x2, nu2, tau2 = npga.project(to_dev(v), to_dev(mu), r)
            assert torch.equal(x, x2) and (nu, tau) == (nu2, tau2)
