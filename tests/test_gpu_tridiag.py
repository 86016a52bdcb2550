"""Sketch eigensolver, tridiagonalisation in one launch: the sketch sizes
where its split changes (columns per thread, rows per workgroup, the largest
order held on the chip), against the float64 singular values of the sketched
factor and against a launch per stage of a column; and the way out of a wait
that does not end.

Bars.  Both ways are Householder reductions of the same float64 Gram matrix:
each moves an eigenvalue by at most about k 2^-53 lambda_1, below 1e-10 of
the eigenvalues compared here (all within a factor of ten of lambda_1), so
the float32 singular values agree to one rounding, 2^-23.  Against float64
the bar is the one of the float32 sketch product, 2e-5.
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


class tri_wait:
    """npga_set_loop_wait for the block (us; negative: a launch per stage)."""

    def __init__(self, us):
        self.us = us

    def __enter__(self):
        from paper_2604_02917_amd import api
        self.old = api._lib.npga_set_loop_wait(self.us)

    def __exit__(self, *exc):
        from paper_2604_02917_amd import api
        api._lib.npga_set_loop_wait(self.old)


def _case(k):
    n, T = k + 5, k + 21
    rng = np.random.default_rng(4000 + k)
    L = rng.standard_normal((T, n), dtype=np.float32)
    S = rng.standard_normal((k, T), dtype=np.float32) / np.float32(np.sqrt(k))
    return L, S, min(k, 8)


@pytest.mark.parametrize("k", [2, 3, 16, 17, 33, 255, 256, 257, 511, 512, 513, 1024, 1025, 2048, 2049, 3072, 3073,
                               3584, 3585])
def test_one_launch_tridiagonal(npga, k):
    banner(f"tridiagonalisation k={k}")
    L, S, ell = _case(k)
    Ld, Sd = to_dev(L), to_dev(S)
    Le, sg, gam = npga.sketch_str(Ld, Sd, ell)
    with tri_wait(-1):
        Le1, sg1, gam1 = npga.sketch_str(Ld, Sd, ell)
    s, s1 = sg.cpu().numpy().astype(np.float64), sg1.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(s, s1, rtol=2.0 ** -23)
    assert gam == gam1
    if k <= 1025:
        Y = L.astype(np.float64).T @ S.astype(np.float64).T
        np.testing.assert_allclose(s, np.linalg.svd(Y, compute_uv=False)[:ell], rtol=2e-5)
    # orthonormal eigenvectors: L_eff^T L_eff = diag(sigma^2)
    for M, sv in ((Le, s), (Le1, s1)):
        F = M.cpu().numpy().astype(np.float64)
        assert np.abs(F @ F.T - np.diag(sv * sv)).max() <= 1e-5 * sv[0] ** 2


@pytest.mark.parametrize("k", [40, 600, 3073])
def test_tridiagonal_wait_runs_out(npga, k):
    """With no time to wait the launch gives up; its columns are done again
    by launches, with the results of those alone."""
    banner(f"tridiagonalisation, bounded wait k={k}")
    L, S, ell = _case(k)
    Ld, Sd = to_dev(L), to_dev(S)
    with tri_wait(0):
        Le, sg, gam = npga.sketch_str(Ld, Sd, ell)
    with tri_wait(-1):
        Le1, sg1, gam1 = npga.sketch_str(Ld, Sd, ell)
    if k > 40:
        assert torch.equal(sg, sg1) and torch.equal(Le, Le1)
    else:  # few workgroups: their words may be there at the first look
        np.testing.assert_allclose(sg.cpu().numpy(), sg1.cpu().numpy(), rtol=2.0 ** -23)
    assert gam == gam1


@pytest.mark.parametrize("k", [2049, 3584 + 64])
def test_tridiagonal_later_launch_gives_up(npga, k):
    """Orders whose chain takes more than one launch, with no time to wait.
    k = 2049: the first launch has one column and needs no wait, the second
    gives up, so the launches go on from the matrix between the two."""
    banner(f"tridiagonalisation, bounded wait in a later launch k={k}")
    L, S, ell = _case(k)
    Ld, Sd = to_dev(L), to_dev(S)
    with tri_wait(0):
        Le, sg, gam = npga.sketch_str(Ld, Sd, ell)
    with tri_wait(-1):
        Le1, sg1, gam1 = npga.sketch_str(Ld, Sd, ell)
    s, s1 = sg.cpu().numpy().astype(np.float64), sg1.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(s, s1, rtol=2.0 ** -23)
    F = Le.cpu().numpy().astype(np.float64)
    assert np.abs(F @ F.T - np.diag(s * s)).max() <= 1e-5 * s[0] ** 2
    assert gam == gam1


@pytest.mark.parametrize("k", [3600, 3839, 3841, 4095, 4096, 4097])
def test_one_launch_tridiagonal_edge(npga, k):
    """Orders of which two rows a workgroup and a slot of columns stay in memory."""
    test_one_launch_tridiagonal(npga, k)


def test_tridiagonal_gives_up_after_the_edge(npga):
    """k = 3585: the launch with elements in memory has one column and needs
    no wait, the one after it gives up."""
    test_tridiagonal_later_launch_gives_up(npga, 3585)
