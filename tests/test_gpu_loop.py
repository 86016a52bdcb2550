"""Small solves whose phases run as one launch: the shapes where the kernel's
split changes (entries per thread, items held on the compute unit, one or
several workgroups, streamed items), against the oracle's minimiser and
against the same solve with a launch per step; and the way out of a wait
that does not end.

Bars: the solver's own (relative objective 1e-6, entries 1e-5).  On the
covariance path a step's arithmetic is the launches' own, so the iteration
count and the iterates agree exactly.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import gen
from oracle import factor as ofactor
from oracle.reference import exact_mv_factor, factor_objective
from tests.gpu_util import banner, spec_with, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


class loop_wait:
    """npga_set_loop_wait for the block (us; negative: a launch per step)."""

    def __init__(self, us):
        self.us = us

    def __enter__(self):
        from paper_2604_02917_amd import api
        self.old = api._lib.npga_set_loop_wait(self.us)

    def __exit__(self, *exc):
        from paper_2604_02917_amd import api
        api._lib.npga_set_loop_wait(self.old)


def _case(npga, n, T, dtype):
    Rt = gen.returns_TxN(spec_with("c2", n, T, seed=900 + n + T))
    mu, L = ofactor.build_factor(Rt.T)
    Ld = to_dev(np.ascontiguousarray(L.T).astype(np.float32))
    if dtype == "bf16":
        Ld = npga.to_bf16(Ld)
    Lo = Ld[:, :n].float().cpu().numpy().astype(np.float64).T
    gamma = 0.0 if T > n else 1e-2 * float((Lo * Lo).sum()) / n
    r = float(np.percentile(mu, 60)) if n > 1 else float(mu[0]) - 1e-9
    return Ld, to_dev(mu), mu, Lo, gamma, r


CASES = [
    (1, 5, "f32", "syrk"), (2, 9, "f32", "syrk"), (64, 130, "f32", "syrk"), (128, 300, "f32", "syrk"),
    (129, 300, "f32", "syrk"), (256, 400, "f32", "syrk"), (257, 400, "f32", "syrk"), (512, 700, "f32", "syrk"),
    (513, 700, "f32", "syrk"), (1024, 1300, "f32", "syrk"), (1025, 1300, "f32", "syrk"),
    (3, 2, "f32", "gemv"), (100, 64, "f32", "gemv"), (100, 65, "f32", "gemv"), (256, 200, "bf16", "gemv"),
    (257, 48, "f32", "gemv"), (257, 49, "bf16", "gemv"), (300, 1400, "f32", "gemv"), (513, 16, "f32", "gemv"),
    (513, 17, "f32", "gemv"), (600, 290, "bf16", "gemv"), (1024, 333, "f32", "gemv"),
]


@pytest.mark.parametrize("n,T,dtype,path", CASES)
def test_one_launch_phases(npga, n, T, dtype, path):
    banner(f"one-launch phases n={n} T={T} {dtype} {path}")
    L, mu_d, mu, Lo, gamma, r = _case(npga, n, T, dtype)
    x, info = npga.solve(L, mu_d, r, gamma=gamma, path=path)
    with loop_wait(-1):
        xs, infos = npga.solve(L, mu_d, r, gamma=gamma, path=path)
    assert info["status"] == infos["status"] == 0 and infos["sweep_samples"] >= info["sweep_samples"] == 0
    xh = x.cpu().numpy().astype(np.float64)
    assert xh.min() >= 0.0 and abs(xh.sum() - 1.0) <= 1e-6 and mu @ xh >= r - 1e-6 * max(1.0, abs(r))
    assert np.abs(xh - xs.cpu().numpy()).max() <= 1e-5
    if path == "syrk":
        assert info["iters"] == infos["iters"] and info["residual"] == infos["residual"]
        assert info["alpha"] == infos["alpha"]
    ref = exact_mv_factor(Lo, gamma, mu, r)
    assert np.abs(xh - ref["x"]).max() <= 1e-5
    assert abs(factor_objective(Lo, gamma, xh) - ref["f"]) <= 1e-6 * abs(ref["f"])
    assert abs(info["objective"] - ref["f"]) <= 1e-6 * abs(ref["f"])


def test_one_launch_largest(npga):
    """2048 assets (streamed rows of Sigma) and a cut-off after a few steps:
    the iterates of both ways."""
    banner("one-launch phases n=2048, iterates")
    L, mu_d, mu, Lo, gamma, r = _case(npga, 2048, 2100, "f32")
    for k in (1, 7):
        x, info = npga.solve(L, mu_d, r, path="syrk", max_iter=k, refine=False)
        with loop_wait(-1):
            xs, infos = npga.solve(L, mu_d, r, path="syrk", max_iter=k, refine=False)
        assert info["status"] == infos["status"] == 3 and info["iters"] == infos["iters"] == k
        assert torch.equal(x, xs)


@pytest.mark.parametrize("n,T,path", [(300, 500, "syrk"), (700, 300, "gemv")])
def test_wait_runs_out(npga, n, T, path):
    """With no time to wait the launch gives up and the solve goes on with a
    launch per step, to the same minimiser."""
    banner(f"bounded wait n={n} T={T} {path}")
    L, mu_d, mu, Lo, gamma, r = _case(npga, n, T, "f32")
    with loop_wait(0):
        x, info = npga.solve(L, mu_d, r, gamma=gamma, path=path)
    assert info["status"] == 0
    ref = exact_mv_factor(Lo, gamma, mu, r)
    xh = x.cpu().numpy().astype(np.float64)
    assert np.abs(xh - ref["x"]).max() <= 1e-5
    assert abs(info["objective"] - ref["f"]) <= 1e-6 * abs(ref["f"])
