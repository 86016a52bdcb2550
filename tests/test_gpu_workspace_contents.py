"""No result depends on what the workspace holds when a call begins (a caller's
buffer is used again and again, and freshly allocated memory holds what was
there before): every entry point on a workspace of zeros and on one of 0xFF
bytes (not a number as float64, float32 or bfloat16) gives the same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import banner

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def npga():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02917_amd as p
    return p


def _factor(n, T, dtype="f32"):
    import paper_2604_02917_amd as npga
    g = torch.Generator(device=DEV).manual_seed(1000 * n + T)
    B = torch.randn((n, 4), generator=g, device=DEV)
    L = (0.02 * torch.randn((T, 4), generator=g, device=DEV) @ B.T +
         0.02 * torch.randn((T, n), generator=g, device=DEV)) / np.sqrt(T)
    mu = 5e-4 + 3e-4 * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    return (npga.to_bf16(L) if dtype == "bf16" else L), mu, float(mu.quantile(0.6))


def _bits(out):
    """The outputs, flat; floating-point values as bytes, so that NaN compares."""
    if torch.is_tensor(out):
        return [out.detach().cpu().numpy().tobytes()]
    if isinstance(out, dict):
        return [v for k in sorted(out) if not k.endswith("_ms") for v in _bits(out[k])]
    if isinstance(out, (list, tuple)):
        return [v for o in out for v in _bits(o)]
    return [np.asarray(out).tobytes()]


def _both(monkeypatch, npga, call):
    from paper_2604_02917_amd import api
    got = []
    for byte in (0, 255):
        monkeypatch.setattr(api, "_workspace",
                            lambda nbytes, device, b=byte: torch.full((max(int(nbytes), 256),), b, dtype=torch.uint8,
                                                                      device=device))
        try:
            got.append(_bits(call()))
        except npga.NpgaError as e:
            got.append([e.code])
    assert got[0] == got[1]


@pytest.mark.parametrize("n,T,dtype,kw", [
    (3, 5, "f32", {}), (40, 200, "f32", {}), (100, 60, "f32", {}), (300, 500, "f32", {}), (300, 500, "f32", {"alpha": 0.5}),
    (700, 300, "f32", {}), (700, 300, "f32", {"alpha": 0.5}), (1100, 1500, "f32", {"path": "syrk"}),
    (1100, 1500, "f32", {"path": "gemv"}), (1500, 700, "bf16", {"refine_method": "cg"}), (1100, 1500, "bf16", {"alpha": 0.5}),
    (2100, 2200, "f32", {"path": "gemv"}), (2100, 2200, "f32", {"path": "syrk"}), (2100, 2200, "bf16", {}),
    (3000, 3100, "f32", {"path": "gemv", "refine_precond": False}), (4500, 900, "f32", {"max_iter": 40}),
    (1100, 300, "f32", {"restart": True}), (1100, 300, "f32", {"momentum": "constant"}),
    (1100, 300, "f32", {"backtrack_rho": 0.5, "max_iter": 100}), (1100, 1300, "f32", {"step_estimator": "power"}),
    (1100, 300, "f32", {"projection": "dykstra", "dykstra_iters": 50, "max_iter": 60}),
])
def test_solve(npga, monkeypatch, n, T, dtype, kw):
    banner(f"workspace contents, solve n={n} T={T} {dtype} {kw}")
    L, mu, r = _factor(n, T, dtype)
    gamma = 0.0 if T > n else 1e-5
    _both(monkeypatch, npga, lambda: npga.solve(L, mu, r, gamma=gamma, **kw))


@pytest.mark.parametrize("n,T,m,dtype,kw", [
    (100, 300, 5, "f32", {}), (100, 60, 40, "f32", {}), (200, 100, 33, "bf16", {}), (1030, 1200, 3, "f32", {}),
    (300, 700, 70, "bf16", {"path": "syrk"}), (300, 20000, 70, "f32", {"path": "gemv"}), (130, 90, 17, "bf16", {"alpha": 0.5}),
    (2100, 300, 9, "f32", {"batch_config": 3}), (1500, 701, 24, "bf16", {"batch_config": 9}), (600, 900, 130, "f32", {}),
])
def test_batched(npga, monkeypatch, n, T, m, dtype, kw):
    banner(f"workspace contents, batched n={n} T={T} m={m} {dtype} {kw}")
    L, mu, _ = _factor(n, T, dtype)
    gamma = 0.0 if T > n else 1e-5
    mean, top = float(mu.mean()), float(mu.max())
    rs = [float(v) for v in np.linspace(mean, mean + 0.9 * (top - mean), m)]
    _both(monkeypatch, npga, lambda: npga.solve_batched(L, mu, rs, gamma=gamma, max_iter=400, **kw))
    X = torch.rand((m, n), device=DEV, generator=torch.Generator(device=DEV).manual_seed(m))
    _both(monkeypatch, npga, lambda: npga.gradient_batched(L, X, gamma=gamma, config=kw.get("batch_config", -1)))


@pytest.mark.parametrize("n,T,gamma", [(5, 9, 0.0), (100, 300, 0.0), (700, 300, 1e-4), (1500, 3000, 0.0), (2100, 2300, 0.0),
                                       (2600, 500, 1e-4)])
def test_backward(npga, monkeypatch, n, T, gamma):
    banner(f"workspace contents, backward n={n} T={T}")
    L, mu, r = _factor(n, T)
    x, _ = npga.solve(L, mu, r, gamma=gamma)
    g = torch.randn(n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(n))
    _both(monkeypatch, npga, lambda: npga.backward(L, mu, r, x, g, gamma=gamma))


@pytest.mark.parametrize("n,T,k,ell", [(30, 50, 8, 3), (300, 700, 130, 40), (700, 900, 600, 16), (2200, 2300, 2100, 8)])
def test_sketch(npga, monkeypatch, n, T, k, ell):
    banner(f"workspace contents, sketch n={n} T={T} k={k}")
    L, _, _ = _factor(n, T)
    g = torch.Generator(device=DEV).manual_seed(k)
    S = torch.randn((k, T), generator=g, device=DEV) / np.sqrt(k)
    h = torch.randint(0, k, (T,), generator=g, device=DEV, dtype=torch.int32)
    sgn = 2.0 * torch.randint(0, 2, (T,), generator=g, device=DEV).float() - 1.0
    _both(monkeypatch, npga, lambda: npga.sketch_str(L, S, ell))
    _both(monkeypatch, npga, lambda: npga.sketch_str_ex(L, k, ell))
    _both(monkeypatch, npga, lambda: npga.sketch_str_ex(L, k, ell, sketch="count", h=h, sgn=sgn))
    _both(monkeypatch, npga, lambda: npga.sketch_str_ex(L, k, ell, ell_rule="knee", tau=1e-6, rho=0.999999))


@pytest.mark.parametrize("n,T", [(3, 5), (300, 90), (1100, 700), (2500, 333)])
def test_single_steps(npga, monkeypatch, n, T):
    banner(f"workspace contents, single steps n={n} T={T}")
    L, mu, r = _factor(n, T)
    x = torch.rand(n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(n))
    v = torch.randn(n, device=DEV, dtype=torch.float64, generator=torch.Generator(device=DEV).manual_seed(T)) / n
    _both(monkeypatch, npga, lambda: npga.project(v, mu, r))
    _both(monkeypatch, npga, lambda: npga.project_dykstra(v, mu, r, max_iter=100))
    for dt in (L, npga.to_bf16(L)):
        _both(monkeypatch, npga, lambda: npga.gradient(dt, x, gamma=1e-4))
        for method in ("power", "lanczos"):
            _both(monkeypatch, npga, lambda: npga.spectral_norm_sq(dt, method=method))
    _both(monkeypatch, npga, lambda: npga.build_factor(L))
    _both(monkeypatch, npga, lambda: npga.syrk(L, method="split"))
