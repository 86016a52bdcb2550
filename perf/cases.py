"""Timed workloads of the mean-variance solver, through its public entry points.

Six kinds of call, each at the sizes where programs meet it:

  project   the feasible-set projection alone (a caller's own first-order loop)
  solve     one portfolio: L and mu in hand, float32 or bfloat16 storage
  rebuild   one portfolio from raw returns: build_factor, then the solve
  str       the sketch-truncate-ridge model: build it, then solve on it
  frontier  an efficient frontier: many targets on one factor
  train     decision-focused learning: the solve as a layer, forward and
            backward to mu and L

Inputs follow the factor-model recipe of the benchmark (ten factors,
Student-t(4) noise, a drift per asset), drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_2604_02917_amd as npga

DEV = "cuda:0"
FACTORS, FACTOR_SD, NOISE, DRIFT, DRIFT_SD = 10, 0.01, 0.015, 4e-4, 3e-4
RIDGE_SHORT = 1e-2   # ridge of a panel with fewer periods than assets, times the mean variance
RIDGE_STR = 1e-4     # ridge coefficient of the sketched model


def listed():
    return [
        # one projection inside a caller's own loop: the smallest call
        {"name": "project_n500", "kind": "project", "n": 500},
        # a desk-sized universe: every launch and synchronisation counts
        {"name": "solve_n64_T256", "kind": "solve", "n": 64, "T": 256, "dtype": "f32", "path": "auto"},
        # the small end of the paper's synthetic grid (T = 4 n), odd sizes
        {"name": "solve_n501_T2003", "kind": "solve", "n": 501, "T": 2003, "dtype": "f32", "path": "auto"},
        # fewer periods than assets, with a ridge
        {"name": "solve_n1001_T403_ridge", "kind": "solve", "n": 1001, "T": 403, "dtype": "f32", "path": "auto"},
        # the large end of the paper's synthetic grid
        {"name": "solve_n4000_T16000", "kind": "solve", "n": 4000, "T": 16000, "dtype": "f32", "path": "auto"},
        # the full model, re-estimated from returns each time: the benchmark's step
        {"name": "rebuild_n5440_T48374", "kind": "rebuild", "n": 5440, "T": 48374, "path": "gemv"},
        # the full model in 16-bit storage
        {"name": "solve_n5440_T48374_bf16", "kind": "solve", "n": 5440, "T": 48374, "dtype": "bf16", "path": "auto"},
        # a sketched model of ordinary size, sparse sketch, odd sizes
        {"name": "str_n1003_T6001_count", "kind": "str", "n": 1003, "T": 6001, "k": 403, "ell": 101,
         "sketch": "count"},
        # the sketched full model
        {"name": "str_n5440_T48374_gauss", "kind": "str", "n": 5440, "T": 48374, "k": 4096, "ell": 512,
         "sketch": "gaussian"},
        # a whole efficient frontier
        {"name": "frontier_n2000_T20000_m128", "kind": "frontier", "n": 2000, "T": 20000, "m": 128, "dtype": "f32"},
        # a few targets on a short panel in 16-bit storage
        {"name": "frontier_n1500_T701_m24_bf16", "kind": "frontier", "n": 1500, "T": 701, "m": 24, "dtype": "bf16"},
        # the full model as a layer of a training step
        {"name": "train_n5440_T48374", "kind": "train", "n": 5440, "T": 48374},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["project", "solve", "solve", "solve", "short", "rebuild", "str", "frontier", "train"])
    if kind == "project":
        return {"kind": "project", "n": _log(rng, 8, 8192)}
    if kind == "short":
        n = _log(rng, 100, 1500)
        return {"kind": "solve", "n": n, "T": max(16, int(n * rng.uniform(0.3, 0.8))),
                "dtype": rng.choice(["f32", "bf16"]), "path": "auto"}
    if kind == "solve":
        n = _log(rng, 32, 5440)
        return {"kind": "solve", "n": n, "T": min(48374, int(n * math.exp(rng.uniform(math.log(1.5), math.log(9.0))))),
                "dtype": rng.choice(["f32", "f32", "bf16"]), "path": "auto"}
    if kind == "rebuild":
        n = _log(rng, 32, 4000)
        return {"kind": "rebuild", "n": n, "T": int(n * rng.uniform(2.0, 9.0)), "path": rng.choice(["gemv", "auto"])}
    if kind == "str":
        n = _log(rng, 200, 4000)
        k = _log(rng, 64, max(65, min(2048, (3 * n) // 4)))
        return {"kind": "str", "n": n, "T": int(n * rng.uniform(2.0, 8.0)), "k": k,
                "ell": max(16, int(k * rng.uniform(0.12, 0.4))), "sketch": rng.choice(["gaussian", "count"])}
    if kind == "frontier":
        n = _log(rng, 50, 2000)
        return {"kind": "frontier", "n": n, "T": max(32, int(n * math.exp(rng.uniform(math.log(0.4), math.log(9.0))))),
                "m": rng.randint(2, 128), "dtype": rng.choice(["f32", "bf16"])}
    n = _log(rng, 32, 3000)
    return {"kind": "train", "n": n, "T": int(n * math.exp(rng.uniform(math.log(1.5), math.log(8.0))))}


# ---------------------------------------------------------------------- inputs

def _returns(n, T, seed, chunk=8192):
    """(T, n) float32 returns on the GPU."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    B = torch.randn((n, FACTORS), generator=g, device=DEV)
    d = DRIFT + DRIFT_SD * torch.randn(n, generator=g, device=DEV)
    R = torch.empty((T, n), device=DEV)
    for t0 in range(0, T, chunk):
        t1 = min(T, t0 + chunk)
        F = FACTOR_SD * torch.randn((t1 - t0, FACTORS), generator=g, device=DEV)
        z = torch.randn((t1 - t0, n), generator=g, device=DEV)
        q = 1.0 - torch.rand((t1 - t0, n), generator=g, device=DEV)
        q *= 1.0 - torch.rand((t1 - t0, n), generator=g, device=DEV)
        z /= q.log_().mul_(-0.5).sqrt_()      # normal over sqrt(chi^2_4 / 4)
        R[t0:t1] = (F @ B.T).add_(z, alpha=NOISE).add_(d)
    return R


def _factor64(R):
    """mu and L = (R - mu)/sqrt(T - 1) in float64."""
    mu = torch.zeros(R.shape[1], dtype=torch.float64, device=R.device)
    for t0 in range(0, R.shape[0], 8192):
        mu += R[t0:t0 + 8192].double().sum(0)
    mu /= R.shape[0]
    return (R.double() - mu).mul_(1.0 / math.sqrt(R.shape[0] - 1)), mu


def _factor(case, seed):
    """(L float32 (T, n), mu float64, r at the 60th percentile of mu)."""
    L, mu = _factor64(_returns(case["n"], case["T"], seed))
    return L.float(), mu, float(torch.quantile(mu, 0.6))


def _gamma(case, L):
    if case["T"] >= case["n"]:
        return 0.0
    return RIDGE_SHORT * float(L.double().square().sum()) / case["n"]


def _targets(case, mu):
    mean, top = float(mu.mean()), float(mu.max())
    return [float(v) for v in np.linspace(mean, mean + 0.95 * (top - mean), case["m"])]


def _sketch(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed + 7919)
    k, T = case["k"], case["T"]
    if case["sketch"] == "gaussian":
        return {"S": torch.randn((k, T), generator=g, device=DEV).mul_(1.0 / math.sqrt(k))}
    return {"h": torch.randint(0, k, (T,), generator=g, device=DEV, dtype=torch.int32),
            "sgn": 2.0 * torch.randint(0, 2, (T,), generator=g, device=DEV).float() - 1.0}


def _projected(case, seed):
    """The point a gradient step hands to the projection, with mu and r."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n = case["n"]
    mu = DRIFT + DRIFT_SD * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    v = (1.0 + torch.randn(n, generator=g, device=DEV, dtype=torch.float64)) / n
    return v, mu, float(torch.quantile(mu, 0.6))


def _heldout(case, seed):
    Rt = _returns(case["n"], 500, seed + 104729)
    return _factor64(Rt)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "project":
        v, mu, r = _projected(case, seed)
        return {"case": case, "v": v, "mu": mu, "r": r}
    if kind == "rebuild":
        R = _returns(case["n"], case["T"], seed)
        mu = _factor64(R)[1]
        return {"case": case, "R": R, "r": float(torch.quantile(mu, 0.6))}
    L, mu, r = _factor(case, seed)
    s = {"case": case, "L": L, "mu": mu, "r": r}
    if kind == "str":
        s.update(_sketch(case, seed))
        return s
    if kind == "train":
        Lt, mut = _heldout(case, seed)
        s.update(L=L.requires_grad_(), mu=mu.float().requires_grad_(), Lt=Lt.float(), mut=mut.float())
        return s
    s["gamma"] = _gamma(case, L)
    if kind == "frontier":
        s["targets"] = _targets(case, mu)
    if case["dtype"] == "bf16":
        s["L"] = npga.to_bf16(L)
    return s


# ------------------------------------------------------------------- one pass

def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "project":
        x, nu, tau = npga.project(s["v"], s["mu"], s["r"])
        return {"x": x, "tau": tau}
    if kind == "solve":
        x, info = npga.solve(s["L"], s["mu"], s["r"], gamma=s["gamma"], path=case["path"])
        return {"x": x, "objective": info["objective"], "status": info["status"]}
    if kind == "rebuild":
        L, mu = npga.build_factor(s["R"])
        x, info = npga.solve(L, mu, s["r"], path=case["path"])
        return {"mu": mu, "x": x, "objective": info["objective"], "status": info["status"]}
    if kind == "str":
        if case["sketch"] == "gaussian":
            Leff, sigma, gamma = npga.sketch_str(s["L"], s["S"], case["ell"], ridge_coef=RIDGE_STR)
        else:
            Leff, sigma, gamma, _ = npga.sketch_str_ex(s["L"], case["k"], case["ell"], sketch="count", h=s["h"],
                                                       sgn=s["sgn"], ridge_coef=RIDGE_STR)
        x, info = npga.solve(Leff, s["mu"], s["r"], gamma=gamma)
        return {"sigma": sigma, "gamma": gamma, "x": x, "objective": info["objective"], "status": info["status"]}
    if kind == "frontier":
        X, infos = npga.solve_batched(s["L"], s["mu"], s["targets"], gamma=s["gamma"])
        return {"X": X, "objective": np.array([i["objective"] for i in infos], dtype=np.float32),
                "status": np.array([i["status"] for i in infos])}
    x = npga.NPGAFunction.apply(s["mu"], s["L"], s["r"])
    loss = (s["Lt"] @ x).square().sum() - s["mut"] @ x
    dmu, dL = torch.autograd.grad(loss, (s["mu"], s["L"]))
    return {"x": x.detach(), "dmu": dmu, "dL": dL}


def work(case):
    n, T, kind = case["n"], case.get("T", 1), case["kind"]
    if kind == "project":
        return {"bytes": 24.0 * n, "flops": 4.0 * n}
    size = 2.0 if case.get("dtype") == "bf16" else 4.0
    if kind == "str":
        k, ell = case["k"], case["ell"]
        dense = case["sketch"] == "gaussian"
        return {"bytes": 4.0 * n * T + (4.0 * k * T if dense else 8.0 * T) + 4.0 * n * ell,
                "flops": (2.0 * n * T * k if dense else 2.0 * n * T) + 1.0 * n * k * k + 4.0 / 3.0 * k ** 3
                + 2.0 * k * k * ell + 2.0 * n * k * ell + 4.0 * n * ell}
    if kind == "frontier":
        return {"bytes": size * n * T + 4.0 * n * case["m"], "flops": 4.0 * n * T * case["m"]}
    if kind == "rebuild":
        return {"bytes": 8.0 * n * T, "flops": 8.0 * n * T}
    if kind == "train":
        return {"bytes": 8.0 * n * T, "flops": 12.0 * n * T}
    return {"bytes": size * n * T + 12.0 * n, "flops": 4.0 * n * T}


# ------------------------------------------- the same results in 64 bits (torch)

def _gram(L):
    """L^T L of a (cols, n) factor, float64."""
    n = L.shape[1]
    S = torch.zeros((n, n), dtype=torch.float64, device=L.device)
    for t0 in range(0, L.shape[0], 8192):
        C = L[t0:t0 + 8192].double()
        S += C.T @ C
    return S


def _on_face(Q, mu, r, F):
    """Minimiser of x'Qx with 1'x = 1, mu'x >= r and x = 0 off F (signs free):
    (x on F, nu, lambda, the Cholesky factor)."""
    one = torch.ones(F.numel(), dtype=torch.float64)
    m = mu[F]
    C = torch.linalg.cholesky(Q[F][:, F])
    P = torch.cholesky_solve(torch.stack([one, m], 1), C)
    p1, pm = P[:, 0], P[:, 1]
    a, b = 1.0 / float(p1.sum()), 0.0
    if a * float(m @ p1) < r:
        A = np.array([[float(p1.sum()), float(pm.sum())], [float(m @ p1), float(m @ pm)]])
        a, b = np.linalg.solve(A, np.array([1.0, r]))
    return a * p1 + b * pm, 2.0 * b, 2.0 * a, C


def _minimiser(Q, mu, r, F=None, most=400):
    """min x'Qx, 1'x = 1, mu'x >= r, x >= 0 by block principal pivoting (one
    index at a time while the blocks do not settle): (x, F, nu, C) or None."""
    n = Q.shape[0]
    free = torch.ones(n, dtype=torch.bool)
    if F is not None:
        free[:] = False
        free[F] = True
    best, patience = n + 1, 8
    for _ in range(most):
        F = free.nonzero()[:, 0]
        xF, nu, lam, C = _on_face(Q, mu, r, F)
        s = 2.0 * (Q[:, F] @ xF) - nu * mu - lam
        scale = float((2.0 * (Q[F][:, F] @ xF)).abs().max())
        bad = torch.zeros(n, dtype=torch.bool)
        bad[F] = xF < 0.0
        bad |= ~free & (s < -1e-12 * scale)
        count = int(bad.sum())
        if count == 0:
            x = torch.zeros(n, dtype=torch.float64)
            x[F] = xF
            return x, F, nu, C
        if count < best:
            best, patience = count, 8
            free ^= bad
        elif patience > 0:
            patience -= 1
            free ^= bad
        else:
            j = int(bad.nonzero()[-1, 0])
            free[j] = ~free[j]
        if not bool(free.any()):
            return None
    return None


def _exact_project(v, mu, r):
    v, mu = v.cpu(), mu.cpu()

    def simplex(w):
        u = torch.sort(w, descending=True).values
        k = torch.arange(1, u.numel() + 1, dtype=torch.float64)
        t = (torch.cumsum(u, 0) - 1.0) / k
        return float(t[int((u - t > 0).nonzero()[-1, 0])])

    def point(nu):
        w = v + nu * mu
        tau = simplex(w)
        return torch.clamp(w - tau, min=0.0), tau

    x, tau = point(0.0)
    if float(mu @ x) >= r:
        return x, tau
    lo, hi = 0.0, 1.0
    while float(mu @ point(hi)[0]) < r:
        lo, hi = hi, 2.0 * hi
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        if float(mu @ point(mid)[0]) < r:
            lo = mid
        else:
            hi = mid
    x, tau = point(hi)
    F = x > 0.0
    m, w, k = mu[F], v[F], int(F.sum())
    A = np.array([[float(k), float(m.sum())], [float(m.sum()), float(m @ m)]])
    if k > 1 and np.linalg.cond(A / np.outer(np.sqrt(np.diag(A)), np.sqrt(np.diag(A)))) < 1e10:
        neg, nu = np.linalg.solve(A, np.array([1.0 - float(w.sum()), r - float(m @ w)]))
        tau = -neg
        x[F] = w + nu * m - tau
    return x, float(tau)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "project":
        x, tau = _exact_project(*_projected(case, seed))
        return {"x": x, "tau": tau}
    if kind == "rebuild":
        L, mu = _factor64(_returns(n, case["T"], seed))
        r = float(torch.quantile(mu, 0.6))
        Q = _gram(L).cpu()
        got = _minimiser(Q, mu.cpu(), r)
        return got and {"mu": mu, "x": got[0], "objective": float(got[0] @ (Q @ got[0])), "status": None}
    L, mu, r = _factor(case, seed)
    m = mu.cpu()
    if kind == "str":
        if case["k"] > 2048:
            return None
        sk = _sketch(case, seed)
        if case["sketch"] == "gaussian":
            Y = sk["S"].double() @ L.double()
        else:
            Y = torch.zeros((case["k"], n), dtype=torch.float64, device=DEV)
            Y.index_add_(0, sk["h"].long(), L.double() * sk["sgn"].double()[:, None])
        gamma = RIDGE_STR * float(Y.square().sum()) / n
        w, V = torch.linalg.eigh((Y @ Y.T).cpu())
        V = V[:, -case["ell"]:].flip(1)
        Leff = V.T @ Y.cpu()
        Q = _gram(Leff) + gamma * torch.eye(n, dtype=torch.float64)
        got = _minimiser(Q, m, r)
        return got and {"sigma": w[-case["ell"]:].flip(0).clamp(min=0.0).sqrt(), "gamma": gamma, "x": got[0],
                        "objective": float(got[0] @ (Q @ got[0])), "status": None}
    if kind == "train":
        mu32 = mu.float().double()
        Q = _gram(L).cpu()
        got = _minimiser(Q, mu32.cpu(), r)
        if got is None:
            return None
        x, F, nu, C = got
        Lt, mut = _heldout(case, seed)
        Lt, mut = Lt.float().double(), mut.float().double()
        xd = x.to(DEV)
        g = (2.0 * (Lt.T @ (Lt @ xd)) - mut).cpu()[F]
        # adjoint on the face: [2Q, -mu, -1; mu', 0; 1', 0] [u; a; b] = [g; 0; 0]
        A = torch.stack([torch.ones(F.numel(), dtype=torch.float64)] + ([mu32.cpu()[F]] if nu > 0.0 else []), 1)
        P = torch.cholesky_solve(torch.cat([A, g[:, None]], 1), C) / 2.0
        PA, Pg = P[:, :-1], P[:, -1]
        w = torch.linalg.solve(A.T @ PA, -(A.T @ Pg))
        uF = Pg + PA @ w
        u = torch.zeros(n, dtype=torch.float64)
        u[F] = uF
        dmu = nu * u + (float(w[1]) * x if nu > 0.0 else 0.0)
        ud, Ld = u.to(DEV), L.double()
        dL = torch.outer(Ld @ xd, ud).add_(torch.outer(Ld @ ud, xd)).mul_(-2.0)
        return {"x": x, "dmu": dmu, "dL": dL}
    gamma = _gamma(case, L)
    if case["dtype"] == "bf16":
        L = L.bfloat16()
    Q = _gram(L).cpu() + gamma * torch.eye(n, dtype=torch.float64)
    if kind == "solve":
        got = _minimiser(Q, m, r)
        return got and {"x": got[0], "objective": float(got[0] @ (Q @ got[0])), "status": None}
    X, obj, F = [], [], None
    for t in _targets(case, mu):
        got = _minimiser(Q, m, t, F)
        if got is None:
            return None
        X.append(got[0])
        obj.append(float(got[0] @ (Q @ got[0])))
        F = got[1]
    return {"X": torch.stack(X), "objective": np.array(obj), "status": None}
