"""The workloads that the library's speed is measured on: calls that a user's program makes through
the public API, from the smallest fit to complete pruning paths.

    listed()            the workloads with fixed sizes
    draw(rng)           one more workload of the same ranges
    prepare(case, seed) inputs on the GPU, and the plan or handle a program keeps between calls
    run(state)          one pass through the API; returns its outputs
    work(case)          bytes and operations that one pass cannot do without
    exact(case, seed)   the same outputs in 64 bits, in plain torch

A case is a dict of plain values.  "op" names the call:

    fit        api.fit on a new series: the one-shot call of an interactive program
    refit      a kept Fitter on a new series of its shape; the program takes the VAR, the causal
               order and the structural matrices (the pairwise statistics are what "pairwise"
               returns)
    pairwise   api.pairwise_stats on residuals that are there already
    orderb     api.approx_order on a score matrix, then api.estimate_B on its order
    batch      a kept BatchFitter: uneven problems, one launch per stage
    rolling    a kept EnsembleFitter over the windows of one series, then its aggregate
    bootstrap  api.bootstrap: fit, resampled series, their fits, aggregate
    prune      api.prune of a fitted model, complete lasso paths
    grad       api.pairwise_score forward and backward: a training step on the residuals
    search     api.order_iterative, the original search (the heuristic's comparator)
    lags       api.select_lag
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2409_05500_amd import api

DEV = torch.device("cuda:0")
K1, K2, GAMMA = 79.047, 7.4129, 0.37457      # constants of the entropy approximation
LN2 = math.log(2.0)


# ------------------------------------------------------------------------------------------
# The cases
# ------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: a handful of series, one-shot, where launches and latency count
        dict(name="fit_m10_n1000", op="fit", m=10, n=1000, p=1, prec="mixed", noise="uniform"),
        # a medium panel refitted as new data arrives, default precision
        dict(name="refit_m100_n5000", op="refit", m=100, n=5000, p=1, prec="mixed",
             noise="laplace"),
        # the benchmark's workload: 400 heavy-tailed return series, two lags
        dict(name="refit_m400_n10000_p2", op="refit", m=400, n=10000, p=2, prec="sliced",
             noise="t4"),
        # the precompute alone at the largest series, ragged sample count
        dict(name="pairwise_m1000_n49999", op="pairwise", m=1000, n=49999, prec="mixed",
             noise="laplace"),
        # ordering and structural matrices from kept statistics; odd number of variables
        dict(name="orderb_m317_p3", op="orderb", m=317, p=3),
        # many small uneven problems at once
        dict(name="batch_256", op="batch", count=256, m_lo=20, m_hi=200, n_lo=500, n_hi=8000,
             p=1, prec="mixed", noise="laplace"),
        # a window moved along one series
        dict(name="rolling_m50_w2000", op="rolling", m=50, n=20000, window=2000, stride=100, p=1,
             prec="mixed", noise="laplace"),
        # edge probabilities from resampled series
        dict(name="bootstrap_m100_r100", op="bootstrap", m=100, n=5000, resamples=100, p=1,
             prec="mixed", noise="laplace"),
        # pruning of the benchmark's fit, complete paths: the longest call there is
        dict(name="prune_m400_p2", op="prune", m=400, n=10000, p=2, noise="t4"),
        # a gradient step on the residuals of the benchmark's size
        dict(name="grad_m400_n9998", op="grad", m=400, n=9998, prec="mixed", noise="t4"),
        # the original search on the medium panel's residuals
        dict(name="search_m100_n4999", op="search", m=100, n=4999, prec="mixed", noise="laplace"),
        # choice of the lag order before the fit
        dict(name="lags_m400_p4", op="lags", m=400, n=10000, p=4, noise="t4"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["fit", "refit", "refit", "pairwise", "orderb", "batch", "rolling",
                     "bootstrap", "prune", "grad", "search", "lags"])
    noise = rng.choice(["uniform", "laplace", "t4"])
    prec = rng.choice(["mixed", "mixed", "sliced"])
    if op == "fit":
        m, p = _log_int(rng, 5, 40), rng.choice([1, 1, 2])
        return dict(op=op, m=m, n=_log_int(rng, max(300, 8 * m * p), 6000), p=p, prec=prec,
                    noise=noise)
    if op == "refit":
        m, p = _log_int(rng, 20, 400), rng.choice([1, 1, 2, 3])
        return dict(op=op, m=m, n=_log_int(rng, max(1000, 4 * m * p), 20000), p=p, prec=prec,
                    noise=noise)
    if op == "pairwise":
        m = _log_int(rng, 10, 1000)
        return dict(op=op, m=m, n=_log_int(rng, 800, 50000), prec=prec, noise=noise)
    if op == "orderb":
        return dict(op=op, m=_log_int(rng, 10, 600), p=rng.choice([1, 2, 3]))
    if op == "batch":
        m_lo, n_lo = _log_int(rng, 10, 40), _log_int(rng, 500, 1500)
        return dict(op=op, count=_log_int(rng, 8, 256), m_lo=m_lo,
                    m_hi=m_lo + rng.randint(10, 160), n_lo=n_lo,
                    n_hi=n_lo + rng.randint(200, 6500), p=1, prec="mixed", noise=noise)
    if op == "rolling":
        n = _log_int(rng, 4000, 20000)
        return dict(op=op, m=_log_int(rng, 10, 80), n=n, window=rng.randint(800, n // 3),
                    stride=rng.randint(60, 400), p=1, prec="mixed", noise=noise)
    if op == "bootstrap":
        m, p = _log_int(rng, 10, 120), rng.choice([1, 1, 2])
        return dict(op=op, m=m, n=_log_int(rng, max(600, 8 * m * p), 5000),
                    resamples=_log_int(rng, 10, 128), p=p, prec="mixed", noise=noise)
    if op == "prune":
        m, p = _log_int(rng, 10, 300), rng.choice([1, 2])
        return dict(op=op, m=m, n=_log_int(rng, max(1000, 8 * m * (p + 1)), 12000), p=p,
                    noise=noise)
    if op == "grad":
        m = _log_int(rng, 20, 600)
        return dict(op=op, m=m, n=_log_int(rng, 1000, 20000), prec="mixed", noise=noise)
    if op == "search":
        m = _log_int(rng, 10, 250)
        return dict(op=op, m=m, n=_log_int(rng, 1000, 10000), prec="mixed", noise=noise)
    m, p = _log_int(rng, 10, 400), rng.choice([2, 3, 4, 5])
    return dict(op="lags", m=m, n=_log_int(rng, max(1000, 4 * m * p), 12000), p=p, noise=noise)


# ------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------
def _shocks(g, n, m, kind):
    """n x m independent values of mean 0 and variance 1."""
    if kind == "uniform":
        return (torch.rand((n, m), generator=g, device=DEV, dtype=torch.float64) - 0.5) \
            * math.sqrt(12.0)
    if kind == "laplace":
        u = torch.rand((n, m), generator=g, device=DEV, dtype=torch.float64) - 0.5
        return -torch.sign(u) * torch.log1p(-2.0 * u.abs()) / math.sqrt(2.0)
    z = torch.randn((n, m), generator=g, device=DEV, dtype=torch.float64)
    u = torch.rand((2, n, m), generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-300)
    chi2 = -2.0 * torch.log(u[0] * u[1])       # four degrees of freedom
    return z / torch.sqrt(chi2 / 4.0) / math.sqrt(2.0)


def _model(r, m, p):
    """A sparse acyclic B0 in a hidden order, A = (I - B0)^-1 and p dense lag matrices."""
    perm = r.permutation(m)
    low = np.tril(r.random((m, m)) < min(0.3, 8.0 / m), -1)
    w = np.where(r.random((m, m)) < 0.5, -1.0, 1.0) * r.uniform(0.1, 0.5, (m, m)) * low
    B0 = np.zeros((m, m))
    B0[np.ix_(perm, perm)] = w
    A = np.linalg.inv(np.eye(m) - B0)
    scale = 0.45 / math.sqrt(m * p) / max(1.0, np.linalg.norm(A) / math.sqrt(m))
    M = r.normal(0.0, scale, (p, m, m))
    return perm, B0, A, M


def _series(seed, n, m, p, kind):
    """An n x m float32 stationary series: the reduced-form VAR driven by A e(t)."""
    r = np.random.default_rng(np.random.SeedSequence(seed))
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    perm, _, A, M = _model(r, m, p)
    At = torch.from_numpy(np.ascontiguousarray(A.T)).to(DEV)
    Mt = [torch.from_numpy(np.ascontiguousarray(M[k].T)).to(DEV) for k in range(p)]
    s = _shocks(g, n + 32, m, kind) @ At
    x = s
    for _ in range(12):                        # the recursion's moving-average form, 12 terms
        y = s.clone()
        for k in range(p):
            y[k + 1:] += x[: x.shape[0] - k - 1] @ Mt[k]
        x = y
    return x[32:].float().contiguous(), perm


def _residuals(seed, n, m, kind):
    """n x m float32 residuals A e(t), what the fit of a series hands on."""
    r = np.random.default_rng(np.random.SeedSequence(seed))
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    _, _, A, _ = _model(r, m, 1)
    At = torch.from_numpy(np.ascontiguousarray(A.T)).to(DEV)
    return (_shocks(g, n, m, kind) @ At).float().contiguous()


def _lagged(X, p):
    """Centred targets and lags of the VAR regression, in 64 bits."""
    X = X.double()
    n = X.shape[0]
    Y = X[p:]
    Z = torch.cat([X[p - k: n - k] for k in range(1, p + 1)], 1)
    return Y, Z


def _var64(X, p):
    """The least-squares VAR with intercept: M, c, E in 64 bits."""
    Y, Z = _lagged(X, p)
    ym, zm = Y.mean(0), Z.mean(0)
    Yc, Zc = Y - ym, Z - zm
    coef = torch.linalg.solve(Zc.T @ Zc, Zc.T @ Yc)        # (m p) x m
    m = Y.shape[1]
    M = torch.stack([coef[k * m:(k + 1) * m].T for k in range(p)])
    return M, ym - coef.T @ zm, Yc - Zc @ coef


def _b64(cov, M, order):
    """B0 = regressions on the predecessors in `order`, and B_tau = (I - B0) M_tau."""
    m = cov.shape[0]
    L = torch.linalg.cholesky(cov[order][:, order])
    Li = torch.linalg.inv(L)
    Bp = torch.tril(-Li * torch.diagonal(L)[:, None], -1)
    B0 = torch.zeros_like(cov)
    B0[order[:, None], order[None, :]] = Bp
    return B0, (torch.eye(m, dtype=cov.dtype, device=cov.device) - B0) @ M


def _batch_shapes(case, seed):
    """The uneven sizes are the case's own, the same for every seed."""
    r = np.random.default_rng(np.random.SeedSequence(case["count"] * 1000 + case["m_hi"]))
    ms = r.integers(case["m_lo"], case["m_hi"] + 1, case["count"])
    ns = r.integers(case["n_lo"], case["n_hi"] + 1, case["count"])
    return [(max(int(n), 3 * int(m) + 50), int(m)) for n, m in zip(ns, ms)]


def _batch_series(case, seed):
    return [_series(seed * 1009 + b, n, m, case["p"], case["noise"])[0]
            for b, (n, m) in enumerate(_batch_shapes(case, seed))]


def _scores(seed, m, p):
    """A score matrix as the precompute leaves it (small antisymmetric noise, strong entries along
    the edges of a hidden order), a covariance and lag matrices."""
    r = np.random.default_rng(np.random.SeedSequence(seed))
    perm, B0, A, M = _model(r, m, p)
    pos = np.empty(m, dtype=np.int64)
    pos[perm] = np.arange(m)
    up = np.triu(r.normal(0.0, 0.01, (m, m)), 1)
    noise = up - up.T
    strong = np.abs(A) * r.uniform(0.02, 0.2, (m, m)) * (pos[:, None] > pos[None, :])
    S = noise + strong.T - strong               # S[i, j] > 0 favours i before j
    e = r.uniform(0.5, 1.5, m)
    cov = (A * e) @ A.T
    return S, (cov + cov.T) / 2, M


def prepare(case, seed):
    op = case["op"]
    if op in ("fit", "refit", "lags"):
        X, _ = _series(seed, case["n"], case["m"], case["p"], case["noise"])
        s = {"case": case, "X": X}
        if op == "refit":
            s["fitter"] = api.Fitter(case["n"], case["m"], case["p"], case["prec"], DEV)
        return s
    if op in ("pairwise", "search"):
        return {"case": case, "E": _residuals(seed, case["n"], case["m"], case["noise"])}
    if op == "grad":
        r = np.random.default_rng(np.random.SeedSequence([seed, 1]))
        G = torch.from_numpy(r.normal(0.0, 1.0, (case["m"], case["m"]))).to(DEV)
        return {"case": case, "E": _residuals(seed, case["n"], case["m"], case["noise"]), "G": G}
    if op == "orderb":
        S, cov, M = _scores(seed, case["m"], case["p"])
        return {"case": case, "S": torch.from_numpy(S).to(DEV),
                "cov": torch.from_numpy(cov).to(DEV), "M": torch.from_numpy(M).to(DEV)}
    if op == "batch":
        Xs = _batch_series(case, seed)
        bf = api.BatchFitter([tuple(x.shape) for x in Xs], case["p"], case["prec"], DEV)
        bf.load(Xs)
        return {"case": case, "bf": bf}
    if op == "rolling":
        X, _ = _series(seed, case["n"], case["m"], case["p"], case["noise"])
        w = case["window"]
        views = [X[t: t + w] for t in range(0, case["n"] - w + 1, case["stride"])]
        return {"case": case, "X": X, "ef": api.EnsembleFitter(views, case["p"], case["prec"])}
    if op == "bootstrap":
        X, _ = _series(seed, case["n"], case["m"], case["p"], case["noise"])
        T = case["n"] - case["p"]
        g = torch.Generator(device=DEV).manual_seed(int(seed) + 7)
        idx = torch.randint(0, T, (case["resamples"], T), generator=g, device=DEV,
                            dtype=torch.int32)
        return {"case": case, "X": X, "idx": idx}
    assert op == "prune"
    X, perm = _series(seed, case["n"], case["m"], case["p"], case["noise"])
    M, _, E = _var64(X, case["p"])
    order = torch.from_numpy(perm.astype(np.int64)).to(DEV)
    B0, Bl = _b64(E.T @ E / E.shape[0], M, order)
    return {"case": case, "X": X, "order": order.to(torch.int32), "B0": B0, "Bl": Bl}


# ------------------------------------------------------------------------------------------
# One pass
# ------------------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    op = c["op"]
    if op == "fit":
        f = api.fit(s["X"], c["p"], c["prec"])
        return {"M": f.M, "intercept": f.intercept, "E": f.E, "Hx": f.Hx, "Hr": f.Hr, "S": f.S,
                "Cov": f.Cov, "order": f.order, "margin": f.margin, "B0": f.B0,
                "B_lags": f.B_lags}
    if op == "refit":
        f = s["fitter"]
        f.run(s["X"])
        return {"M": f.M, "intercept": f.intercept, "E": f.E, "Cov": f.Cov, "order": f.order,
                "B0": f.B0, "B_lags": f.B_lags}
    if op == "pairwise":
        Hx, Hr, S, Cov = api.pairwise_stats(s["E"], c["prec"])
        return {"Hx": Hx, "Hr": Hr, "S": S, "Cov": Cov}
    if op == "orderb":
        order, margin = api.approx_order(s["S"])
        B0, Bl = api.estimate_B(s["cov"], s["M"], order)
        return {"order": order, "margin": margin, "B0": B0, "B_lags": Bl}
    if op == "batch":
        s["bf"].run()
        r = s["bf"].results
        # the graphs of all problems gathered, as a program stores them
        return {"order": torch.cat([x.order for x in r]),
                "B0": torch.cat([x.B0.view(-1) for x in r]),
                "B_lags": torch.cat([x.B_lags.view(-1) for x in r]),
                "M": torch.cat([x.M.view(-1) for x in r]),
                "intercept": torch.cat([x.intercept for x in r])}
    if op == "rolling":
        ef = s["ef"]
        ef.run()
        P0, Pl, Po, count = ef.aggregate()
        return {"P0": P0, "P_lags": Pl, "P_order": Po, "count": count, "order": ef.order,
                "B0": ef.B0, "B_lags": ef.B_lags, "M": ef.M, "intercept": ef.intercept,
                "E": ef.E}
    if op == "bootstrap":
        ef = api.bootstrap(s["X"], c["p"], s["idx"], prec=c["prec"])
        return {"series": ef.series, "P0": ef.P0, "P_lags": ef.P_lags, "P_order": ef.P_order,
                "count": ef.count, "order": ef.order, "B0": ef.B0, "B_lags": ef.B_lags,
                "M": ef.M, "intercept": ef.intercept, "E": ef.E}
    if op == "prune":
        B0, Bl, info = api.prune(s["X"], c["p"], s["order"], s["B0"], s["Bl"])
        return {"B0": B0, "B_lags": Bl, "info": info}
    if op == "grad":
        E = s["E"].detach().requires_grad_(True)
        S = api.pairwise_score(E, c["prec"])
        S.backward(s["G"])
        return {"S": S.detach(), "dE": E.grad}
    if op == "search":
        order, margin = api.order_iterative(s["E"], c["prec"])
        return {"order": order, "margin": margin}
    assert op == "lags"
    logdet, aic, bic, best = api.select_lag(s["X"], c["p"])
    return {"logdet": logdet, "aic": aic, "bic": bic, "best": list(best)}


# ------------------------------------------------------------------------------------------
# What a pass cannot do without
# ------------------------------------------------------------------------------------------
# Operations of one pair, sample and direction of the precompute: the residual (3), two
# exponentials, one logarithm, and their products and sums.
EVAL_FLOPS = 12


def _fit_work(n, m, p):
    T = n - p
    by = 4.0 * n * m + 4.0 * T * m + 8.0 * (2 * p * m * m + 2 * m * m + 2 * m)
    fl = T * m * m * (p + 1) * 2.0                # lag products
    fl += (m * p) ** 3 / 3.0 + 2.0 * (m * p) ** 2 * m
    fl += 2.0 * T * m * m * p                     # residuals
    fl += 1.0 * T * m * m + EVAL_FLOPS * float(m) * (m - 1) * T
    fl += m ** 3 / 3.0 + 2.0 * p * m ** 3 + 3.0 * m * m
    return by, fl


def work(case):
    op, m, n, p = case["op"], case.get("m", 0), case.get("n", 0), case.get("p", 1)
    if op in ("fit", "refit"):
        by, fl = _fit_work(n, m, p)
    elif op == "pairwise":
        by = 4.0 * n * m + 8.0 * (3.0 * m * m + m)
        fl = n * m * m + EVAL_FLOPS * float(m) * (m - 1) * n
    elif op == "orderb":
        by = 8.0 * m * m * (3 + 2 * p) + 12.0 * m
        fl = 3.0 * m * m + m ** 3 / 3.0 + 2.0 * p * m ** 3
    elif op == "batch":
        by = fl = 0.0
        for nb, mb in _batch_shapes(case, 0):
            b, f = _fit_work(nb, mb, p)
            by, fl = by + b, fl + f
    elif op == "rolling":
        k = (n - case["window"]) // case["stride"] + 1
        b, f = _fit_work(case["window"], m, p)
        by, fl = k * (b - 4.0 * case["window"] * m) + 4.0 * n * m + 24.0 * m * m, k * f
    elif op == "bootstrap":
        b, f = _fit_work(n, m, p)
        k = case["resamples"]
        by, fl = (k + 1) * b + 4.0 * k * (n - p), (k + 1) * f + k * 2.0 * n * m * m * p
    elif op == "prune":
        by = 4.0 * n * m + 16.0 * (p + 1) * m * m + 12.0 * m
        fl = float(n) * (m * (p + 1)) ** 2
        # a path of d steps: the active inverse and the inactive correlations, d^3 / 3 each in all
        fl += sum(2.0 * (k + m * p) ** 3 / 3.0 for k in range(m))
    elif op == "grad":
        by = 8.0 * n * m + 16.0 * m * m
        fl = n * m * m + (EVAL_FLOPS + 24) * float(m) * (m - 1) * n
    elif op == "search":
        by = 4.0 * n * m + 12.0 * m
        fl = EVAL_FLOPS * float(n) * sum(u * (u - 1) for u in range(2, m + 1))
        fl += 2.0 * n * m * m
    else:
        by = 4.0 * n * m + 24.0 * p
        fl = (n - p) * m * m * (p + 1) * 2.0 + (m * p) ** 3 / 3.0 + 2.0 * p * (m * p) * m * m
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------------------------------
# The same outputs in 64 bits
# ------------------------------------------------------------------------------------------
def _logcosh(u):
    a = u.abs()
    return a + torch.log1p(torch.exp(-2.0 * a)) - LN2


def _entropy(A, B):
    return (1.0 + math.log(2.0 * math.pi)) / 2.0 - K1 * (A - GAMMA) ** 2 - K2 * B * B


def _pairwise64(E):
    """Hx, Hr, S, Cov and the moments of every ordered pair, one variable at a time."""
    E = E.double()
    n, m = E.shape
    mu = E.mean(0)
    cov = (E - mu).T @ (E - mu) / n
    sd = torch.sqrt(torch.diagonal(cov))
    x = ((E - mu) / sd).T.contiguous()             # m x n
    rho = cov / sd[:, None] / sd[None, :]
    A, B = torch.zeros_like(cov), torch.zeros_like(cov)
    step = max(1, int(1e8 // (8 * n)))
    for i in range(m):
        for j0 in range(0, m, step):
            j = slice(j0, min(m, j0 + step))
            r = rho[i, j][:, None]
            s = torch.sqrt((1.0 - r * r).clamp_min(1e-12))
            u = (x[i][None, :] - r * x[j]) / s
            A[i, j] = _logcosh(u).mean(1)
            B[i, j] = (u * torch.exp(-0.5 * u * u)).mean(1)
    Ax, Bx = _logcosh(x).mean(1), (x * torch.exp(-0.5 * x * x)).mean(1)
    Hx, Hr = _entropy(Ax, Bx), _entropy(A, B)
    Hr.fill_diagonal_(0.0)
    S = (Hx[None, :] + Hr) - (Hx[:, None] + Hr.T)
    S.fill_diagonal_(0.0)
    return Hx, Hr, S, cov, x, rho, sd, A, B, Ax, Bx


def _order64(S):
    """The lookup-only order and its margins."""
    S = S.cpu().numpy()
    m = S.shape[0]
    P = np.minimum(0.0, S) ** 2
    np.fill_diagonal(P, 0.0)
    live = np.ones(m, dtype=bool)
    order, margin = [], []
    for _ in range(m):
        idx = np.nonzero(live)[0]
        a = P[np.ix_(idx, idx)].sum(1)
        k = int(np.argmin(a))
        order.append(int(idx[k]))
        rest = np.delete(a, k)
        margin.append(float(rest.min() - a[k]) if rest.size else math.inf)
        live[idx[k]] = False
    return order, torch.tensor(margin, dtype=torch.float64, device=DEV)


def _grad64(E, G):
    """d<G, S(E)>/dE by the chain rule, one variable at a time."""
    n, m = E.shape
    Hx, Hr, S, cov, x, rho, sd, A, B, Ax, Bx = _pairwise64(E)
    Gh = G - G.T
    al, be = -2.0 * K1 * (A - GAMMA) * Gh / n, -2.0 * K2 * B * Gh / n
    dx = torch.zeros_like(x)
    step = max(1, int(1e8 // (8 * n)))

    def slope(u, a, b):
        return a * torch.tanh(u) + b * (1.0 - u * u) * torch.exp(-0.5 * u * u)

    for i in range(m):
        for j0 in range(0, m, step):
            j = slice(j0, min(m, j0 + step))
            r = rho[i, j][:, None]
            s2 = (1.0 - r * r).clamp_min(1e-12)
            s = torch.sqrt(s2)
            xi, xj = x[i][None, :], x[j]
            on = torch.ones((xj.shape[0], 1), dtype=torch.float64, device=x.device)
            if j0 <= i < j0 + xj.shape[0]:
                on[i - j0] = 0.0
            gij = slope((xi - r * xj) / s, al[i, j][:, None], be[i, j][:, None]) * on
            gji = slope((xj - r * xi) / s, al[j, i][:, None], be[j, i][:, None]) * on
            # u_ij = (x_i - r x_j) / s: through x_i directly, and through r = mean(x_i x_j)
            dx[i] += ((gij - r * gji) / s).sum(0)
            uij, uji = (xi - r * xj) / s, (xj - r * xi) / s
            R = (gij * (r * uij / s2 - xj / s) + gji * (r * uji / s2 - xi / s)).sum(1) / n
            dx[i] += R @ xj
    ci = Gh.sum(0)
    dx += slope(x, (-2.0 * K1 * (Ax - GAMMA) * ci / n)[:, None],
                (-2.0 * K2 * Bx * ci / n)[:, None])
    dx = dx - dx.mean(1, keepdim=True) - x * (x * dx).mean(1, keepdim=True)
    return S, (dx / sd[:, None]).T.contiguous()


def _search64(E):
    """Margins of the original search: scores recomputed on the updated data at every step."""
    X = E.double()
    margin = []
    while X.shape[1] > 1:
        n, u = X.shape
        _, _, S, _, x, rho, _, _, _, _, _ = _pairwise64(X)
        a = (S.clamp_max(0.0) ** 2).sum(1)
        v, k = torch.sort(a, stable=True)
        margin.append(float(v[1] - v[0]))
        c = int(k[0])
        keep = [j for j in range(u) if j != c]
        X = (x[keep] - rho[keep, c][:, None] * x[c][None, :]).T
    return torch.tensor(margin + [math.inf], dtype=torch.float64, device=DEV)


def _lasso_path64(Z, y, b):
    """Adaptive lasso of y on the columns of Z with weights |b|: the LARS path's knot of the
    smallest BIC, back in the columns' own scale."""
    T = len(y)
    sc = np.abs(b)
    Zs = Z * sc
    G, c0 = Zs.T @ Zs, Zs.T @ y
    d = len(b)
    act, sign = [], []
    beta, c = np.zeros(d), c0.copy()
    best, bic0 = beta.copy(), T * math.log(y @ y / T)
    free = [j for j in range(d) if sc[j] > 0]
    k = max(free, key=lambda j: abs(c[j]))
    Cc = Ct = abs(c[k])
    act.append(k)
    free.remove(k)
    for _ in range(8 * d):
        s = np.sign(c[act])
        q = np.linalg.solve(G[np.ix_(act, act)], s)
        AA = 1.0 / math.sqrt(s @ q)
        w = AA * q
        a = G[:, act] @ w
        full = Cc / AA
        best_g, event = full, None
        for j in free:
            for den, num in ((AA - a[j], Cc - c[j]), (AA + a[j], Cc + c[j])):
                if den != 0.0 and 1e-12 * full < num / den < best_g:
                    best_g, event = num / den, (1, j)
        for r, j in enumerate(act):
            if beta[j] != 0.0 and w[r] != 0.0 and 1e-12 * full < -beta[j] / w[r] < best_g:
                best_g, event = -beta[j] / w[r], (-1, j)
        beta[act] += best_g * w
        Cc -= best_g * AA
        c = c0 - G @ beta
        if event and event[0] < 0:
            beta[event[1]] = 0.0
            act.remove(event[1])
            free.append(event[1])
        elif event:
            act.append(event[1])
            free.remove(event[1])
        res = y - Zs @ beta
        bic = T * math.log(res @ res / T) + np.count_nonzero(beta) * math.log(T)
        if bic < bic0:
            bic0, best = bic, beta.copy()
        if event is None or Cc <= 1e-12 * Ct:
            break
    return best * sc


def _prune64(X, p, order, B0, Bl):
    Y, Z = (v.cpu().numpy() for v in _lagged(X, p))
    Yc, Zc = Y - Y.mean(0), Z - Z.mean(0)
    m = Y.shape[1]
    order, B0, Bl = order.cpu().numpy(), B0.cpu().numpy(), Bl.cpu().numpy()
    B0o, Blo = np.zeros_like(B0), np.zeros_like(Bl)
    for k, i in enumerate(order):
        pre = order[:k]
        b = np.concatenate([B0[i, pre], Bl[:, i, :].reshape(-1)])
        w = _lasso_path64(np.concatenate([Yc[:, pre], Zc], 1), Yc[:, i], b)
        B0o[i, pre] = w[:k]
        Blo[:, i, :] = w[k:].reshape(p, m)
    return torch.from_numpy(B0o), torch.from_numpy(Blo)


def _lags64(X, pmax):
    X = X.double()
    n, m = X.shape
    T = n - pmax
    Y = X[pmax:]
    Yc = Y - Y.mean(0)
    ld, aic, bic = [], [], []
    for p in range(1, pmax + 1):
        Z = torch.cat([X[pmax - k: n - k] for k in range(1, p + 1)], 1)
        Zc = Z - Z.mean(0)
        R = Yc - Zc @ torch.linalg.solve(Zc.T @ Zc, Zc.T @ Yc)
        v = float(torch.linalg.slogdet(R.T @ R / T)[1])
        ld.append(v)
        aic.append(v + 2.0 * p * m * m / T)
        bic.append(v + math.log(T) * p * m * m / T)
    return [torch.tensor(v, dtype=torch.float64) for v in (ld, aic, bic)]


def _stack_var64(Xs, p):
    M, c, E = zip(*[_var64(x, p) for x in Xs])
    return torch.stack(M), torch.stack(c), torch.stack(E)


def exact(case, seed):
    op, p = case["op"], case.get("p", 1)
    if op == "batch":
        fits = [_var64(x, p) for x in _batch_series(case, seed)]
        # the order's tie-breaks belong to the library's scores: no 64-bit value for what follows it
        return {"order": None, "B0": None, "B_lags": None,
                "M": torch.cat([f[0].reshape(-1) for f in fits]),
                "intercept": torch.cat([f[1] for f in fits])}
    if op == "prune" and case["m"] * (p + 1) > 60:
        return None                                # a plain path search takes minutes
    if op == "search" and case["m"] > 64:
        return None
    s = prepare(case, seed)
    if op == "fit":
        M, c, E = _var64(s["X"], p)
        Hx, Hr, S, cov = _pairwise64(E)[:4]
        order, margin = _order64(S)
        B0, Bl = _b64(cov, M, torch.tensor(order, device=DEV))
        # B0 and B_lags follow the order: they have a value where no step of it is a near-tie
        same = bool(margin.min() > 1e-5)
        return {"M": M, "intercept": c, "E": E, "Hx": Hx, "Hr": Hr, "S": S, "Cov": cov,
                "order": None, "margin": margin, "B0": B0 if same else None,
                "B_lags": Bl if same else None}
    if op == "refit":
        M, c, E = _var64(s["X"], p)
        return {"M": M, "intercept": c, "E": E, "Cov": E.T @ E / E.shape[0], "order": None,
                "B0": None, "B_lags": None}
    if op == "pairwise":
        Hx, Hr, S, cov = _pairwise64(s["E"])[:4]
        return {"Hx": Hx, "Hr": Hr, "S": S, "Cov": cov}
    if op == "orderb":
        order, margin = _order64(s["S"])
        B0, Bl = _b64(s["cov"], s["M"], torch.tensor(order, device=DEV))
        return {"order": None, "margin": margin, "B0": B0, "B_lags": Bl}
    if op == "rolling":
        M, c, E = _stack_var64(s["ef"].views, p)
        return {"P0": None, "P_lags": None, "P_order": None, "count": None, "order": None,
                "B0": None, "B_lags": None, "M": M, "intercept": c, "E": E}
    if op == "bootstrap":
        M, c, E = _var64(s["X"], p)
        E = E.float().double()
        idx = s["idx"].long()
        x = torch.empty((idx.shape[0], case["n"], case["m"]), dtype=torch.float64, device=DEV)
        x[:, :p] = s["X"][:p].double()
        Mt = [M[k].T.contiguous() for k in range(p)]
        for t in range(p, case["n"]):              # rounded to the stored float32 at every step
            v = c + E[idx[:, t - p]]
            for k in range(p):
                v = v + x[:, t - k - 1] @ Mt[k]
            x[:, t] = v.float().double()
        Ms, cs, Es = _stack_var64(list(x), p)
        return {"series": x, "P0": None, "P_lags": None, "P_order": None, "count": None,
                "order": None, "B0": None, "B_lags": None, "M": Ms, "intercept": cs, "E": Es}
    if op == "prune":
        B0, Bl = _prune64(s["X"], p, s["order"], s["B0"], s["Bl"])
        return {"B0": B0, "B_lags": Bl, "info": None}
    if op == "grad":
        S, dE = _grad64(s["E"], s["G"])
        return {"S": S, "dE": dE}
    if op == "search":
        return {"order": None, "margin": _search64(s["E"])}
    logdet, aic, bic = _lags64(s["X"], p)
    return {"logdet": logdet, "aic": aic, "bic": bic, "best": None}
