"""GPU pruning of designs past 1280 columns to the least-squares end of the path: one variable
depends on every other at lag 0 and lag 1 strongly enough that BIC keeps the last knot, where the
lasso's coefficients are the ordinary least-squares ones (numpy, FP64, on the same FP32 data).
The active set then passes through every size: rows in registers to 1280 columns, by panels of
1024 beyond (one and two panel edges here).

|GPU - least squares| <= 1e-9 max|B|: a path of 2.2e3 steps in FP64 on a design of condition
number < 10 stays below 1e-11.
"""
import numpy as np
import pytest
import torch

from oracle import prune as P

pytestmark = pytest.mark.gpu
TOL = 1e-9


def _dense(m, n, seed):
    r = np.random.default_rng(seed)
    w = r.uniform(0.5, 1.0, 2 * m) * r.choice([-1.0, 1.0], 2 * m)
    x = r.normal(size=(n, m)).astype(np.float32)
    x[1:, m - 1] = (x[1:, :m - 1] @ w[:m - 1] + x[:-1, :m - 1] @ w[m:2 * m - 1]
                    + r.normal(size=n - 1))
    B0 = np.zeros((m, m))
    Bl = np.zeros((1, m, m))
    B0[m - 1, :m - 1] = w[:m - 1]
    Bl[0, m - 1, :m - 1] = w[m:2 * m - 1]           # its own lag stays out (weight 0)
    return x, B0, Bl


@pytest.mark.parametrize("m,n", [(650, 4000), (1100, 6000)])
def test_prune_long_design_to_least_squares(m, n):
    from paper_2409_05500_amd import api
    print(f"prune m={m} n={n}", flush=True)
    X, B0, Bl = _dense(m, n, 3)
    y, Z, cols = P.regression_design(X.astype(np.float64), 1, range(m), m - 1)
    Z = Z[:, :-1]                                    # (the last column is its own lag)
    want = np.linalg.solve(Z.T @ Z, Z.T @ y)
    dev = [torch.from_numpy(a).cuda() for a in (X, np.arange(m, dtype=np.int32), B0, Bl)]
    B0o, Blo, info = (t.cpu().numpy() for t in api.prune(dev[0], 1, *dev[1:]))
    steps, knot, df = info[m - 1]
    print(f"  steps {steps} knot {knot} df {df}", flush=True)
    assert knot == steps and df == 2 * m - 2
    got = np.concatenate([B0o[m - 1, :m - 1], Blo[0, m - 1, :m - 1]])
    err = np.abs(got - want).max() / np.abs(want).max()
    print(f"  max |err| / max|B| {err:.1e}", flush=True)
    assert err <= TOL
    assert np.count_nonzero(B0o) == m - 1 and np.count_nonzero(Blo) == m - 1
