"""GPU pruning on linearly dependent designs, against the FP64 oracle: integer-valued predecessors
of one variable, some of them sums and differences of others, so a column whose combination is
active is excluded when it tries to join.  In every listed design but the duplicate's a column is
active at the best knot so far, leaves the active set, and is excluded at the step whose knot is
chosen: its coefficient there is 0.

Coefficients: |GPU - oracle| <= 1e-9 max|B|, exactly the same zeros, knot and df.  The step at
which a dependent column comes up is the one to the least-squares fit (its correlation keeps a
fixed ratio to the active ones from the moment its combination is active), so that step's
candidates are equal but for rounding; each of them leads to the same knot.
"""
import numpy as np
import pytest
import torch

from oracle import prune as P

pytestmark = pytest.mark.gpu
TOL = 1e-9


@pytest.fixture(scope="module")
def api():
    from paper_2409_05500_amd import api as _api
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return _api


def _dependent(seed, T, k):
    """T x k integer design with 1 .. 3 dependent columns, weights, target."""
    r = np.random.default_rng(seed)
    dep = int(r.integers(1, 4))
    k0 = k - dep
    f = r.integers(-3, 4, (T, 1))
    Z = r.integers(-4, 5, (T, k0)).astype(float) + f * r.integers(0, 3, (1, k0))
    for _ in range(dep):
        n = int(r.integers(1, min(4, k0) + 1))
        idx = r.choice(k0, n, replace=False)
        Z = np.column_stack([Z, Z[:, idx] @ r.choice([-2, -1, 1, 2], n)])
    Z = Z[:, r.permutation(k)]
    w = r.uniform(0.2, 1.0, k)
    y = np.rint(Z @ (r.uniform(-1, 1, k) * (r.random(k) < 0.6))
                + r.normal(size=T) * r.choice([2, 6, 12])).astype(float)
    return Z, w, y


def _duplicated(T):
    """Columns 1 and 4 equal, with different weights."""
    r = np.random.default_rng(5)
    Z = r.integers(-4, 5, (T, 6)).astype(float)
    Z[:, 4] = Z[:, 1]
    w = np.array([0.4, 0.5, 0.9, 0.3, 0.8, 0.6])
    y = np.rint(Z @ np.array([1.0, -2.0, 0.5, 1.0, 1.0, 0.25]) + r.normal(size=T) * 2.0)
    return Z, w, y


def _series(Z, w, y, m):
    """The design as predecessors 0 .. k-1 of variable k of a series of m variables (p = 1, row 0
    outside the sample, every other weight 0)."""
    T, k = Z.shape
    X = np.random.default_rng(1).integers(-4, 5, (T + 1, m)).astype(np.float32)
    X[0] = 0.0
    X[1:, :k] = Z
    X[1:, k] = y
    B0 = np.zeros((m, m))
    B0[k, :k] = w
    return X, np.arange(m, dtype=np.int32), B0, np.zeros((1, m, m))


def _run(api, X, order, B0, Bl):
    dev = [torch.from_numpy(a).cuda() for a in (X, order, B0, Bl)]
    return [t.cpu().numpy() for t in api.prune(dev[0], 1, *dev[1:])]


def _check(got, want, k, m):
    B0, Bl, info = got
    oi = want["info"][0]
    assert tuple(info[k][1:]) == (oi["knot"], oi["df"]), (info[k], oi)
    assert np.array_equal(B0 != 0, want["B0"] != 0)
    assert np.all(Bl == 0)
    err = np.abs(B0 - want["B0"]).max() / np.abs(want["B0"]).max()
    print(f"  m {m} k {k}: knot {oi['knot']} df {oi['df']} err {err:.1e}", flush=True)
    assert err <= TOL


# (T, k, seed, m): the state in LDS, then in memory (2 m - 1 > 1280 columns)
CASES = [(26, 6, 10081, 7), (26, 8, 7023, 9), (40, 9, 13929, 10), (60, 8, 53852, 20),
         (1400, 9, 17588, 641), (1400, 9, 48812, 645)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"T{c[0]}_k{c[1]}_m{c[3]}_{c[2]}")
def test_prune_column_leaves_and_is_excluded(api, case):
    T, k, seed, m = case
    print(f"prune dependent T={T} k={k} seed={seed} m={m}", flush=True)
    X, order, B0, Bl = _series(*_dependent(seed, T, k), m)
    want = P.prune(X.astype(np.float64), 1, order, B0, Bl, positions=[k])
    oi = want["info"][0]
    left = [j for e, j in oi["events"] if e == -1]
    assert any(want["B0"][k, j] == 0.0 and (1, j) in oi["events"][oi["events"].index((-1, j)):]
               for j in left), "a column leaves, comes up again and stays out"
    _check(_run(api, X, order, B0, Bl), want, k, m)


@pytest.mark.parametrize("m", [7, 641])
def test_prune_duplicated_column(api, m):
    print(f"prune duplicated m={m}", flush=True)
    X, order, B0, Bl = _series(*_duplicated(1400), m)
    want = P.prune(X.astype(np.float64), 1, order, B0, Bl, positions=[6])
    assert (want["B0"][6, 1] == 0.0) != (want["B0"][6, 4] == 0.0)
    _check(_run(api, X, order, B0, Bl), want, 6, m)
