"""FP64 Gram tiles at their edges: 16-wide blocks and 64-wide tiles of columns, quarters and groups
of 16 samples, last groups of 1 to 15, splits that end inside a quarter.

Each entry is a sum of n exact products rounded in FP64: |C - C_ref| <= (n + 8) 2^-53 times the sum
of the absolute products, at most n sd_i sd_j by Cauchy-Schwarz; the tests allow 4 times that (the
reference rounds too, and the means are rounded sums themselves).
"""
import numpy as np
import pytest
import torch

from oracle import varlingam as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2409_05500_amd import api as _api
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return _api


def _data(n, m, seed):
    rng = np.random.default_rng(seed)
    X = rng.laplace(0.0, 1.0, (n, m)) * rng.uniform(0.5, 3.0, m) + rng.normal(0.0, 2.0, m)
    return X.astype(np.float32)


@pytest.mark.parametrize("m", [2, 15, 16, 17, 48, 49, 64, 65, 130])
@pytest.mark.parametrize("n", [40, 63, 64, 65, 127, 128, 129, 271, 1000, 4099])
def test_covariance_edges(api, m, n):
    E = _data(n, m, 31 * m + n)
    print(f"covariance m={m} n={n}", flush=True)
    X = torch.zeros((n, m + 3), device="cuda")          # a leading dimension of its own
    X[:, :m] = torch.from_numpy(E)
    cov = api.pairwise_stats(X[:, :m], "mixed")[3].cpu().numpy()
    E64 = E.astype(np.float64)
    d = E64 - E64.mean(0)
    ref = d.T @ d / n
    sd = np.sqrt(np.diag(ref))
    assert np.array_equal(cov, cov.T)
    assert np.all(np.abs(cov - ref) <= 4 * (n + 8) * 2.0 ** -53 * np.outer(sd, sd))


@pytest.mark.parametrize("shape", [(17, 40, 1), (16, 66, 2), (33, 150, 1), (49, 256, 1),
                                   (64, 300, 1), (65, 401, 2), (130, 1031, 1)],
                         ids=lambda s: f"m{s[0]}_n{s[1]}_p{s[2]}")
def test_batched_and_single_var_edges(api, shape):
    """The VAR fits through both forms of the Gram (one problem's splits, a batch's whole sums)
    against least squares on the data, 1e-9 of max|M| as the other fits."""
    m, n, p = shape
    print(f"var m={m} n={n} p={p}", flush=True)
    X = _data(n, m, 7 * m + n)
    M = O.fit_var(X.astype(np.float64), p)[0]
    single = api.fit_var(torch.from_numpy(X).cuda(), p, "mixed")[0].cpu().numpy()
    res, st = api.fit_batched([X, X[: n - 3]], p, "mixed")
    assert st == [0, 0]
    assert np.abs(single - M).max() <= 1e-9 * np.abs(M).max()
    assert np.abs(res[0].M.cpu().numpy() - M).max() <= 1e-9 * np.abs(M).max()


@pytest.mark.parametrize("m,n", [(3, 8319), (3, 8320), (64, 8319), (64, 8320), (200, 8192),
                                 (400, 8319), (600, 1100)])
def test_covariance_means_inside_and_before(api, m, n):
    """At the line between means formed inside the Gram (at most 64 column sums, one round of
    workgroups) and before it, and at its largest; with a NaN in the last column's last row."""
    test_covariance_edges(api, m, n)
    from paper_2409_05500_amd._lib import VarLiNGAMError, VL_ERR_NONFINITE
    E = _data(n, m, 5)
    E[n - 1, m - 1] = np.nan
    with pytest.raises(VarLiNGAMError) as ei:
        api.pairwise_stats(torch.from_numpy(E).cuda(), "mixed")
    assert ei.value.code == VL_ERR_NONFINITE


@pytest.mark.parametrize("m,p", [(1, 4), (13, 5), (16, 4), (21, 3), (33, 2), (43, 3), (64, 1),
                                 (65, 2), (128, 2)])
@pytest.mark.parametrize("prec", ["mixed", "sliced"])
def test_normal_equations_from_lag_products(api, m, p, prec):
    """The normal equations assembled from lag products, in tiles of 64 columns that end inside,
    at and past the lag blocks, against least squares on the data (1e-9 of max|M|, as above)."""
    n = 3 * m * p + 200 + m % 7
    X = _data(n, m, 13 * m + p)
    M = O.fit_var(X.astype(np.float64), p)[0]
    got = api.fit_var(torch.from_numpy(X).cuda(), p, prec)[0].cpu().numpy()
    assert np.abs(got - M).max() <= 1e-9 * np.abs(M).max()
