"""GPU parity of the ensemble workloads (rolling windows and the residual bootstrap on the
batched path, varlingam_var_simulate, varlingam_edge_frequency) against the FP64 oracle
(oracle.ensemble).

Tolerances:
* resampled series: the GPU stores every step in FP32 (relative rounding 2^-24) and runs the
  recursion from the stored rows; the generated processes are stable (spectral radius <= 0.9),
  so the accumulated difference from the FP64 recursion stays within a few tens of roundings
  of the series' scale: 1e-5 max|x| (measured 5e-8 .. 2e-7).  A wrong lag, a transposed M or a
  dropped intercept moves values by O(max|x|);
* per-problem orders and B: the batched fit's own bar (order within the oracle's near-tie
  margin, B within 1e-5 relative) where the GPU and the oracle fit the same series; 1e-4 for
  bootstrap resamples, whose series already differ by the FP32 rounding above (conditioning
  ~10 on these laws);
* aggregation: exact (integer counts divided once), on identical inputs, or when every
  problem's order matches the oracle's and no |B| lies within 1e-6 of the threshold.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import ensemble as EN
from oracle import varlingam as O
import parity as PA

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2409_05500_amd import api as _api
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return _api


def _dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t.to(dtype) if dtype is not None else t).cuda()


@pytest.mark.parametrize("case", [(7, 2, 5, 800), (300, 1, 3, 300), (40, 3, 9, 500)],
                         ids=lambda c: f"m{c[0]}_p{c[1]}_R{c[2]}_T{c[3]}")
def test_var_simulate_matches_oracle(api, case):
    m, p, R, T = case
    print(f"simulate m={m} p={p} R={R} T={T}", flush=True)
    inst = synth.make_custom(m, max(2 * m * p + 50, 900), p, "laplace", m + p,
                             edge_prob=0.1, w_lo=0.1, w_hi=0.5)
    X32 = inst.X32
    M, c, E = O.fit_var(X32.astype(np.float64), p)
    E32 = E.astype(np.float32)
    idx = np.random.default_rng(m).integers(0, len(E32), size=(R, T)).astype(np.int32)
    got = api.var_simulate(_dev(M), _dev(c), _dev(X32[:p]), _dev(E32), _dev(idx)).cpu().numpy()
    for r in range(R):
        ref = EN.simulate_var(M, c, X32[:p].astype(np.float64), E32.astype(np.float64), idx[r])
        err = np.abs(got[r] - ref).max() / np.abs(ref).max()
        assert np.array_equal(got[r][:p], X32[:p])
        assert err <= 1e-5, (r, err)
    print(f"  max rel err {err:.1e}", flush=True)


# Sizes at the edges of the recursion kernels' tiles (16 variables a task, 64 a group, one or two
# tasks a wave, past them the kernels without row broadcasts) and of the 8-step blocks of draws.
@pytest.mark.parametrize("case", [(1, 1, 9), (16, 1, 8), (17, 2, 7), (64, 1, 17), (65, 1, 16),
                                  (100, 2, 50), (128, 2, 15), (160, 1, 33), (161, 1, 12),
                                  (33, 5, 40), (10, 12, 25), (5, 17, 24)],
                         ids=lambda c: f"m{c[0]}_p{c[1]}_T{c[2]}")
def test_var_simulate_tile_edges(api, case):
    m, p, T = case
    print(f"simulate edges m={m} p={p} T={T}", flush=True)
    rng = np.random.default_rng(100 * m + p)
    M = rng.normal(0.0, 0.5 / np.sqrt(m * p), (p, m, m))
    c = rng.normal(0.0, 0.3, m)
    X0 = rng.normal(0.0, 1.0, (p, m)).astype(np.float32)
    E32 = rng.laplace(0.0, 1.0, (40, m)).astype(np.float32)
    idx = rng.integers(0, 40, size=(3, T)).astype(np.int32)
    got = api.var_simulate(_dev(M), _dev(c), _dev(X0), _dev(E32), _dev(idx)).cpu().numpy()
    for r in range(3):
        ref = EN.simulate_var(M, c, X0.astype(np.float64), E32.astype(np.float64), idx[r])
        assert np.array_equal(got[r][:p], X0)
        assert np.abs(got[r] - ref).max() / np.abs(ref).max() <= 1e-5, r


def test_var_simulate_identity_draws_full_size(api):
    """m = 400, n = 10000, p = 2: drawing the GPU fit's residuals in their own order
    regenerates the series (a property that holds at any size)."""
    wl = synth.FINANCE
    inst = synth.make_instance(wl, 0)
    X = _dev(inst.X32)
    M, c, E = api.fit_var(X, wl.p)
    T = wl.n - wl.p
    idx = np.stack([np.arange(T), np.random.default_rng(1).integers(0, T, T)]).astype(np.int32)
    out = api.var_simulate(M, c, X[:wl.p].contiguous(), E, _dev(idx))
    err = (out[0] - X).abs().max().item() / X.abs().max().item()
    print(f"  identity resample rel err {err:.1e}", flush=True)
    assert err <= 1e-5
    assert torch.isfinite(out[1]).all()


def test_edge_frequency_matches_oracle(api):
    rng = np.random.default_rng(5)
    K, m, p = 37, 23, 2
    orders = np.stack([rng.permutation(m) for _ in range(K)]).astype(np.int32)
    B0s = rng.normal(0, 0.2, (K, m, m)) * (rng.random((K, m, m)) < 0.6)
    Bls = rng.normal(0, 0.2, (K, p, m, m)) * (rng.random((K, p, m, m)) < 0.6)
    pst = np.where(rng.random(K) < 0.2, -3, 0).astype(np.int32)
    for thr, st in ((0.0, None), (0.1, pst)):
        P0, Pl, Po, cnt = api.edge_frequency(_dev(orders), _dev(B0s), _dev(Bls), thr,
                                             _dev(st) if st is not None else None)
        ref = EN.edge_frequency(orders, B0s, Bls, thr, None if st is None else st == 0)
        assert cnt == ref["count"]
        assert np.array_equal(P0.cpu().numpy(), ref["P0"])
        assert np.array_equal(Pl.cpu().numpy(), ref["P_lags"])
        assert np.array_equal(Po.cpu().numpy(), ref["P_order"])
    # no lags
    P0, Pl, Po, cnt = api.edge_frequency(_dev(orders), _dev(B0s), None, 0.05)
    ref = EN.edge_frequency(orders, B0s, np.zeros((K, 0, m, m)), 0.05)
    assert cnt == K and Pl.shape[0] == 0 and np.array_equal(P0.cpu().numpy(), ref["P0"])


def _check_fits(orders, B0s, Bls, series, p, tol):
    """Every problem against the oracle fit of its series; returns the oracle fits."""
    refs = [O.fit(np.asarray(s, dtype=np.float64), p) for s in series]
    for k, ref in enumerate(refs):
        assert PA.order_violations(orders[k], ref["S"]) == [], k
        if np.array_equal(orders[k], ref["order"]):
            B0r, Blr = ref["B0"], ref["B_lags"]
        else:
            B0r, Blr = O.estimate_B(ref["E"], orders[k], ref["M"])
        e = max(PA.b_rel_error(B0s[k], B0r), PA.b_rel_error(Bls[k], Blr))
        assert e <= tol, (k, e)
    return refs


def _aggregate_exact_if_determined(ef, refs, thr):
    """The GPU's aggregate equals the oracle's when every order agrees and no |B| sits within
    1e-6 of the threshold (both hold for the seeds used)."""
    orders = [np.asarray(r["order"]) for r in refs]
    assert all(np.array_equal(o, g) for o, g in zip(orders, ef.order.cpu().numpy()))
    B0 = np.array([r["B0"] for r in refs])
    Bl = np.array([r["B_lags"] for r in refs])
    assert np.abs(np.abs(np.concatenate([B0.ravel(), Bl.ravel()])) - thr).min() > 1e-6
    ref = EN.edge_frequency(orders, B0, Bl, thr)
    assert ef.count == ref["count"]
    assert np.array_equal(ef.P0.cpu().numpy(), ref["P0"])
    assert np.array_equal(ef.P_lags.cpu().numpy(), ref["P_lags"])
    assert np.array_equal(ef.P_order.cpu().numpy(), ref["P_order"])


def test_rolling_windows_match_oracle(api):
    inst = synth.make_custom(6, 3000, 1, "uniform", 11, edge_prob=0.5, w_lo=0.3, w_hi=0.7)
    X32 = inst.X32
    ef = api.rolling_windows(_dev(X32), 1, 800, 400, threshold=0.05)
    assert ef.starts == [0, 400, 800, 1200, 1600, 2000]
    assert ef.check() == [0] * 6
    series = [X32[s: s + 800] for s in ef.starts]
    refs = _check_fits(ef.order.cpu().numpy(), ef.B0.cpu().numpy(), ef.B_lags.cpu().numpy(),
                       series, 1, PA.B_TOL_FP32)
    _aggregate_exact_if_determined(ef, refs, 0.05)


def test_bootstrap_matches_oracle(api):
    """The resampled series differ from the oracle's by FP32 rounding, so the seed is one whose
    oracle order margins (>= 1.1e-4) and threshold distances (>= 2.8e-4) leave no decision to
    that rounding."""
    inst = synth.make_custom(5, 1500, 1, "uniform", 20, edge_prob=0.5, w_lo=0.3, w_hi=0.7)
    X32 = inst.X32
    idx = np.random.default_rng(20).integers(0, 1499, size=(6, 1499)).astype(np.int32)
    ef = api.bootstrap(_dev(X32), 1, idx, threshold=0.05)
    assert ef.check() == [0] * 6
    ref = EN.bootstrap(X32.astype(np.float64), 1, idx, 0.05)
    for r in range(6):
        err = np.abs(ef.series[r].cpu().numpy() - ref["series"][r]).max() / \
            np.abs(ref["series"][r]).max()
        assert err <= 1e-5, (r, err)
    refs = _check_fits(ef.order.cpu().numpy(), ef.B0.cpu().numpy(), ef.B_lags.cpu().numpy(),
                       ref["series"], 1, 1e-4)
    _aggregate_exact_if_determined(ef, refs, 0.05)


def test_bootstrap_workload_identity_draw(api):
    """The m = 100, n = 5000 series: a resample drawn in the residuals' own order is the
    series itself, and its batched fit gives the single-problem fit's order and B."""
    wl = synth.MEDIUM
    inst = synth.make_instance(wl, 0)
    X = _dev(inst.X32)
    T = wl.n - wl.p
    rng = np.random.default_rng(4)
    idx = np.stack([np.arange(T), rng.integers(0, T, T), rng.integers(0, T, T)])
    ef = api.bootstrap(X, wl.p, idx.astype(np.int32), threshold=0.05)
    assert ef.check() == [0, 0, 0] and ef.count == 3
    assert (ef.series[0] - X).abs().max().item() <= 1e-5 * X.abs().max().item()
    one = api.fit(X, wl.p)
    assert torch.equal(ef.order[0], one.order)
    assert PA.b_rel_error(ef.B0[0].cpu().numpy(), one.B0.cpu().numpy()) <= 1e-4
    Po = ef.P_order.cpu().numpy()
    assert np.all(np.isin(np.round(Po * 3), [0, 1, 2, 3]))


def test_failed_window_is_left_out(api):
    inst = synth.make_custom(5, 2400, 1, "laplace", 13, edge_prob=0.4, w_lo=0.2, w_hi=0.6)
    X32 = inst.X32.copy()
    X32[:800, 2] = 1.5                        # window 0 has a constant series
    ef = api.rolling_windows(_dev(X32), 1, 800, 400, threshold=0.0)
    st = ef.check()
    assert st[0] != 0 and all(s == 0 for s in st[1:])
    assert ef.count == len(st) - 1
    P0, Pl, Po, cnt = api.edge_frequency(ef.order[1:], ef.B0[1:], ef.B_lags[1:], 0.0)
    assert cnt == ef.count
    assert torch.equal(P0, ef.P0) and torch.equal(Po, ef.P_order)


# Group counts whose partials are padded to an odd number of pairs (3, 4, 7, 8, 12 groups), with one
# and two tasks a wave.
@pytest.mark.parametrize("case", [(80, 2, 20), (64, 3, 9), (64, 4, 17), (48, 7, 24), (64, 8, 25),
                                  (33, 8, 10), (42, 12, 16)],
                         ids=lambda c: f"m{c[0]}_p{c[1]}_T{c[2]}")
def test_var_simulate_padded_partials(api, case):
    test_var_simulate_tile_edges(api, case)
