"""GPU parity of the original iterative DirectLiNGAM ordering (varlingam_order_iterative, the
search of Sec. 3 steps 1-5 that the heuristic replaces) against the FP64 oracle.

Protocol (parity.iterative_order_violations): the GPU order is walked with the oracle's own
arithmetic; at every step the oracle's aggregate M over its current data must put the GPU's
pick within 1e-9 of the minimum (near-ties either way), and the oracle's data is then refined
with the GPU's pick.  The pairwise scores at each step are the heuristic path's (tolerance
6e-6 on S), so only steps whose oracle margin is below that could differ; the workloads here
have none."""
import numpy as np
import pytest
import torch

import synth
from oracle import varlingam as O
import parity as PA

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_2409_05500_amd import api as _api
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return _api


def _residuals(inst, p):
    _, _, E = O.fit_var(inst.X_parity, p)
    return E.astype(np.float32)


CASES = [(synth.make_instance(synth.SMALL, 0), 1), (synth.make_instance(synth.SMALL, 4), 1),
         (synth.make_custom(3, 600, 1, "laplace", 1), 1),
         (synth.make_custom(17, 900, 1, "uniform", 2), 1),
         (synth.make_custom(40, 2000, 1, "laplace", 3, edge_prob=0.1, w_lo=0.1, w_hi=0.5), 1),
         (synth.make_custom(65, 1500, 2, "t4", 4, edge_prob=0.05, w_lo=0.05, w_hi=0.4,
                            lag_radius=0.4), 2)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0].workload.name)
@pytest.mark.parametrize("prec", ["mixed", "fp32"])
def test_iterative_order_matches_oracle(api, case, prec):
    inst, p = case
    E = _residuals(inst, p)
    print(f"iterative {inst.workload.name} prec={prec}", flush=True)
    order, margin = api.order_iterative(torch.from_numpy(E).cuda(), prec)
    order = order.cpu().numpy()
    margin = margin.cpu().numpy()
    m = E.shape[1]
    assert sorted(order.tolist()) == list(range(m))
    assert np.isinf(margin[-1]) and np.all(margin[:-1] >= 0.0)
    bad = PA.iterative_order_violations(order, E)
    print(f"  min margin {margin[:-1].min() if m > 1 else np.inf:.2e}; violations {bad}",
          flush=True)
    assert bad == []


def test_iterative_first_pick_and_m2_equal_the_heuristic(api):
    """Step 1 scores the original data, so its pick is the heuristic's first pick; with two
    variables the two searches are the same."""
    for inst, p in CASES[:5]:
        E = torch.from_numpy(_residuals(inst, p)).cuda()
        it, _ = api.order_iterative(E)
        _, _, S, _ = api.pairwise_stats(E)
        he, _ = api.approx_order(S)
        assert int(it[0]) == int(he[0])
    E2 = torch.from_numpy(_residuals(synth.make_custom(2, 800, 1, "laplace", 9), 1)).cuda()
    it, mi = api.order_iterative(E2)
    _, _, S, _ = api.pairwise_stats(E2)
    he, mh = api.approx_order(S)
    assert torch.equal(it, he)
    assert float(mi[0]) == pytest.approx(float(mh[0]), rel=1e-12, abs=0.0)


def test_iterative_recovers_the_generating_order(api):
    """Strongly non-Gaussian noise, long series: the search recovers a topological order of
    the true B0 (no edge from a later to an earlier variable)."""
    inst = synth.make_custom(8, 20000, 1, "uniform", 5, edge_prob=0.4, w_lo=0.5, w_hi=0.9)
    E = _residuals(inst, 1)
    order = api.order_iterative(torch.from_numpy(E).cuda())[0].cpu().numpy()
    pos = {int(v): k for k, v in enumerate(order)}
    B0 = inst.B0
    viol = [(i, j) for i in range(8) for j in range(8) if B0[i, j] != 0 and pos[j] > pos[i]]
    assert viol == []


def test_iterative_degenerate_raises(api):
    from paper_2409_05500_amd._lib import VarLiNGAMError
    E = _residuals(synth.make_instance(synth.SMALL, 2), 1)
    E[:, 5] = 0.25
    with pytest.raises(VarLiNGAMError):
        api.order_iterative(torch.from_numpy(E).cuda())


@pytest.mark.parametrize("case", CASES[2:], ids=lambda c: c[0].workload.name)
def test_hybrid_order_matches_oracle(api, case):
    """k exact picks of the original search, then the lookup ordering on the refined data of
    the rest: walked with parity.hybrid_order_violations at several splits.  k = 0 is the
    heuristic's order of E itself and k >= m - 1 the original search's."""
    inst, p = case
    E = _residuals(inst, p)
    m = E.shape[1]
    Ed = torch.from_numpy(E).cuda()
    _, _, S, _ = api.pairwise_stats(Ed)
    he, mh = api.approx_order(S)
    it, mi = api.order_iterative(Ed)
    for k in sorted({0, 1, min(3, m), m // 2, m - 1, m, m + 5}):
        print(f"hybrid {inst.workload.name} k={k}", flush=True)
        order, margin = api.order_hybrid(Ed, k)
        assert sorted(order.cpu().tolist()) == list(range(m))
        assert np.isinf(float(margin[-1]))
        if k == 0:
            assert torch.equal(order, he) and torch.equal(margin, mh)
        if k >= m - 1:
            assert torch.equal(order, it) and torch.equal(margin, mi)
        if 0 < k < m - 1:
            assert torch.equal(order[:k], it[:k])
            bad = PA.hybrid_order_violations(order.cpu().numpy(), E, k)
            assert bad == [], (k, bad)


def test_hybrid_recovers_the_generating_order(api):
    """Strongly non-Gaussian data with a known DAG, every split k walked against the oracle.
    The heuristic tail is an approximation: here, as in the oracle's own hybrid, k <= 1 puts
    two effects before their causes, and from k = 2 on the order is a topological order of
    the generating B0."""
    inst = synth.make_custom(8, 20000, 1, "uniform", 5, edge_prob=0.4, w_lo=0.5, w_hi=0.9)
    E = _residuals(inst, 1)
    Ed = torch.from_numpy(E).cuda()
    for k in range(9):
        order = api.order_hybrid(Ed, k)[0].cpu().numpy()
        assert PA.hybrid_order_violations(order, E, k) == [], k
        pos = {int(v): s for s, v in enumerate(order)}
        viol = [(i, j) for i in range(8) for j in range(8)
                if inst.B0[i, j] != 0 and pos[j] > pos[i]]
        assert (viol == []) == (k >= 2), (k, viol)


@pytest.mark.parametrize("m,n", [(2, 5), (2, 131), (3, 255), (10, 256), (64, 384), (65, 515),
                                 (66, 900), (129, 1290), (260, 700)])
def test_iterative_steps_at_the_edges(api, m, n):
    """Step by step against the precompute and a host refinement, at the edges of the refinement's
    grid (64 columns by 128 rows), of its groups of rows and of the selection's column slices.
    Both sides score (nearly) the same FP32 data: a rounding of the refined data that falls the
    other way moves S by 1e-7 / n at most, so M (m squares of scores of order 1) by less than 1e-6;
    a pick may differ only inside that."""
    rng = np.random.default_rng(100 * m + n)
    D = (rng.laplace(size=(n, m)) @ (np.eye(m) + 0.3 * rng.standard_normal((m, m)) / np.sqrt(m))
         ).astype(np.float32)
    order, margin = (v.cpu().numpy() for v in api.order_iterative(torch.from_numpy(D).cuda()))
    assert sorted(order.tolist()) == list(range(m)) and np.isinf(margin[-1])
    idx = np.arange(m)
    steps = m - 1 if m <= 66 else 40
    for k in range(steps):
        _, _, S, _ = api.pairwise_stats(torch.from_numpy(np.ascontiguousarray(D)).cuda())
        M = (np.minimum(S.cpu().numpy(), 0.0) ** 2).sum(axis=1)
        r = np.sort(M)
        assert abs((r[1] - r[0]) - margin[k]) <= 1e-6, k
        c = int(np.where(idx == order[k])[0][0])
        assert M[c] - r[0] <= 1e-6, k
        X = D.astype(np.float64)
        Z = (X - X.mean(axis=0)) / X.std(axis=0)
        rho = (Z * Z[:, [c]]).mean(axis=0)
        keep = np.arange(len(idx)) != c
        D = (Z - rho * Z[:, [c]])[:, keep].astype(np.float32)
        idx = idx[keep]
