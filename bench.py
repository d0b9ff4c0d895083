"""Benchmark of the heuristic VarLiNGAM hot path on one MI355X.

A step is one whole fit of the path on one synthetic series resident in HBM: VAR(p) fit ->
pairwise entropy precompute -> lookup-only ordering -> B0 / B_tau (all on the GPU, one
stream).  Workload: m = 400 variables, n = 10000 samples, p = 2, Student-t(4) shocks.

Prints ONE JSON line.  value = ordered-pair sample-evaluations per second of the whole step
(m (m - 1) (n - p) per step / step time).  The line also carries the pairwise kernel's own
rate, the stage breakdown, the plain-FP32 and BF16 step times, the roofline of the dominant
kernel (from HIP events recorded on its launch stream during the timed loop), the oracle's CPU
rate on a bounded sample, and sections for the original iterative DirectLiNGAM search on the
same residuals, VAR lag-order selection and adaptive-lasso pruning on the same series, the
bootstrap / rolling-window ensembles, the 256-problem batched workload and the score backward.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "pairwise m²n sample-evals/s + end-to-end fit time vs plain FP32, m=400"
# Transcendental issue rate of gfx950: 256 CUs x 4 SIMDs x 8 lanes/clock (a quarter of the
# 32-lane FP32 rate) x 2.4 GHz; each sample-evaluation needs 3 transcendentals (exp and log
# for log cosh, exp for the Gaussian weight).
TRANS_PEAK = 256 * 32 * 2.4e9
TRANS_PER_EVAL = 3
# HBM bytes per launch of the pairwise kernel, from rocprofv3 --pmc FETCH_SIZE and WRITE_SIZE runs
# of this workload (KiB per dispatch x 1024), each scaled by the counter's reading for a plain
# 256 MiB device copy (FETCH_SIZE reads half of the bytes a copy reads: x2; WRITE_SIZE reads them
# exactly: x1).  Keyed by the SHA-256 of the kernel sources the counters were taken with
# (kernel_source_digest); any other source reports null.
MEASURED_TRAFFIC = {
    # FETCH_SIZE 36368.4 KiB x 2, WRITE_SIZE 8873.9 KiB x 1 per dispatch (24 dispatches)
    "425989bbf3880fd3b9d6af856842e4cadcf01e6409fb3f0c3fa3e785d34f7dc7": 83569308,
}
HEADLINE_PREC = "sliced"
STAGES = ("var_gram", "var_solve", "var_residual", "var_refine", "pairwise_cov",
          "pairwise_prep", "pairwise_moments", "pairwise_combine", "order", "estimate_b")
BATCH_STAGES = ("batch_var", "batch_pairwise", "batch_moments", "batch_order_b")


def kernel_source_digest():
    """SHA-256 over the sources of the pairwise-moment kernel (launcher and device body)."""
    import hashlib
    h = hashlib.sha256()
    for f in ("pairwise.hip", "pairwise_dev.hpp"):
        h.update(open(os.path.join(ROOT, "paper_2409_05500_amd", "csrc", f), "rb").read())
    return h.hexdigest()


def measured_traffic():
    return MEASURED_TRAFFIC.get(kernel_source_digest())


def _oracle_rows(args):
    """Worker of the all-core CPU baseline: rows i0 .. i1 - 1 of the oracle's precompute."""
    from oracle import varlingam as O
    X, i0, i1 = args
    return i0, [O.pair_row(X, i) for i in range(i0, i1)]


def cpu_baseline(seed: int, cols: int) -> dict:
    """The oracle as it stands, on the host cores, before anything touches the GPU (the pool
    is forked): its VAR fit of the workload series, the pairwise precompute of all 400
    residual columns on every host core (processes over row blocks; bit-identical to the
    serial oracle), the same precompute on one core for the first `cols` columns, its ordering
    and its B (normal equations on the residual covariance).  value = all-core precompute
    rate."""
    import multiprocessing as mp
    from oracle import varlingam as O
    import synth
    wl = synth.FINANCE
    X = synth.make_instance(wl, seed).X_parity
    t0 = time.perf_counter()
    M, _, E = O.fit_var(X, wl.p)
    t_var = time.perf_counter() - t0
    Xs = O.standardize_columns(E)
    n_eff, m = E.shape
    cores = max(1, min(16, len(os.sched_getaffinity(0))))
    t0 = time.perf_counter()
    with mp.get_context("fork").Pool(cores) as pool:
        blocks = pool.map(_oracle_rows, [(Xs, i, min(i + 10, m)) for i in range(0, m, 10)])
    rows = [r for _, rs in sorted(blocks, key=lambda b: b[0]) for r in rs]
    _, _, S = O.pairwise_stats(E, rows=rows)
    t_pre = time.perf_counter() - t0
    t0 = time.perf_counter()
    O.pairwise_stats(E[:, :cols])
    t_one = time.perf_counter() - t0
    t0 = time.perf_counter()
    order, _ = O.approx_order(S)
    t_ord = time.perf_counter() - t0
    t0 = time.perf_counter()
    O.estimate_B_cov(O.population_cov(E), order, M)
    t_b = time.perf_counter() - t0
    evals = m * (m - 1) * n_eff
    return {"value": evals / t_pre, "unit": "sample-evals/s", "cores": cores, "kind": "oracle",
            "sample": f"oracle pairwise_stats over all {m} residual columns of the "
                      f"{wl.name} series ({m * (m - 1)} ordered pairs, n_eff={n_eff}), rows "
                      f"split over {cores} host processes, {t_pre:.1f} s wall",
            "single_core": {"value": cols * (cols - 1) * n_eff / t_one, "cores": 1,
                            "sample": f"the first {cols} columns on one core, {t_one:.1f} s"},
            "stage_s": {"var_fit": round(t_var, 3), "precompute": round(t_pre, 3),
                        "ordering": round(t_ord, 3), "estimate_b": round(t_b, 3)}}


def time_steps(fitter, X, steps, torch):
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        fitter.run(X)
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / steps


def bench_batched(api, torch, steps: int, seed: int):
    """The batched workload: 256 problems, m in [20, 200], n in [500, 8000], p = 1, uniform or
    Laplace shocks.  Times one batched fit (one launch per stage for all problems, after the
    chunk-length autotuner) against fitting the problems one after another through the
    single-problem path (preallocated Fitters, no host synchronisation in between)."""
    import synth
    insts = synth.make_batch(seed)
    shapes = [i.X32.shape for i in insts]
    evals = sum(m * (m - 1) * (n - 1) for n, m in shapes)
    dev = torch.device("cuda:0")
    out = {"workload": f"{len(insts)} problems, m in [20, 200], n in [500, 8000], p=1",
           "problems": len(insts), "sample_evals": evals}
    for prec in ("mixed", "fp32"):
        bf = api.BatchFitter(shapes, 1, prec, dev)
        bf.load([i.X32 for i in insts])
        out[f"chunk_len_{prec}"] = bf.autotune()
        hist = {}
        for c in bf.chunk_lens():
            hist[str(c)] = hist.get(str(c), 0) + 1
        out[f"chunk_len_histogram_{prec}"] = hist
        for _ in range(2):
            bf.run()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            bf.run()
        torch.cuda.synchronize()
        out[f"batched_ms_{prec}"] = (time.perf_counter() - t0) / steps * 1e3
        # the same fit captured once in a HIP graph and replayed
        g = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            bf.run()
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            bf.run()
        g.replay()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            g.replay()
        torch.cuda.synchronize()
        out[f"batched_graph_ms_{prec}"] = (time.perf_counter() - t0) / steps * 1e3
        del g
        if prec == "mixed":
            from paper_2409_05500_amd import _lib
            _lib.profile_enable("*")
            bf.run()
            torch.cuda.synchronize()
            out["batched_stage_ms_mixed"] = {st: round(_lib.profile_read(st)[0], 4)
                                             for st in BATCH_STAGES}
            _lib.profile_enable(None)
        if any(bf.check()):
            out[f"batched_status_{prec}"] = bf.check()
        del bf
        Xs = [torch.from_numpy(i.X32).to(dev) for i in insts]
        fitters = [api.Fitter(n, m, 1, prec, dev) for n, m in shapes]
        for f, X in zip(fitters, Xs):
            f.run(X)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(max(1, steps // 5)):
            for f, X in zip(fitters, Xs):
                f.run(X)
        torch.cuda.synchronize()
        out[f"looped_ms_{prec}"] = (time.perf_counter() - t0) / max(1, steps // 5) * 1e3
        del fitters, Xs
        torch.cuda.empty_cache()
    out["batched_sample_evals_per_s_mixed"] = evals / (out["batched_ms_mixed"] / 1e3)
    out["speedup_batched_mixed_vs_looped_fp32"] = out["looped_ms_fp32"] / out["batched_ms_mixed"]
    return out


def bench_certified(api, torch, fit, steps):
    """The certified ordering (near-ties re-decided on FP64 scores) on the fit's residuals and
    scores, at the default score bound: its time against the plain ordering stage, the rows it
    recomputes and whether its order differs from the plain one."""
    E, S0 = fit.E, fit.S
    order, _, _, nref = api.approx_order_certified(E, S0.clone())
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        api.approx_order_certified(E, S0.clone())
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / steps * 1e3
    return {"eps_S": api.CERT_EPS_S, "ms": ms, "rows_refined": nref,
            "same_order_as_plain": bool(torch.equal(order, fit.order))}


def bench_iterative(api, torch, E, stage_ms, steps):
    """The original iterative DirectLiNGAM search (Sec. 3 steps 1-5) on the fit's residuals,
    against the heuristic's precompute + ordering stages of the same fit."""
    n_eff, m = E.shape
    api.order_iterative(E)                          # warm-up (and status check)
    torch.cuda.synchronize()
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    t0.record()
    for _ in range(steps):
        order, _ = api.order_iterative(E)
    t1.record()
    torch.cuda.synchronize()
    it_ms = t0.elapsed_time(t1) / steps
    heur = sum(stage_ms.get(k, 0.0) for k in ("pairwise_cov", "pairwise_prep", "pairwise_moments",
                                              "pairwise_combine", "order"))
    evals = sum(u * (u - 1) for u in range(2, m + 1)) * n_eff
    out = {"m": m, "n_eff": n_eff, "ms": it_ms, "sample_evals": evals,
           "sample_evals_per_s": evals / (it_ms / 1e3),
           "heuristic_precompute_plus_order_ms": heur,
           "speedup_heuristic_vs_iterative": it_ms / heur if heur else None}
    for k in (10,):                                 # hybrid: k exact picks, then the heuristic
        if k >= m - 1:
            continue
        api.order_hybrid(E, k)
        torch.cuda.synchronize()
        t0.record()
        for _ in range(steps):
            api.order_hybrid(E, k)
        t1.record()
        torch.cuda.synchronize()
        out[f"hybrid_k{k}_ms"] = t0.elapsed_time(t1) / steps
    return out


def bench_lag_select(api, torch, X, p_max, steps):
    """VAR lag-order selection over p = 1 .. p_max (one Gram of the p_max design, one fused
    factorisation, scores from the leading blocks), against p_max separate VAR fits."""
    n, m = X.shape
    api.select_lag(X, p_max)                        # warm-up (and status check)
    for p in range(1, p_max + 1):
        api.fit_var(X, p)
    torch.cuda.synchronize()

    def timed(fn):
        t0 = torch.cuda.Event(enable_timing=True)
        t1 = torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(steps):
            fn()
        t1.record()
        torch.cuda.synchronize()
        return t0.elapsed_time(t1) / steps

    # the C entry point with preallocated outputs, so that no call synchronises; one status
    # word, read after the loops
    from paper_2409_05500_amd._lib import lib
    dev = X.device
    outs = [torch.empty(p_max, dtype=torch.float64, device=dev) for _ in range(3)]
    best = torch.empty(2, dtype=torch.int32, device=dev)
    nb = lib.varlingam_select_lag_workspace_bytes(n, m, p_max)
    ws = torch.empty(nb, dtype=torch.uint8, device=dev)
    st = api.DeviceStatus(dev)
    stream = torch.cuda.current_stream(dev).cuda_stream

    def select():
        rc = lib.varlingam_select_lag(X.data_ptr(), n, m, X.stride(0), p_max,
                                      *[o.data_ptr() for o in outs], best.data_ptr(),
                                      ws.data_ptr(), nb, st.ptr, stream)
        assert rc == 0, rc

    sel_ms = timed(select)
    loop_ms = timed(lambda: [api.fit_var(X, p, status=st) for p in range(1, p_max + 1)])
    st.read("lag selection bench")
    _, _, _, (pa, pb) = api.select_lag(X, p_max)
    return {"m": m, "n": n, "p_max": p_max, "ms": sel_ms, "separate_fits_ms": loop_ms,
            "p_aic": pa, "p_bic": pb}


def bench_prune(api, torch, X, fit, steps):
    """Adaptive-lasso pruning of the fit's B0 / B_tau (complete LARS-lasso paths, BIC knot),
    through the C entry point with preallocated outputs (no synchronisation inside the loop).
    Reports the algorithmic bytes of the path arithmetic: per step the inverse of the active
    Gram is read once (to form G_A^{-1} b) and read and written once per 8 steps (the deferred
    rank-one terms applied together): (1 + 2/8) |A|^2 doubles; |A| entries of the covariance
    are read for every inactive column (|A| (d - |A|) doubles)."""
    import numpy as np
    from paper_2409_05500_amd._lib import lib
    n, m = X.shape
    p = fit.B_lags.shape[0]
    dev = X.device
    B0o = torch.empty((m, m), dtype=torch.float64, device=dev)
    Blo = torch.empty((p, m, m), dtype=torch.float64, device=dev)
    info = torch.empty((m, 3), dtype=torch.int32, device=dev)
    nb = lib.varlingam_prune_workspace_bytes(n, m, p, 0)
    ws = torch.empty(nb, dtype=torch.uint8, device=dev)
    st = api.DeviceStatus(dev)
    K = fit.order.to(torch.int32).contiguous()
    B0c, Blc = fit.B0.contiguous(), fit.B_lags.contiguous()
    stream = torch.cuda.current_stream(dev).cuda_stream

    def run():
        rc = lib.varlingam_prune(X.data_ptr(), n, m, X.stride(0), p, K.data_ptr(),
                                 B0c.data_ptr(), Blc.data_ptr(), 0, B0o.data_ptr(),
                                 Blo.data_ptr(), info.data_ptr(), ws.data_ptr(), nb, st.ptr,
                                 stream)
        assert rc == 0, rc

    run()
    torch.cuda.synchronize()
    st.read("prune bench")
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    t0.record()
    for _ in range(steps):
        run()
    t1.record()
    torch.cuda.synchronize()
    st.read("prune bench")
    ms = t0.elapsed_time(t1) / steps
    inf = info.cpu().numpy()
    order = K.cpu().numpy()
    byts = 0
    for pos in range(m):
        # model: the active set grows by one column per step (exact when no column leaves); a step
        # reads the lower triangle of the inverse factor once and the active rows' inactive columns
        d = pos + m * p
        a = np.minimum(np.arange(1, int(inf[order[pos]][0]) + 1, dtype=np.float64), d)
        byts += int(8 * (0.5 * a * a + a * (d - a)).sum())
    nnz0 = int((B0o != 0).sum().item())
    return {"m": m, "n": n, "p": p, "ms": ms, "workspace_bytes": nb,
            "path_steps_total": int(inf[:, 0].sum()), "df_mean": float(inf[:, 2].mean()),
            "B0_nonzeros_before": int((fit.B0 != 0).sum().item()), "B0_nonzeros_after": nnz0,
            "path_bytes": byts, "path_GB_per_s": byts / (ms / 1e3) / 1e9}


def bench_ensembles(api, torch, steps: int, seed: int):
    """Ensembles on the batched path.
    * Residual bootstrap of the m = 100, n = 5000, p = 1 series (Laplace shocks): 100 resamples
      per step -- VAR fit of the series, 100 simulated series, their batched fit, aggregation.
    * Rolling windows of an m = 50, n = 20000, p = 1 series: windows of 2000 rows every 100
      rows (181 windows) per step -- batched fit of the window views, aggregation.
    Buffers are allocated once; a step ends with the aggregation's count read (one sync)."""
    import numpy as np
    import synth
    dev = torch.device("cuda:0")
    out = {}
    wl = synth.MEDIUM
    X = torch.from_numpy(synth.make_instance(wl, seed).X32).to(dev)
    R, T = 100, wl.n - wl.p
    idx = torch.from_numpy(np.random.default_rng(seed).integers(0, T, (R, T)).astype(np.int32))
    idx = idx.to(dev)
    series = torch.empty((R, wl.n, wl.m), dtype=torch.float32, device=dev)
    ef = api.EnsembleFitter(list(series), wl.p, "mixed", 0.05)
    st = api.DeviceStatus(dev)

    def boot():
        M, c, E = api.fit_var(X, wl.p, status=st)
        api.var_simulate(M, c, X[:wl.p].contiguous(), E, idx, out=series, status=st)
        ef.run()
        return ef.aggregate()

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / steps * 1e3

    boot_ms = timed(boot)
    st.read("bootstrap bench")
    assert ef.count == R, ef.check()
    from paper_2409_05500_amd import _lib
    _lib.profile_enable("*")
    boot()
    torch.cuda.synchronize()
    stages = {k: round(_lib.profile_read(k)[0], 4)
              for k in ("var_gram", "var_solve", "var_residual", "simulate", "batch_var",
                        "batch_pairwise", "batch_moments", "batch_order_b")}
    _lib.profile_enable(None)
    out["bootstrap"] = {"workload": wl.name, "resamples": R, "ms": boot_ms,
                        "resamples_per_s": R / (boot_ms / 1e3), "stage_ms": stages}
    inst = synth.make_custom(50, 20000, 1, "laplace", seed, edge_prob=0.1, w_lo=0.1, w_hi=0.5)
    Xr = torch.from_numpy(inst.X32).to(dev)
    starts = list(range(0, 20000 - 2000 + 1, 100))
    er = api.EnsembleFitter([Xr[s: s + 2000] for s in starts], 1, "mixed", 0.05)

    def roll():
        er.run()
        return er.aggregate()

    roll_ms = timed(roll)
    assert er.count == len(starts), er.check()
    out["rolling"] = {"workload": "m50_n20000_p1_laplace, windows of 2000 every 100",
                      "windows": len(starts), "ms": roll_ms,
                      "windows_per_s": len(starts) / (roll_ms / 1e3)}
    return out


def bench_backward(api, _lib, torch, steps: int, seed: int):
    """Gradient of the score matrix, dE = d<G, S(E)>/dE, at m = 1000, n = 50000 (Laplace
    shocks, p = 1): E is the GPU VAR fit's residual matrix, G a seeded N(0, 1) cotangent.
    Algorithmic transcendentals: dL/du of both directions of every unordered pair and sample
    (tanh: exp + reciprocal; Gaussian: exp) = 3 m (m - 1) n_eff; the pair-tile kernel evaluates
    each unordered pair once per sample (its padding to 64-variable blocks aside)."""
    import numpy as np
    import synth
    wl = synth.LARGE
    inst = synth.make_instance(wl, seed)
    dev = torch.device("cuda:0")
    _, _, E = api.fit_var(torch.from_numpy(inst.X32).to(dev), wl.p, "mixed")
    m, n_eff = E.shape[1], E.shape[0]
    G = torch.from_numpy(np.random.default_rng(seed + 1).normal(size=(m, m))).to(dev)
    for _ in range(2):
        api.pairwise_stats_backward(E, G)
    torch.cuda.synchronize()
    _lib.profile_enable("pairwise_cov,pairwise_prep,pairwise_moments,pairwise_combine,"
                        "backward_prep,backward_pairs,backward_reduce,backward_tail")
    t0 = time.perf_counter()
    for _ in range(steps):
        api.pairwise_stats_backward(E, G)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / steps
    st = {k: _lib.profile_read(k) for k in ("pairwise_cov", "pairwise_prep", "pairwise_moments",
                                            "pairwise_combine", "backward_prep",
                                            "backward_pairs", "backward_reduce",
                                            "backward_tail")}
    _lib.profile_enable(None)
    # with the forward's saved statistics (the autograd path): no recompute of the moments
    saved = api.pairwise_stats_save(E)[4]
    api.pairwise_stats_backward(E, G, saved=saved)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        api.pairwise_stats_backward(E, G, saved=saved)
    torch.cuda.synchronize()
    dt_saved = (time.perf_counter() - t0) / steps
    # per backward call (the pair pass runs in several launches, one per sample window)
    ms = {k: v[0] / steps for k, v in st.items()}
    pairs_s = ms["backward_pairs"] / 1e3
    alg = 3.0 * m * (m - 1) * n_eff
    return {"workload": f"{wl.name}, residuals of the GPU VAR fit, N(0,1) cotangent",
            "m": m, "n_eff": n_eff, "backward_ms": dt * 1e3,
            "backward_with_saved_ms": dt_saved * 1e3,
            "forward_recompute_ms": sum(ms[k] for k in ("pairwise_cov", "pairwise_prep",
                                                        "pairwise_moments", "pairwise_combine")),
            "stage_ms": {k: round(v, 4) for k, v in ms.items()},
            "pair_kernel_roofline": {"kernel": "bwd_tile_kernel", "bound": "alu",
                                     "achieved": alg / pairs_s / 1e12,
                                     "peak": TRANS_PEAK / 1e12, "unit": "Ttrans/s",
                                     "frac": alg / pairs_s / TRANS_PEAK}}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-cols", type=int, default=100,
                    help="columns of the single-core oracle sample")
    ap.add_argument("--no-batch", action="store_true",
                    help="skip the batched-workload section (256 uneven problems)")
    ap.add_argument("--no-backward", action="store_true",
                    help="skip the score-gradient section (m = 1000, n = 50000)")
    ap.add_argument("--no-iterative", action="store_true",
                    help="skip the original iterative DirectLiNGAM search on the fit's residuals")
    ap.add_argument("--no-lag-select", action="store_true",
                    help="skip the VAR lag-order selection section")
    ap.add_argument("--no-prune", action="store_true",
                    help="skip the adaptive-lasso pruning section")
    ap.add_argument("--no-ensembles", action="store_true",
                    help="skip the bootstrap / rolling-window section")
    ap.add_argument("--only", choices=("batch", "backward", "prune", "ensembles"), default=None,
                    help="profiling runs: run just one extra section and print its JSON")
    ap.add_argument("--copy-calibration-mb", type=int, default=0,
                    help="run one device-to-device copy of this many MiB first (a plain copy "
                         "kernel of known traffic, for calibrating hardware byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the library has no "
              "multi-GPU path", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    # the oracle's CPU baseline runs first: its worker processes are forked before anything
    # has initialised the GPU (rank 0, one GPU)
    cpu = None
    if not args.only and not args.no_cpu_baseline:
        cpu = cpu_baseline(args.seed, args.cpu_cols)
        print("bench: cpu baseline done", file=sys.stderr, flush=True)
    import torch
    import synth
    from paper_2409_05500_amd import api, _lib

    if args.only == "batch":
        print(json.dumps({"batched": bench_batched(api, torch, max(3, args.steps // 2),
                                                   args.seed)}), flush=True)
        return
    if args.only == "backward":
        print(json.dumps({"backward": bench_backward(api, _lib, torch, max(3, args.steps // 2),
                                                     args.seed)}), flush=True)
        return
    if args.only == "ensembles":
        print(json.dumps({"ensembles": bench_ensembles(api, torch, max(3, args.steps // 2),
                                                       args.seed)}), flush=True)
        return
    if args.only == "prune":
        wl = synth.FINANCE
        X = torch.from_numpy(synth.make_instance(wl, args.seed).X32).to("cuda:0")
        fit = api.Fitter(wl.n, wl.m, wl.p, "mixed", X.device)
        fit.run(X)
        print(json.dumps({"prune": bench_prune(api, torch, X, fit, max(2, args.steps // 4))}),
              flush=True)
        return

    wl = synth.FINANCE
    inst = synth.make_instance(wl, args.seed)
    dev = torch.device("cuda:0")
    X = torch.from_numpy(inst.X32).to(dev)
    n, m, p = wl.n, wl.m, wl.p
    n_eff = n - p
    evals = m * (m - 1) * n_eff

    if args.copy_calibration_mb:
        src = torch.empty(args.copy_calibration_mb << 18, dtype=torch.float32, device=dev)
        src.fill_(1.0)
        dst = src.clone()          # reads and writes copy_calibration_mb MiB once
        torch.cuda.synchronize()
        del src, dst

    # the headline: the fastest form that meets the FP64-grade accuracy bar (the int8-slice
    # products, SLICED: the same config-2 parity tests as MIXED)
    fit = api.Fitter(n, m, p, HEADLINE_PREC, dev)
    for _ in range(args.warmup):
        fit.run(X)
    fit.check()
    _lib.profile_enable("pairwise_moments")
    step_s = time_steps(fit, X, args.steps, torch)
    kms, kcount = _lib.profile_read("pairwise_moments")
    _lib.profile_enable(None)
    fit.check()
    k_s = kms / kcount / 1e3

    # stage breakdown (separate pass, every stage bracketed by events)
    _lib.profile_enable("*")
    time_steps(fit, X, max(3, args.steps // 4), torch)
    stage_ms = {}
    for st in STAGES:
        ms, cnt = _lib.profile_read(st)
        if cnt:
            stage_ms[st] = round(ms / cnt, 4)
    _lib.profile_enable(None)

    # the plain FP32 form on the same input, and the FP32 Gram with one FP64 refinement step
    # (the cheapest form on the FP32 Gram that reaches the mixed mode's accuracy)
    f32 = api.Fitter(n, m, p, "fp32", dev)
    for _ in range(args.warmup):
        f32.run(X)
    fp32_s = time_steps(f32, X, args.steps, torch)
    f32r = api.Fitter(n, m, p, "fp32_refined", dev)
    for _ in range(args.warmup):
        f32r.run(X)
    fp32r_s = time_steps(f32r, X, args.steps, torch)
    f32r.check()

    # MIXED (the FP64-MFMA products) on the same input, and its stages
    fm = api.Fitter(n, m, p, "mixed", dev)
    for _ in range(args.warmup):
        fm.run(X)
    mixed_s = time_steps(fm, X, args.steps, torch)
    fm.check()
    _lib.profile_enable("*")
    time_steps(fm, X, max(3, args.steps // 4), torch)
    mixed_stage_ms = {}
    for st in STAGES:
        ms, cnt = _lib.profile_read(st)
        if cnt:
            mixed_stage_ms[st] = round(ms / cnt, 4)
    _lib.profile_enable(None)

    # the BF16-Gram form with FP64 refinement, its VAR stages, and its distance from MIXED
    bf = api.Fitter(n, m, p, "bf16", dev)
    for _ in range(args.warmup):
        bf.run(X)
    bf16_s = time_steps(bf, X, args.steps, torch)
    bf.check()
    _lib.profile_enable("*")
    time_steps(bf, X, 3, torch)
    bf16_stage_ms = {}
    for st in ("var_gram", "var_solve", "var_refine", "var_residual"):
        ms, cnt = _lib.profile_read(st)
        if cnt:
            bf16_stage_ms[st] = round(ms / cnt, 4)
    _lib.profile_enable(None)

    # MIXED with the compensated moment sums (VL_PAIRWISE_COMPENSATED): whole fit and its
    # moment kernel
    fc = api.Fitter(n, m, p, "mixed", dev, compensated=True)
    for _ in range(args.warmup):
        fc.run(X)
    _lib.profile_enable("pairwise_moments")
    comp_s = time_steps(fc, X, args.steps, torch)
    cms, ccount = _lib.profile_read("pairwise_moments")
    _lib.profile_enable(None)
    fc.check()

    def b_rel(a, b):
        return float((a - b).abs().max() / max(float(b.abs().max()), 1e-2))
    def dist(o):
        return {"B0_rel": b_rel(o.B0, fm.B0), "B_lags_rel": b_rel(o.B_lags, fm.B_lags),
                "same_order": bool(torch.equal(o.order, fm.order))}
    bf16_dev = dist(bf)
    modes_vs_mixed = {"fp32": dist(f32), "fp32_refined": dist(f32r), "bf16": bf16_dev,
                      "sliced": dist(fit),
                      "mixed_compensated": dict(dist(fc), S_max_abs_diff=float(
                          (fc.S - fm.S).abs().max()))}

    # measured issue rates of this part (the roofline denominators' check)
    rates = api.probe_rates(dev)
    achieved = TRANS_PER_EVAL * evals / k_s
    # transcendentals the kernel issues per sample-eval: two exp2, and one log per 64 samples
    # of a lane (the running product of log cosh)
    issued = (2.0 + 1.0 / 64.0) * evals / k_s
    out = {
        "metric": METRIC,
        "value": evals / step_s,
        "unit": "sample-evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": step_s * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "m": m, "n": n, "p": p, "noise": "student-t(4)",
                   "precision": HEADLINE_PREC, "seed": args.seed},
        "roofline": {"kernel": "pairwise_moments_kernel", "bound": "alu",
                     "achieved": achieved / 1e12, "peak": TRANS_PEAK / 1e12,
                     "unit": "Ttrans/s", "frac": achieved / TRANS_PEAK,
                     "traffic": measured_traffic(),
                     "counting": "algorithmic: 3 transcendentals per sample-eval",
                     "issued_achieved": issued / 1e12, "issued_frac": issued / TRANS_PEAK,
                     "peak_measured": rates["exp2_per_s"] / 1e12,
                     "frac_of_measured": achieved / rates["exp2_per_s"]},
        "probe_rates": {"exp2_per_s": rates["exp2_per_s"],
                        "fp32_fma_tflops": rates["fp32_fma_flops"] / 1e12,
                        "fp64_mfma_tflops": rates["fp64_mfma_flops"] / 1e12},
        "pairwise_kernel_ms": k_s * 1e3,
        "pairwise_kernel_sample_evals_per_s": evals / k_s,
        "sample_evals_per_step": evals,
        "fit_ms_sliced": step_s * 1e3,
        "fit_ms_mixed": mixed_s * 1e3,
        "fit_ms_fp32": fp32_s * 1e3,
        "fit_ms_fp32_refined": fp32r_s * 1e3,
        "fit_ms_bf16": bf16_s * 1e3,
        "fit_ms_mixed_compensated": comp_s * 1e3,
        "mixed_stage_ms": mixed_stage_ms,
        "pairwise_kernel_ms_compensated": cms / ccount,
        "bf16_stage_ms": bf16_stage_ms,
        "bf16_vs_mixed": bf16_dev,
        "modes_vs_mixed": modes_vs_mixed,
        "stage_ms": stage_ms,
    }
    def progress(msg):
        print(f"bench: {msg}", file=sys.stderr, flush=True)

    progress("fit timings done")
    out["certified_order"] = bench_certified(api, torch, fit, 5)
    progress("certified ordering done")
    if not args.no_iterative:
        out["iterative"] = bench_iterative(api, torch, fit.E, stage_ms, 3)
    progress("iterative done")
    if not args.no_lag_select:
        out["lag_select"] = bench_lag_select(api, torch, X, 2 * p, 5)
    progress("lag selection done")
    if not args.no_prune:
        out["prune"] = bench_prune(api, torch, X, fit, 2)
    progress("pruning done")
    if not args.no_ensembles:
        out["ensembles"] = bench_ensembles(api, torch, 3, args.seed)
    progress("ensembles done")
    if not args.no_batch:
        out["batched"] = bench_batched(api, torch, max(3, args.steps // 2), args.seed)
    progress("batched done")
    if not args.no_backward:
        out["backward"] = bench_backward(api, _lib, torch, 3, args.seed)
    progress("backward done")
    if cpu is not None:
        out["cpu_baseline"] = cpu
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
