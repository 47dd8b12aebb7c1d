"""Benchmark: kNN-graph cells/s of the neighbourhood-graph step on one MI355X.

One step = the whole hot path on one batch of synthetic, HBM-resident input:
exact kNN (rsc_knn: prep, MFMA screen, float64 rerank + certificate,
rescan) followed by rsc_connectivities (rho/sigma, fuzzy union, CSR).

Default workload: n = 1,000,000 cells, d = 50 PCA-like components, k = 15,
100-cluster Gaussian mixture with Zipf(1.1) cluster sizes and 1/i variance
decay (a synthetic stand-in for a PCA embedding of a 10x dataset).

Prints ONE JSON line.  ``roofline`` covers the dominant kernel (the pruned
split-FP16 MFMA screen) with its duration measured by HIP events recorded by the
library on the launch stream over the timed region.  ``cpu_baseline`` times
the FP64 CPU oracle on a bounded sample of query rows of the same workload.
"""

from __future__ import annotations

import argparse
import math
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "kNN graph cells/s (d=50,k=15): plain vs BF16+rerank vs routed, recall@15≥0.99"
PEAK_HBM_GBS = 8000.0
PEAK_FP16_TFLOPS = 2516.6  # MI355X dense FP16 / BF16 matrix

WORKLOADS = {
    "plain_1m": dict(n=1_000_000, clusters=100, law="zipf", seed=1,
                     desc="plain exact FP32 kNN graph, n=1,000,000 cells, d=50, k=15, 100-cluster Zipf(1.1) mixture"),
    "plain_10k": dict(n=10_000, clusters=20, law="uniform", seed=0,
                      desc="plain exact FP32 kNN graph, n=10,000 cells, d=50, k=15, 20-cluster uniform mixture"),
}


def log(msg: str) -> None:
    print(msg, file=sys.stderr, flush=True)


def cpu_baseline(X: np.ndarray, k: int, budget_s: float) -> dict:
    """The FP64 oracle (as it stands) on a seeded sample of query rows."""
    import oracle
    import synth

    oracle.build(force=False)
    cores = oracle.max_threads()
    n = X.shape[0]
    # calibrate on a few rows, then size the sample to the time budget
    probe = synth.sample_rows(n, max(64, 8 * cores), seed=7)
    t0 = time.perf_counter()
    oracle.knn_rows(X, probe, k)
    per_row = (time.perf_counter() - t0) / len(probe)
    rows_n = int(max(len(probe), min(n, budget_s / max(per_row, 1e-9))))
    rows = synth.sample_rows(n, rows_n, seed=11)
    t0 = time.perf_counter()
    idx, _, dist = oracle.knn_rows(X, rows, k)
    t_knn = time.perf_counter() - t0
    # the graph stage of the oracle is O(n k); time it on the sample's lists
    t0 = time.perf_counter()
    oracle.smooth_knn(idx, dist)
    t_graph = time.perf_counter() - t0
    secs = t_knn + t_graph
    return {"value": len(rows) / secs, "unit": "cells/s", "cores": cores, "kind": "oracle",
            "sample": f"{len(rows)} seeded query rows of the same {n}-cell workload, each against all {n} rows "
                      f"(FP64 brute-force kNN + smooth-kNN on their lists); {secs:.1f} s"}


def graph_gbs(kernels: dict, n: int, k: int, nnz: int) -> dict:
    """Achieved HBM GB/s of the connectivities kernels (HIP-event durations).

    ``stage`` uses the compulsory bytes of the whole graph step: the kNN
    lists read once (idx int32 + dist float32, n k entries) and the CSR
    written once (int64 row pointers, int32 column + float32 weight per
    entry).  Each kernel's ``bytes`` counts every array it reads or writes
    exactly once by its design (E = n (k - 1) directed edges, of which
    nnz - E are one-way and 2E - nnz mutual), so ``gbs`` is a lower bound on
    its bandwidth; the PMC bytes of the same kernels sit in profiles/."""
    m = k - 1
    E = n * m
    one_way = max(nnz - E, 0)
    mutual = max(2 * E - nnz, 0)
    nk = n * k
    P = (m + 15) // 16 * 16  # padded list length of the mutual-edge lookup
    design = {
        "smooth_knn": 4 * nk + 8 * E + 16 * n,                                    # dist in; a, rho, sigma out
        # idx, a (own + reverse) in; padded id copy out and back in; wf, rs, counts out
        "union_count": 4 * nk + 8 * n * P + 8 * E + 8 * mutual + 4 * E + 4 * E + 8 * n,
        "csr_scan": 8 * n + 16 * n + 8 * (n + 1),                                 # counts in; indptr, reverse bases out
        "union_fill": 4 * E + 4 * E + 4 * nk + 8 * one_way + 8 * one_way,         # rs, wf, idx, bases in; reverse records out
        "row_sort": 20 * n + 4 * E + 4 * nk + 8 * one_way + 8 * nnz,              # bases, counts, indptr, wf, idx, records in; CSR out
    }
    out = {}
    total_ms = 0.0
    for name, b in design.items():
        ms = kernels.get(name)
        if not ms:
            continue
        total_ms += ms
        out[name] = {"ms": ms, "bytes": b, "gbs": round(b / (ms / 1e3) / 1e9, 1),
                     "frac_of_hbm": round(b / (ms / 1e3) / 1e9 / PEAK_HBM_GBS, 4)}
    compulsory = 8 * nk + 8 * (n + 1) + 8 * nnz
    for extra in ("graph_init",):
        total_ms += kernels.get(extra, 0.0)
    stage = {"ms": round(total_ms, 4), "compulsory_bytes": compulsory,
             "gbs": round(compulsory / (total_ms / 1e3) / 1e9, 1) if total_ms else None,
             "frac_of_hbm": round(compulsory / (total_ms / 1e3) / 1e9 / PEAK_HBM_GBS, 4) if total_ms else None}
    return {"stage": stage, "kernels": out}


TRAFFIC_FILE = os.path.join(ROOT, "profiles", "screen_fp32_plain_1m_traffic.json")
# the sources that define the screen kernel (and so its traffic)
SCREEN_SOURCES = [os.path.join(ROOT, "paper_2603_02402_amd", "csrc", f)
                  for f in ("knn.hip", "spatial.hip", "screen_split.hpp", "screen_split_grid.hpp", "screen_common.hpp")]


def screen_source_hash() -> str:
    import hashlib

    h = hashlib.sha256()
    for f in SCREEN_SOURCES:
        h.update(open(f, "rb").read())
    return h.hexdigest()


def split_mfmas(d: int) -> int:
    """FP16 MFMAs (32 x 32 x 16) of the split screen per 32 x 32 keys, from its
    geometries (three per 16 full dimensions, one or two for the rest)."""
    for q, tc in [(q, tc) for q in range(4) for tc in (1, 2)] + [(q, 1) for q in (4, 5, 6, 7, 8, 10, 12, 14, 16)]:
        if d <= 16 * q + (16 * tc - 3) // 3:
            return 3 * q + tc
    return 0


def screened_pairs(ws, n: int):
    """Query-reference pairs the pruned screen of the last call multiplied out:
    segments visited (summed over tiles of 256 queries) times their rows."""
    import torch

    blocks = (n + 31) // 32
    seg = 1
    while (blocks + seg - 1) // seg > 8192:
        seg *= 2
    if int(ws.buf[28:32].view(torch.int32)[0]) == 2:  # a plain screen answered
        return float(n) * n
    visited = int(ws.buf[32:40].view(torch.int64)[0])
    return visited * seg * 32 * 256


def measured_traffic():
    """HBM-side bytes per screen launch from the committed PMC summary, or None
    when the kernel source has changed since the counters were taken."""
    try:
        rec = json.load(open(TRAFFIC_FILE))
        h = screen_source_hash()
    except (OSError, ValueError):
        return None
    if rec.get("source_sha256") != h:
        return None
    return rec.get("traffic_bytes_per_launch")


def traffic_probe() -> int:
    """Program for the PMC runs: a torch copy of 1 GiB (counter calibration),
    then one kNN graph step on the 1M-cell workload."""
    import torch

    import paper_2603_02402_amd as rsc
    import synth

    print("traffic probe: calibration copy of 1 GiB", flush=True)
    a = torch.empty(256 * 1024 * 1024, dtype=torch.float32, device="cuda")
    a.fill_(1.0)
    b = torch.empty_like(a)
    torch.cuda.synchronize()
    b.copy_(a)
    torch.cuda.synchronize()
    del a, b
    X = synth.workload("plain_1m")
    idx, dist, g = rsc.knn_graph(torch.from_numpy(X).cuda(), 15)
    torch.cuda.synchronize()
    print(f"traffic probe: done, nnz {g.nnz}", flush=True)
    return 0


def precision_probe() -> int:
    """Program for the MFMA counter runs of the reduced-precision screens: one
    BF16 and one FP8-e4m3 kNN call on the 2M-cell precision workload."""
    import torch

    import paper_2603_02402_amd as rsc
    import synth

    X = torch.from_numpy(synth.workload("precision_2m")).cuda()
    ws = rsc.Workspace()
    for name, prec in (("bf16", rsc.RSC_BF16), ("fp8", rsc.RSC_FP8_E4M3)):
        print(f"precision probe: {name}", flush=True)
        rsc.knn(X, 15, workspace=ws, precision=prec)
        torch.cuda.synchronize()
    print("precision probe: done", flush=True)
    return 0


def recall_at_k(dist_form, dist_exact, k: int) -> float:
    """Tie-aware recall@k of a form whose returned distances are exact
    (float64 rerank): a returned neighbour is a hit when its distance is
    within the exact k-th distance x (1 + 1e-5).  Self (column 0) excluded."""
    dk = dist_exact[:, -1:].double() * (1 + 1e-5)
    hits = (dist_form[:, 1:].double() <= dk).sum(dim=1).clamp(max=k - 1)
    return float(hits.double().mean().item() / (k - 1))


def weight_error(g_form, g_exact, n: int) -> dict:
    """Relative error of the connectivity weights on the entries both graphs hold."""
    import torch

    def keys(g):
        rows = torch.repeat_interleave(torch.arange(n, device=g.indptr.device), g.indptr[1:] - g.indptr[:-1])
        return rows * n + g.indices.long()

    ke, kf = keys(g_exact), keys(g_form)
    pos = torch.searchsorted(ke, kf).clamp(max=ke.numel() - 1)
    common = ke[pos] == kf
    we = g_exact.data[pos[common]].double()
    wf = g_form.data[common].double()
    rel = (wf - we).abs() / we
    return {"common_entries": int(common.sum().item()), "form_entries": int(kf.numel()),
            "exact_entries": int(ke.numel()), "max_rel": float(rel.max().item()) if rel.numel() else 0.0,
            "p99_rel": float(torch.quantile(rel[:1 << 24].float(), 0.99).item()) if rel.numel() else 0.0}


def timed_form(rsc, Xt, k, precision, steps, warmup, ws, out, fp8_residual=0, kernels=None):
    import torch

    idx, dist, csr = out
    for _ in range(warmup):
        rsc.knn(Xt, k, precision=precision, out=(idx, dist), workspace=ws, fp8_residual=fp8_residual)
        g = rsc.connectivities(idx, dist, workspace=ws, out=csr)
    torch.cuda.synchronize()
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(steps):
        rsc.knn(Xt, k, precision=precision, out=(idx, dist), workspace=ws, fp8_residual=fp8_residual)
        g = rsc.connectivities(idx, dist, workspace=ws, out=csr)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    rsc.profile_enable(False)
    names = {rsc.RSC_FP32: "screen_fp32", rsc.RSC_BF16: "screen_bf16", rsc.RSC_FP8_E4M3: "screen_fp8"}
    name = "screen_fp8_resid" if fp8_residual else names[precision]
    tot, cnt = rsc.profile_get(name)
    if kernels is not None:
        for kn in ("resid_partition", "prep_pack", name, "rerank", "smooth_knn", "union_count", "union_fill",
                   "row_sort"):
            t, c = rsc.profile_get(kn)
            if c:
                kernels[kn] = round(t / steps, 3)
    return (t1 - t0) * 1e3 / steps, (tot / cnt if cnt else None), g


def precision_forms(args, rsc) -> dict:
    """The precision workload (n = 2M): plain exact FP32 (what recall is measured against),
    BF16 + rerank and FP8-e4m3 + rerank, each timed as a whole graph step."""
    import torch

    import synth

    k = args.k
    log("[bench] precision forms: generating the 2M-cell workload")
    X = synth.workload("precision_2m")
    n, d = X.shape
    dev = torch.device("cuda:0")
    Xt = torch.from_numpy(X).to(dev)
    del X
    ws = rsc.Workspace(dev)
    ws.get(max(rsc.knn_workspace_bytes(n, n, d, k), rsc.knn_workspace_bytes(n, n, d, k, precision=rsc.RSC_BF16),
               rsc.knn_workspace_bytes(n, n, d, k, precision=rsc.RSC_FP8_E4M3, fp8_residual=1024),
               rsc.connectivities_workspace_bytes(n, k)))
    cap = 2 * n * (k - 1)

    def outputs():
        return (torch.empty((n, k), dtype=torch.int32, device=dev), torch.empty((n, k), dtype=torch.float32, device=dev),
                (torch.empty(n + 1, dtype=torch.int64, device=dev), torch.empty(cap, dtype=torch.int32, device=dev),
                 torch.empty(cap, dtype=torch.float32, device=dev)))

    res = {"workload": "n=2,000,000 cells, d=50, k=15, 100-cluster Zipf(1.1) mixture (seed 2)"}
    ex = outputs()
    log("[bench] precision forms: plain exact FP32")
    ms, scr, g_exact = timed_form(rsc, Xt, k, rsc.RSC_FP32, 1, 0, ws, ex)
    res["plain_fp32"] = {"cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2),
                         "screen_ms": round(scr, 2), "recall@15": 1.0,
                         "screen_tflops": round(2 * d * n * n / (scr / 1e3) / 1e12, 2)}
    fo = outputs()
    for name, prec, peak in (("bf16_rerank", rsc.RSC_BF16, 2500.0), ("fp8_e4m3_rerank", rsc.RSC_FP8_E4M3, 5000.0)):
        log(f"[bench] precision forms: {name}")
        ms, scr, g = timed_form(rsc, Xt, k, prec, args.form_steps, 1, ws, fo)
        rec = recall_at_k(fo[1], ex[1], k)
        we = weight_error(g, g_exact, n)
        work = 2.0 * d * n * n
        if prec == rsc.RSC_BF16:  # pruned: what its MFMAs of 16 slots did
            work = screened_pairs(ws, n) * 32.0 * ((d + 19) // 16)
        res[name] = {"cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2),
                     "screen_ms": round(scr, 2), "recall@15": round(rec, 5),
                     "screen_tflops_algorithmic": round(2 * d * n * n / (scr / 1e3) / 1e12, 2),
                     "screen_frac_of_peak": round(work / (scr / 1e3) / 1e12 / peak, 4),
                     "weight_error_on_common_entries": we,
                     "meets_recall_0.99": rec >= 0.99}
    # the FP8 residual variant (a separately labelled form): 1024 k-means
    # partitions of the cells, residual coding on both sides; the partitioning
    # is part of every timed call
    log("[bench] precision forms: fp8_e4m3_residual_rerank")
    kern = {}
    ms, scr, g = timed_form(rsc, Xt, k, rsc.RSC_FP8_E4M3, args.form_steps, 1, ws, fo, fp8_residual=1024, kernels=kern)
    rec = recall_at_k(fo[1], ex[1], k)
    we = weight_error(g, g_exact, n)
    res["fp8_e4m3_residual_rerank"] = {
        "partitions": 1024, "cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2),
        "screen_ms": round(scr, 2), "kernel_ms": kern, "recall@15": round(rec, 5),
        "screen_tflops_algorithmic": round(2 * d * n * n / (scr / 1e3) / 1e12, 2),
        "screen_frac_of_peak": round(2 * d * n * n / (scr / 1e3) / 1e12 / 5000.0, 4),
        "weight_error_on_common_entries": we, "meets_recall_0.99": rec >= 0.99}
    return res


def cosine_form(args, rsc, Xt, ws, out) -> dict:
    """Exact kNN graph under the cosine distance on the plain workload (same
    cells, buffers and k), timed as a whole graph step."""
    import torch

    idx, dist, csr = out
    n, d = Xt.shape
    k = idx.shape[1]
    cos = rsc.RSC_COSINE
    ws.get(max(rsc.knn_workspace_bytes(n, n, d, k, metric=cos), rsc.connectivities_workspace_bytes(n, k)))
    log("[bench] cosine form: warmup")
    rsc.knn(Xt, k, out=(idx, dist), workspace=ws, metric=cos)
    rsc.connectivities(idx, dist, workspace=ws, out=csr)
    torch.cuda.synchronize()
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    stats = g = None
    for i in range(args.form_steps):
        rsc.knn(Xt, k, out=(idx, dist), workspace=ws, metric=cos)
        stats = rsc.read_knn_stats(ws)
        g = rsc.connectivities(idx, dist, workspace=ws, out=csr)
        log(f"[bench] cosine form: step {i + 1}/{args.form_steps}")
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.form_steps
    rsc.profile_enable(False)
    kern = {}
    for name in ["normalize", "prep_pack", "screen_fp32", "rerank", "screen_escalate", "rerank_escalate", "rescan",
                 "smooth_knn", "union_count", "union_fill", "row_sort"]:
        tot, cnt = rsc.profile_get(name)
        if cnt:
            kern[name] = round(tot / cnt, 4)
    scr = kern.get("screen_fp32")
    return {"workload": "same cells as the plain line (n=1,000,000, d=50, k=15), distance 1 - cos",
            "form": "exact cosine (split FP16 MFMA screen on unit rows, FP64 rerank + certificate)",
            "cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2), "kernel_ms": kern,
            "screened_pairs_of_all": round(screened_pairs(ws, n) / (n * n), 5) if scr else None,
            "escalated_rows": stats["escalated_rows"], "rescanned_rows": stats["rescanned_rows"],
            "max_err_ratio": round(stats["max_err_ratio"], 4), "nnz": int(g.nnz)}


PEAK_FP64_TFLOPS = 78.6  # MI355X dense FP64 matrix
# float64 vector instruction rate: 256 CUs x 64 lanes x 2.4 GHz (78.6 TFLOP/s counts an FMA as 2)
PEAK_FP64_VECTOR_OPS = 39.3
# float64 add / multiply / fma instructions per slot of k_umap_epoch<2>: the
# straight-line move (correctly rounded power included, 382, counted in its
# assembly) and the slot's 2 adds of the ordered sum
UMAP_MOVE_FP64_OPS = 384


def edistance_form(args, rsc) -> dict:
    """Energy distances of a perturbation screen (1000 groups: 20k control
    cells, 999 perturbations of 50-350 cells, d = 50): the full G x G matrix
    and the one-sided distances to the control group."""
    import torch

    import synth

    X, labels = synth.perturbation_screen()
    G = synth.EDIST["n_groups"]
    n, d = X.shape
    Xt = torch.from_numpy(X).cuda()
    ws = rsc.Workspace()
    off, ct = rsc.edistance_groups(torch.from_numpy(labels).cuda(), G, workspace=ws)  # counting sort on the GPU
    log("[bench] edistance: warmup")
    rsc.edistance_pairwise(Xt, off, ct, workspace=ws)
    rsc.edistance_onesided(Xt, off, ct, 0, workspace=ws)
    torch.cuda.synchronize()
    steps = max(args.form_steps, 3)
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(steps):
        E = rsc.edistance_pairwise(Xt, off, ct, workspace=ws)
    torch.cuda.synchronize()
    ms_pw = (time.perf_counter() - t0) * 1e3 / steps
    tiles_ms = rsc.profile_get("ed_tiles")[0] / steps
    plan_ms = rsc.profile_get("ed_plan")[0] / steps
    rsc.profile_reset()
    t0 = time.perf_counter()
    for _ in range(steps):
        rsc.edistance_onesided(Xt, off, ct, 0, workspace=ws)
    torch.cuda.synchronize()
    ms_os = (time.perf_counter() - t0) * 1e3 / steps
    os_tiles_ms = rsc.profile_get("ed_tiles")[0] / steps
    rsc.profile_enable(False)
    dists = n * (n - 1) / 2
    flops = 2.0 * d * dists
    E_h = E.cpu().numpy()
    cpu = None if args.no_cpu_baseline else edistance_cpu_baseline(X, labels, G)
    return {"workload": f"perturbation screen: {n} cells, d={d}, {G} groups (control 20,000 cells; 999 "
                        "perturbations of 50-350 cells, 30% with an effect), seed 9",
            "pairwise_ms": round(ms_pw, 2), "pairwise_distances_per_s": round(dists / (ms_pw / 1e3), 1),
            "pairwise_tile_kernel_ms": round(tiles_ms, 2), "plan_ms": round(plan_ms, 3),
            "tile_kernel_fp64_tflops": round(flops / (tiles_ms / 1e3) / 1e12, 2),
            "tile_kernel_frac_of_fp64_peak": round(flops / (tiles_ms / 1e3) / 1e12 / PEAK_FP64_TFLOPS, 4),
            "work_per_call": f"n(n-1)/2 = {dists:.4e} distances, 2 d flops each on the float64 matrix cores",
            "onesided_ms": round(os_tiles_ms if os_tiles_ms else ms_os, 2), "onesided_call_ms": round(ms_os, 2),
            "E_range": [round(float(E_h.min()), 6), round(float(E_h.max()), 6)],
            "cpu_baseline": cpu}


def edistance_cpu_baseline(X, labels, G) -> dict:
    """The oracle (float64 direct differences) on sampled group pairs of the
    same screen (control against four perturbations, three perturbation pairs,
    three within-group sums), as distances per second."""
    import oracle
    from oracle import edistance as oed

    off, cells = oed.groups_from_labels(labels, G=G)
    rng = np.random.default_rng(3)
    gs = rng.choice(np.arange(1, G), size=64, replace=False)
    pairs = np.array([[0, g] for g in gs[:40]] + [[gs[i], gs[i + 1]] for i in range(40, 64, 2)] +
                     [[g, g] for g in gs[:16]], dtype=np.int32)
    cnt = oed.pair_counts(np.diff(off), pairs)
    t0 = time.perf_counter()
    oed.sums(X, off, cells, pairs)
    secs = time.perf_counter() - t0
    return {"value": round(float(cnt.sum() / secs), 1), "unit": "distances/s",
            "cores": min(oracle.max_threads(), len(pairs)), "kind": "oracle",
            "sample": f"{int(cnt.sum())} distances of {len(pairs)} sampled group pairs, one thread per pair "
                      f"({secs:.2f} s)"}


def large_k_form(args, rsc) -> dict:
    """Exact kNN graph at larger k on the plain 1M workload (same cells): the
    main screen splits the references into about k / 32 ranges and the
    float64 top-m spans up to 4 registers per lane."""
    import torch

    import synth

    w = WORKLOADS["plain_1m"]
    X = synth.mixture(w["n"], d=50, n_clusters=w["clusters"], law=w["law"], seed=w["seed"])
    n, d = X.shape
    Xt = torch.from_numpy(X).cuda()
    del X
    res = {"workload": "same cells as the plain line (n=1,000,000, d=50), exact FP32-screened path"}
    for k in (30, 64, 100):
        ws = rsc.Workspace()
        ws.get(max(rsc.knn_workspace_bytes(n, n, d, k), rsc.connectivities_workspace_bytes(n, k)))
        out = (torch.empty((n, k), dtype=torch.int32, device="cuda"), torch.empty((n, k), dtype=torch.float32, device="cuda"))
        cap = 2 * n * (k - 1)
        csr = (torch.empty(n + 1, dtype=torch.int64, device="cuda"), torch.empty(cap, dtype=torch.int32, device="cuda"),
               torch.empty(cap, dtype=torch.float32, device="cuda"))
        log(f"[bench] large k: k={k}")
        rsc.knn(Xt, k, out=out, workspace=ws)
        rsc.connectivities(out[0], out[1], workspace=ws, out=csr)
        torch.cuda.synchronize()
        rsc.profile_reset()
        rsc.profile_enable(True)
        t0 = time.perf_counter()
        for _ in range(args.form_steps):
            rsc.knn(Xt, k, out=out, workspace=ws)
            st = rsc.read_knn_stats(ws)
            g = rsc.connectivities(out[0], out[1], workspace=ws, out=csr)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / args.form_steps
        rsc.profile_enable(False)
        kern = {}
        for name in ["screen_fp32", "rerank", "screen_escalate", "rerank_escalate", "rescan"]:
            tot, cnt = rsc.profile_get(name)
            if cnt:
                kern[name] = round(tot / cnt, 3)
        res[f"k{k}"] = {"cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2), "kernel_ms": kern,
                        "escalated_rows": st["escalated_rows"], "rescanned_rows": st["rescanned_rows"],
                        "nnz": int(g.nnz)}
        del out, csr, ws, g
        torch.cuda.empty_cache()
    return res


def pca_form(args, rsc) -> dict:
    """Sparse PCA of a cells x genes CSR matrix (Methods, Principal component
    analysis): means, Gram, centring, top-50 eigenpairs, scores."""
    import torch

    import synth

    n, p, k = args.pca_n, synth.SPARSE_PCA["p"], 50
    log(f"[bench] pca: generating {n} x {p} CSR")
    t0 = time.perf_counter()
    ip, ix, v = synth.sparse_expression(n=n)
    gen_s = time.perf_counter() - t0
    nnz = int(ip[-1])
    ipt, ixt, vt = torch.from_numpy(ip).cuda(), torch.from_numpy(ix).cuda(), torch.from_numpy(v).cuda()
    ws = rsc.Workspace()
    log("[bench] pca: warmup")
    rsc.pca(ipt, ixt, vt, p, k, workspace=ws)
    torch.cuda.synchronize()
    steps = max(1, args.form_steps)
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(steps):
        mean, evals, V, Z = rsc.pca(ipt, ixt, vt, p, k, workspace=ws)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    rsc.profile_enable(False)
    kern = {}
    for name in ["pca_densify", "pca_gram", "pca_center", "pca_eigh", "pca_scores"]:
        tot, cnt = rsc.profile_get(name)
        if cnt:
            kern[name] = round(tot / steps, 3)
    P = (p + 1 + 63) // 64 * 64
    gram_flops = 2.0 * n * (P // 64) * (P // 64 + 1) / 2 * 64 * 64  # upper-triangle tiles, all padded columns
    alg_flops = 1.0 * n * p * (p + 1)  # the upper triangle of X^T X, 2 flops per product
    g_ms = kern.get("pca_gram")
    ev = evals.cpu().numpy()
    cpu = None if args.no_cpu_baseline else pca_cpu_baseline(ip, ix, v, p)
    return {"workload": f"CSR {n} cells x {p} genes, {nnz} stored entries ({nnz / (n * p):.3f} dense), "
                        f"k = {k}, latent 8-program model (seed {synth.SPARSE_PCA['seed']})",
            "ms_per_call": round(ms, 2), "cells_per_s": round(n / (ms / 1e3), 1), "kernel_ms": kern,
            "gram_fp64_tflops_algorithmic": round(alg_flops / (g_ms / 1e3) / 1e12, 2) if g_ms else None,
            "gram_fp64_tflops_tiles": round(gram_flops / (g_ms / 1e3) / 1e12, 2) if g_ms else None,
            "gram_frac_of_fp64_peak": round(gram_flops / (g_ms / 1e3) / 1e12 / PEAK_FP64_TFLOPS, 4) if g_ms else None,
            "top_evals": [round(float(x), 5) for x in ev[:5]], "generation_s": round(gen_s, 1), "cpu_baseline": cpu}


def pca_cpu_baseline(ip, ix, v, p) -> dict:
    """The oracle's float64 Gram and means on the first cells of the same
    matrix (cells per second of the covariance step)."""
    from oracle import pca as opca

    m = 20000
    t0 = time.perf_counter()
    opca.covariance(ip[:m + 1], ix, v, p)
    secs = time.perf_counter() - t0
    return {"value": round(m / secs, 1), "unit": "cells/s (covariance)", "cores": 1, "kind": "oracle",
            "sample": f"the first {m} cells ({secs:.2f} s)"}


def umap_samples(w: np.ndarray, n_epochs: int) -> int:
    """Edge samples a layout of n_epochs makes: edge e (eps = w_max / w_e,
    kept if w_e >= w_max / n_epochs) is due at epochs eps, 2 eps, ... below
    n_epochs (the float64 accumulation of eps can move a boundary sample:
    the count is exact up to those)."""
    w = w.astype(np.float64)
    wmax = w.max() if w.size else 0.0
    keep = (w > 0) & (w >= wmax / n_epochs)
    eps = wmax / w[keep]
    return int(np.floor((n_epochs - 1) / eps + 1e-9).sum())


def leiden_form(args, rsc, csr=None) -> dict:
    """Leiden communities of the 1M-cell kNN graph (the clustering step the
    paper runs on this graph), modularity at resolution 1.  ``cpu_baseline``
    runs the oracle on the graph of a 30,000-cell mixture (the oracle is
    sequential; the whole 1M graph would take minutes)."""
    import torch

    import synth

    if csr is None:
        w = WORKLOADS["plain_1m"]
        log("[bench] leiden: building the 1M-cell graph")
        X = torch.from_numpy(synth.mixture(w["n"], d=50, n_clusters=w["clusters"], law=w["law"],
                                           seed=w["seed"])).cuda()
        ws0 = rsc.Workspace()
        idx, dist = rsc.knn(X, args.k, workspace=ws0)
        g = rsc.connectivities(idx, dist, workspace=ws0)
        csr = (g.indptr, g.indices, g.data)
        del X, idx, dist, ws0
    indptr, indices, data = csr
    n = indptr.numel() - 1
    nnz = int(indptr[-1].item())
    graph = (indptr, indices[:nnz], data[:nnz])
    ws = rsc.Workspace()
    log("[bench] leiden: warmup")
    rsc.leiden(graph, workspace=ws)
    torch.cuda.synchronize()
    steps = max(1, args.form_steps)
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(steps):
        labels, st = rsc.leiden(graph, workspace=ws)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    rsc.profile_enable(False)
    kern = {}
    for name in ["leiden", "leiden_move", "leiden_refine", "leiden_aggregate"]:
        tot, cnt = rsc.profile_get(name)
        if cnt:
            kern[name] = round(tot / steps, 3)
    move = None
    if kern.get("leiden_move"):
        # local moving is bound by HBM and L2 gathers: per sweep, every CSR
        # entry's column and fixed-point weight (12 B) and its neighbour's
        # label (4 B); per vertex its row pointer, degree, label in and out
        # (24 B); the library sums these algorithmic bytes over all sweeps
        gbs = st["move_bytes"] / (kern["leiden_move"] / 1e3) / 1e9
        move = {"bound": "hbm", "kernel": "k_lv_move", "unit": "GB/s", "bytes_per_call": st["move_bytes"],
                "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS, "frac": round(gbs / PEAK_HBM_GBS, 4)}
    cpu = None
    if not args.no_cpu_baseline:
        from oracle import leiden as ol

        Xs = synth.mixture(30000, d=50, n_clusters=25, law="zipf", seed=64)
        _, _, gs = rsc.knn_graph(torch.from_numpy(Xs).cuda(), args.k)
        p_, x_, d_ = (t.cpu().numpy() for t in (gs.indptr, gs.indices, gs.data))
        t1 = time.perf_counter()
        ol.leiden(p_, x_, d_)
        secs = time.perf_counter() - t1
        cpu = {"value": round(30000 / secs, 1), "unit": "cells/s", "cores": 1, "kind": "oracle",
               "sample": f"the kNN graph of a 30,000-cell mixture ({len(x_)} entries), whole ({secs:.2f} s)"}
    return {"workload": f"fuzzy kNN graph of the 1M-cell plain workload: {n} vertices, {nnz} stored edges; "
                        "modularity, resolution 1",
            "ms_per_call": round(ms, 2), "cells_per_s": round(n / (ms / 1e3), 1), "kernel_ms": kern,
            "levels": st["levels"], "sweeps": st["sweeps"], "refinement_rounds": st["rounds"],
            "communities": st["n_communities"], "modularity": round(st["quality"], 6),
            "move_roofline": move, "cpu_baseline": cpu}


def umap_form(args, rsc, csr=None) -> dict:
    """UMAP layout of the 1M-cell kNN graph (the embedding step the paper
    runs on this graph): 200 epochs of edge-sampled SGD, 5 negatives per
    sample, 2-D, random initial embedding."""
    import torch

    import synth

    n_epochs, neg, dim = args.umap_epochs, 5, 2
    if csr is None:
        w = WORKLOADS["plain_1m"]
        log("[bench] umap: building the 1M-cell graph")
        X = torch.from_numpy(synth.mixture(w["n"], d=50, n_clusters=w["clusters"], law=w["law"],
                                           seed=w["seed"])).cuda()
        ws0 = rsc.Workspace()
        idx, dist = rsc.knn(X, args.k, workspace=ws0)
        g = rsc.connectivities(idx, dist, workspace=ws0)
        csr = (g.indptr, g.indices, g.data)
        del X, idx, dist, ws0
    indptr, indices, data = csr
    n = indptr.numel() - 1
    nnz = int(indptr[-1].item())
    indices, data = indices[:nnz], data[:nnz]
    Y0 = torch.from_numpy(synth.umap_init(n, dim, seed=13)).cuda()
    ws = rsc.Workspace()
    log("[bench] umap: warmup")
    rsc.umap_layout((indptr, indices, data), Y0, n_epochs=n_epochs, neg=neg, seed=1, workspace=ws)
    torch.cuda.synchronize()
    steps = max(1, args.form_steps)
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(steps):
        Y = rsc.umap_layout((indptr, indices, data), Y0, n_epochs=n_epochs, neg=neg, seed=1, workspace=ws)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    rsc.profile_enable(False)
    kern = {}
    for name in ["umap_init", "umap_epochs", "umap_due", "umap_moves"]:
        tot, cnt = rsc.profile_get(name)
        if cnt:
            kern[name] = round(tot / steps, 3)
    wts = data.cpu().numpy()
    samples = umap_samples(wts, n_epochs)
    ep_ms = kern.get("umap_epochs")
    moves = None
    if kern.get("umap_moves"):
        # the epoch kernel is bound by float64 vector issue (the correctly
        # rounded power): UMAP_MOVE_FP64_OPS float64 instructions per slot, one
        # slot per (edge sample, draw)
        slots = samples * (1 + neg)
        rate = slots * UMAP_MOVE_FP64_OPS / (kern["umap_moves"] / 1e3) / 1e12
        moves = {"bound": "alu", "kernel": "k_umap_epoch<2>", "unit": "T float64 ops/s", "slots": slots,
                 "ops_per_slot": UMAP_MOVE_FP64_OPS, "achieved": round(rate, 2), "peak": PEAK_FP64_VECTOR_OPS,
                 "frac": round(rate / PEAK_FP64_VECTOR_OPS, 4)}
    finite = bool(torch.isfinite(Y).all().item())
    cpu = None
    if not args.no_cpu_baseline:
        cpu = umap_cpu_baseline(indptr.cpu().numpy(), indices.cpu().numpy(), wts, Y0.cpu().numpy(), neg, samples,
                                n_epochs)
    return {"workload": f"fuzzy kNN graph of the 1M-cell plain workload: {n} vertices, {nnz} stored edges; "
                        f"{n_epochs} epochs, {neg} negative samples, dim {dim}, random initial layout",
            "ms_per_call": round(ms, 2), "layouts_per_s": round(1e3 / ms, 3), "kernel_ms": kern,
            "edge_samples": samples, "pow_evaluations_approx": samples * (1 + neg),
            "edge_samples_per_s": round(samples / (ep_ms / 1e3), 1) if ep_ms else None,
            "ms_per_epoch": round(ep_ms / n_epochs, 4) if ep_ms else None, "epoch_kernel_roofline": moves,
            "finite": finite, "cpu_baseline": cpu}


def umap_cpu_baseline(indptr, indices, w, Y0, neg, samples_full, n_epochs_full) -> dict:
    """The oracle's layout of the same graph over 3 epochs (epochs 1 and 2
    sample the edges with w >= w_max / 2), as edge samples per second, and
    scaled to full layouts per second."""
    import oracle
    from oracle import umap as ou

    E = 3
    s = umap_samples(w, E)
    t0 = time.perf_counter()
    ou.layout(indptr, indices, w, Y0, E, 0.5830300203414425, 1.3341669924314914, neg=neg, seed=1)
    secs = time.perf_counter() - t0
    rate = s / secs
    return {"value": round(rate / samples_full, 6), "unit": f"{n_epochs_full}-epoch layouts/s",
            "edge_samples_per_s": round(rate, 1), "cores": oracle.max_threads(), "kind": "oracle",
            "sample": f"{E} epochs of the same graph ({s} edge samples, {secs:.1f} s)"}


def batched_form(args, rsc) -> dict:
    """64 independent samples (log-uniform 2k..200k cells, 10-40 clusters each):
    per-sample exact kNN in one persistent launch + connectivities."""
    import torch

    import synth

    k = args.k
    log("[bench] batched form: generating 64 samples")
    X, off = synth.batched_samples()
    n, d = X.shape
    dev = torch.device("cuda:0")
    Xt = torch.from_numpy(X).to(dev)
    del X
    ws = rsc.Workspace(dev)
    ws.get(max(rsc.knn_batched_workspace_bytes(off, d, k), rsc.connectivities_workspace_bytes(n, k)))
    cap = 2 * n * (k - 1)
    idx = torch.empty((n, k), dtype=torch.int32, device=dev)
    dist = torch.empty((n, k), dtype=torch.float32, device=dev)
    csr = (torch.empty(n + 1, dtype=torch.int64, device=dev), torch.empty(cap, dtype=torch.int32, device=dev),
           torch.empty(cap, dtype=torch.float32, device=dev))
    log("[bench] batched form: autotune")
    chosen, table = rsc.knn_batched_autotune(Xt, off, k, workspace=ws)
    for _ in range(1):
        rsc.knn_batched(Xt, off, k, out=(idx, dist), workspace=ws)
        rsc.connectivities(idx, dist, workspace=ws, out=csr)
    torch.cuda.synchronize()
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for _ in range(args.form_steps):
        rsc.knn_batched(Xt, off, k, out=(idx, dist), workspace=ws)
        stats = rsc.read_knn_stats(ws)
        g = rsc.connectivities(idx, dist, workspace=ws, out=csr)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    rsc.profile_enable(False)
    ms = (t1 - t0) * 1e3 / args.form_steps
    tot, cnt = rsc.profile_get("screen_batched")
    scr = tot / cnt
    sizes = np.diff(off)
    flops = float(2 * d * (sizes.astype(np.float64) ** 2).sum())
    return {"workload": f"64 samples, {n} cells, sizes log-uniform in [2000, 200000] (seed 4), d=50, k=15",
            "cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2), "screen_ms": round(scr, 2),
            "screen_tflops": round(flops / (scr / 1e3) / 1e12, 2),
            "screen_frac_of_fp16_peak": round(flops / (2 * d) * 32 * split_mfmas(d) / (scr / 1e3) / 1e12
                                              / PEAK_FP16_TFLOPS, 4),  # 16 slots per issued MFMA
            "autotune_choice": list(table)[chosen] if 0 <= chosen < len(table) else None,
            "autotune_screen_ms": {kk: round(v, 2) for kk, v in table.items()},
            "escalated_rows": stats["escalated_rows"], "rescanned_rows": stats["rescanned_rows"], "nnz": int(g.nnz),
            "exact": True}


def routed_form(args, rsc) -> dict:
    """The learned-router form: base n = 5M cells (500-cluster Zipf mixture),
    P = 4096 k-means partitions, a 50-256-256-4096 router trained on the
    exact-kNN partition labels of a held-out 1M-cell draw, top-32 probes,
    exact search for rows whose probed softmax mass is below 0.9.

    The index (partitions, labels, training) is built once and timed on its
    own; a timed step is the routed kNN of every base cell plus the
    connectivities.  Recall@15 is measured against the exact path on sampled
    rows, and nearest-centroid probing with the same probe count is measured
    beside it (the method without the router)."""
    import torch

    import synth

    k, P, probes, thr = args.k, synth.ROUTED["parts"], args.routed_probes, args.routed_threshold
    log(f"[bench] routed form: generating base {args.routed_n} + train {args.routed_train}")
    base, train = synth.routed_draws(n_base=args.routed_n, n_train=args.routed_train)
    n, d = base.shape
    dev = torch.device("cuda:0")
    Xb = torch.from_numpy(base).to(dev)
    Xt = torch.from_numpy(train).to(dev)
    del base, train
    ws = rsc.Workspace(dev)
    build = {}

    def clock(name, fn):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out = fn()
        torch.cuda.synchronize()
        build[name] = round(time.perf_counter() - t0, 3)
        log(f"[bench] routed form: {name} {build[name]} s")
        return out

    init = torch.from_numpy(synth.init_rows(n, P, seed=5)).to(dev)
    C, assign, off, perm, relocated = clock(
        "kmeans_s", lambda: rsc.partition_kmeans(Xb, P, init, args.routed_iters, workspace=ws))
    tidx, _ = clock("labels_exact_knn_s", lambda: rsc.knn(Xb, k, Q=Xt, workspace=ws))
    labels = rsc.partition_labels(tidx, assign)
    del tidx
    router = rsc.Router(d, 256, P, seed=1)

    def train_schedule():
        # Adam, learning rate decayed per epoch along a half cosine from 1e-3
        # (one library call per epoch; the optimiser state carries over)
        out = []
        for e in range(args.routed_epochs):
            lr = 1e-3 * 0.5 * (1.0 + math.cos(math.pi * e / args.routed_epochs))
            out += router.train(Xt, labels, epochs=1, batch=4096, lr=lr, workspace=ws)
        return out

    losses = clock("train_s", train_schedule)
    del labels, Xt
    torch.cuda.empty_cache()

    cap = 2 * n * (k - 1)
    idx = torch.empty((n, k), dtype=torch.int32, device=dev)
    dist = torch.empty((n, k), dtype=torch.float32, device=dev)
    csr = (torch.empty(n + 1, dtype=torch.int64, device=dev), torch.empty(cap, dtype=torch.int32, device=dev),
           torch.empty(cap, dtype=torch.float32, device=dev))
    rws = rsc.Workspace(dev)

    def step():
        _, _, route, st = rsc.knn_routed(router, Xb, k, off, perm, probes=probes, mass_threshold=thr,
                                         out=(idx, dist), workspace=rws)
        g = rsc.connectivities(idx, dist, workspace=ws, out=csr)
        return st, g

    step()
    torch.cuda.synchronize()
    rsc.profile_reset()
    rsc.profile_enable(True)
    t0 = time.perf_counter()
    for i in range(args.form_steps):
        st, g = step()
        log(f"[bench] routed form: step {i + 1}/{args.form_steps}")
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.form_steps
    rsc.profile_enable(False)
    kern = {}
    for name in ["router_infer", "probed_prep", "screen_routed", "rerank_probed", "prep_pack", "screen_fp32",
                 "rerank", "screen_escalate", "rescan"]:
        tot, cnt = rsc.profile_get(name)
        if cnt:
            kern[name] = round(tot / args.form_steps, 3)

    routed_idx = idx.clone()
    # the reference for recall: plain exact FP32 kNN + connectivities of all n cells, timed once
    log("[bench] routed form: exact search of every cell (the reference for recall)")
    ews = rsc.Workspace(dev)
    ews.get(rsc.knn_workspace_bytes(n, n, d, k))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rsc.knn(Xb, k, out=(idx, dist), workspace=ews)
    g_exact = rsc.connectivities(idx, dist, workspace=ws, out=csr)
    torch.cuda.synchronize()
    ms_exact = (time.perf_counter() - t0) * 1e3
    exact_stats = rsc.read_knn_stats(ews)
    del ews
    ex_idx = idx

    def recall(found):
        """Mean over all cells of |found ∩ exact| / (k - 1) over the non-self columns."""
        hits = 0
        for s0 in range(0, n, 1 << 20):
            a = found[s0:s0 + (1 << 20), 1:]
            b = ex_idx[s0:s0 + (1 << 20), 1:]
            hits += int((a[:, :, None] == b[:, None, :]).sum())
        return hits / (n * (k - 1))

    rec = recall(routed_idx)
    low_mass = int(st["low_mass_rows"])

    def timed(fn):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out = fn()
        torch.cuda.synchronize()
        return out, (time.perf_counter() - t0) * 1e3

    # the network alone: the same probes, no fallback
    (ro_idx, _, _, st_ro), ms_ro = timed(lambda: rsc.knn_routed(router, Xb, k, off, perm, probes=probes,
                                                                mass_threshold=0.0, workspace=rws))
    rec_ro = recall(ro_idx)
    del ro_idx
    # the method without the router: the nearest centroids (IVF probing), no
    # fallback, at several probe counts; the centroid kNN is part of each step
    nc_probes = sorted({probes, 48, 64})  # the probed search supports up to 64 probes
    nc = {}
    nc_dist = None
    for pr in nc_probes:
        def nc_step(pr=pr):
            parts_, dist_ = rsc.knn(C, pr, Q=Xb, workspace=ws)
            return parts_, dist_, rsc.knn_probed(Xb, k, off, perm, parts_, workspace=rws)
        (parts_, dist_, (nc_idx, _, _, st_nc)), ms_nc = timed(nc_step)
        nc[pr] = {"recall@15": round(recall(nc_idx), 5), "ms_per_step": round(ms_nc, 2),
                  "cells_per_s": round(n / (ms_nc / 1e3), 1), "mean_probed_rows": round(st_nc["mean_probed_rows"], 1)}
        if pr == probes:
            nc_parts = parts_
        if pr == max(nc_probes):
            nc_dist = dist_
        del nc_idx
    reach = [pr for pr in nc_probes if nc[pr]["recall@15"] >= 0.99]
    # nearest centroids + exact search for as many rows as the router sent to
    # exact search, chosen as the rows whose probe boundary is least clear:
    # smallest gap between the squared distances of the (probes+1)-th and the
    # probes-th nearest centroid, or between the (probes+1)-th and the nearest
    gaps = {}
    for name, (a, b) in {"gap_next": (probes, probes - 1), "gap_first": (probes, 0)}.items():
        g2 = nc_dist[:, a].double() ** 2 - nc_dist[:, b].double() ** 2
        mask = torch.zeros(n, dtype=torch.uint8, device=dev)
        if low_mass:
            mask[torch.argsort(g2)[:low_mass]] = 1
        (m_idx, _, _, _), ms_m = timed(lambda: rsc.knn_probed(Xb, k, off, perm, nc_parts, exact_rows=mask,
                                                              workspace=rws))
        gaps[name] = {"recall@15": round(recall(m_idx), 5), "knn_ms": round(ms_m, 2), "exact_rows": low_mass}
        del m_idx, mask
    router.close()
    return {"workload": f"base n={n}, d=50, k=15, 500-cluster Zipf(1.1) mixture (centres seed 5, base seed 50), "
                        f"router trained on {args.routed_train} held-out cells (seed 51)",
            "cells_per_s": round(n / (ms / 1e3), 1), "ms_per_step": round(ms, 2), "kernel_ms_per_step": kern,
            "recall@15": round(rec, 5), "meets_recall_0.99": rec >= 0.99, "recall_measured_on": f"all {n} cells",
            "plain_exact_same_workload": {"cells_per_s": round(n / (ms_exact / 1e3), 1),
                                          "ms_per_step": round(ms_exact, 1), "nnz": int(g_exact.nnz),
                                          "escalated_rows": exact_stats["escalated_rows"],
                                          "rescanned_rows": exact_stats["rescanned_rows"]},
            "speedup_vs_plain_exact": round(ms_exact / ms, 2),
            "parts": P, "probes": probes, "mass_threshold": thr, "stats": st, "nnz": int(g.nnz),
            "index_build_s": build, "kmeans_iters": args.routed_iters, "kmeans_relocated": relocated,
            "train_epochs": args.routed_epochs, "train_loss_per_epoch": [round(v, 4) for v in losses],
            "ablation": {
                "router_plus_fallback": {"recall@15": round(rec, 5), "exact_rows": low_mass,
                                         "cells_per_s": round(n / (ms / 1e3), 1)},
                "router_only": {"recall@15": round(rec_ro, 5), "knn_ms": round(ms_ro, 2)},
                "nearest_centroids": nc,
                "nearest_centroid_probes_reaching_0.99": min(reach) if reach else None,
                "nearest_centroids_plus_fallback_same_rows": gaps}}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="plain_1m", choices=sorted(WORKLOADS))
    ap.add_argument("--k", type=int, default=15)
    ap.add_argument("--cpu-budget", type=float, default=15.0, help="seconds of oracle work for cpu_baseline")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--traffic-probe", action="store_true", help="run the PMC calibration program and exit")
    ap.add_argument("--precision-probe", action="store_true",
                    help="run one BF16 and one FP8 kNN call on the 2M workload (for counter runs) and exit")
    ap.add_argument("--no-forms", action="store_true", help="skip the 2M-cell precision forms")
    ap.add_argument("--form-steps", type=int, default=3)
    ap.add_argument("--no-routed", action="store_true", help="skip the learned-router form")
    ap.add_argument("--pca-n", type=int, default=1_000_000, help="cells of the sparse-PCA form")
    ap.add_argument("--umap-epochs", type=int, default=200)
    ap.add_argument("--only", choices=["cosine", "edistance", "large_k", "pca", "precision", "batched", "routed", "leiden",
                                       "umap"],
                    help="run one form alone and print its record (no benchmark line)")
    ap.add_argument("--routed-n", type=int, default=5_000_000)
    ap.add_argument("--routed-train", type=int, default=1_000_000)
    ap.add_argument("--routed-iters", type=int, default=10, help="k-means iterations")
    ap.add_argument("--routed-epochs", type=int, default=16)
    ap.add_argument("--routed-probes", type=int, default=32)
    ap.add_argument("--routed-threshold", type=float, default=0.9)
    args = ap.parse_args()
    if args.traffic_probe:
        return traffic_probe()
    if args.precision_probe:
        return precision_probe()

    if args.gpus != 1:
        print(f"bench.py measures one GPU only: --gpus {args.gpus} is not supported (the kNN graph here runs "
              "on a single MI355X; multi-GPU sharding is described in the design notes, not built)",
              file=sys.stderr)
        return 2

    import torch

    import paper_2603_02402_amd as rsc
    import synth

    if not torch.cuda.is_available():
        print("no GPU visible", file=sys.stderr)
        return 1
    rsc.load()
    if args.only == "cosine":
        w = WORKLOADS["plain_1m"]
        Xc = torch.from_numpy(synth.mixture(w["n"], d=50, n_clusters=w["clusters"], law=w["law"],
                                            seed=w["seed"])).cuda()
        nc, kc = Xc.shape[0], args.k
        out = (torch.empty((nc, kc), dtype=torch.int32, device="cuda"),
               torch.empty((nc, kc), dtype=torch.float32, device="cuda"),
               (torch.empty(nc + 1, dtype=torch.int64, device="cuda"),
                torch.empty(2 * nc * (kc - 1), dtype=torch.int32, device="cuda"),
                torch.empty(2 * nc * (kc - 1), dtype=torch.float32, device="cuda")))
        print(json.dumps({"cosine": cosine_form(args, rsc, Xc, rsc.Workspace(), out)}), flush=True)
        return 0
    if args.only:
        fn = {"precision": precision_forms, "batched": batched_form, "routed": routed_form,
              "edistance": edistance_form, "large_k": large_k_form, "pca": pca_form, "umap": umap_form,
              "leiden": leiden_form}[args.only]
        print(json.dumps({args.only: fn(args, rsc)}), flush=True)
        return 0

    w = WORKLOADS[args.workload]
    k = args.k
    log(f"[bench] generating {args.workload}")
    X = synth.mixture(w["n"], d=50, n_clusters=w["clusters"], law=w["law"], seed=w["seed"])
    n, d = X.shape
    dev = torch.device("cuda:0")
    Xt = torch.from_numpy(X).to(dev)
    ws = rsc.Workspace(dev)
    ws.get(max(rsc.knn_workspace_bytes(n, n, d, k), rsc.connectivities_workspace_bytes(n, k)))
    idx = torch.empty((n, k), dtype=torch.int32, device=dev)
    dist = torch.empty((n, k), dtype=torch.float32, device=dev)
    cap = 2 * n * (k - 1)
    csr = (torch.empty(n + 1, dtype=torch.int64, device=dev), torch.empty(cap, dtype=torch.int32, device=dev),
           torch.empty(cap, dtype=torch.float32, device=dev))
    torch.cuda.synchronize()

    def step():
        rsc.knn(Xt, k, out=(idx, dist), workspace=ws)
        stats = rsc.read_knn_stats(ws)
        g = rsc.connectivities(idx, dist, workspace=ws, out=csr)
        return stats, g

    for i in range(args.warmup):
        log(f"[bench] warmup {i + 1}/{args.warmup}")
        step()
    torch.cuda.synchronize()

    rsc.profile_reset()
    rsc.profile_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    stats = g = None
    for i in range(args.steps):
        stats, g = step()
        log(f"[bench] step {i + 1}/{args.steps}")
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    rsc.profile_enable(False)

    ms_per_step = (t1 - t0) * 1e3 / args.steps
    value = n / (ms_per_step / 1e3)

    kernels = {}
    for name in ["prep_pack", "screen_fp32", "rerank", "screen_escalate", "rerank_escalate", "rescan", "graph_init",
                 "smooth_knn", "union_count", "csr_scan", "union_fill", "row_sort"]:
        tot, cnt = rsc.profile_get(name)
        if cnt:
            kernels[name] = round(tot / cnt, 4)
    screen_ms = kernels.get("screen_fp32")
    roofline = None
    pairs = screened_pairs(ws, n) if screen_ms and n >= 16384 else float(n) * n
    if screen_ms:
        flops = pairs * 32.0 * split_mfmas(d)  # issued: 16 slots an MFMA
        achieved = flops / (screen_ms / 1e3) / 1e12
        roofline = {"bound": "mfma", "achieved": round(achieved, 2), "peak": PEAK_FP16_TFLOPS, "unit": "TFLOP/s",
                    "frac": round(achieved / PEAK_FP16_TFLOPS, 4),
                    "traffic": measured_traffic() if args.workload == "plain_1m" and k == 15 else None,
                    "kernel": ("k_split_pruned (segments outside every query's reach skipped; " if n >= 16384 else
                               "k_screen_split (") + "split FP16 MFMA 32x32x16 distance screen + per-query top-32 lists)",
                    "screened_pairs": pairs, "screened_pairs_of_all": round(pairs / (float(n) * n), 5),
                    "work_per_launch": f"{split_mfmas(d)} MFMAs of 16 slots per 32 x 32 screened pairs = "
                                       f"{flops:.3e} flop issued; all pairs: 2*d*n^2 = {2.0 * d * n * n:.3e} (d={d}, n={n})"}

    graph = graph_gbs(kernels, n, k, int(g.nnz))

    forms = None
    if not args.no_forms:
        forms = {"cosine_fp32": cosine_form(args, rsc, Xt, ws, (idx, dist, csr))}
        # the layout runs on the plain graph: rebuild it into the CSR buffers
        step()
        del Xt, idx, dist
        ws.buf = None
        torch.cuda.empty_cache()
        forms["umap_layout"] = umap_form(args, rsc, csr)
        forms["leiden"] = leiden_form(args, rsc, csr)
        del csr
        ws.buf = None
        torch.cuda.empty_cache()
        forms.update(precision_forms(args, rsc))
        torch.cuda.empty_cache()
        forms["batched_fp32"] = batched_form(args, rsc)
        torch.cuda.empty_cache()
        forms["edistance_fp64"] = edistance_form(args, rsc)
        torch.cuda.empty_cache()
        forms["sparse_pca"] = pca_form(args, rsc)
        if not args.no_routed:
            torch.cuda.empty_cache()
            forms["routed"] = routed_form(args, rsc)

    cpu = None
    if not args.no_cpu_baseline:
        log("[bench] cpu_baseline (oracle on a sample of rows)")
        cpu = cpu_baseline(X, k, args.cpu_budget)

    out = {
        "metric": METRIC,
        "value": round(value, 1),
        "unit": "cells/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "fp32",
        "data": "synthetic",
        "config": {"workload": w["desc"], "form": "plain exact (split FP16 MFMA screen at FP32 accuracy, FP64 rerank + certificate)",
                   "n": n, "d": d, "k": k, "nnz": int(g.nnz), "escalated_rows": stats["escalated_rows"],
                   "rescanned_rows": stats["rescanned_rows"],
                   "max_err_ratio": round(stats["max_err_ratio"], 4)},
        "kernel_ms": kernels,
        "graph_gbs": graph,
        "roofline": roofline,
        "cpu_baseline": cpu,
        "forms": forms,
    }
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
