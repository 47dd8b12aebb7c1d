"""The work a user of this package has it do, as cases that can be timed and compared.

A case is a dict of plain values; ``listed()`` gives the fixed ones, ``draw``
more of the same ranges.  ``prepare`` makes what a program holds before the
call (inputs on the GPU, a workspace, an index or a network), ``run`` is one
pass through the public calls, ``work`` the bytes and operations that pass
cannot do without, and ``exact`` the same outputs in 64 bits by plain torch.

Inputs are Gaussian mixtures shaped like PCA embeddings of single cells
(cluster centres N(0, 25 I), within-cluster variances 1/i), sparse log-count
matrices, and the graphs built from them, all drawn on the GPU from the seed.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_02402_amd as rsc

# exact() of a neighbour search compares all pairs in float64: up to this many pair-dimensions it takes seconds
_EXACT_PAIR_DIMS = 6e12


def listed():
    return [
        # a small sample or a test run: launches and latency are the whole call
        dict(name="graph_2k", kind="graph", n=2000, d=50, k=15, metric="euclidean", clusters=20),
        # an atlas subset under the cosine metric with a wider neighbourhood; ragged row count, d not a multiple of 16
        dict(name="graph_cosine_70k", kind="graph", n=70001, d=30, k=30, metric="cosine", clusters=40),
        # the benchmark's workload: one large exact graph
        dict(name="graph_1m", kind="graph", n=1000000, d=50, k=15, metric="euclidean", clusters=100),
        # new cells placed against an existing reference (label transfer): a rectangular search
        dict(name="query_20k_400k", kind="query", nq=20011, n=400000, d=50, k=15, metric="euclidean", clusters=100),
        # the approximate graph: BF16 screen with rerank
        dict(name="bf16_500k", kind="precision", n=500000, d=50, k=15, form="bf16", parts=0, clusters=100),
        # many samples of uneven size in one call, then their graphs
        dict(name="batched_48", kind="batched", samples=48, lo=2000, hi=40000, d=50, k=15, size_seed=4),
        # a partition index: every cell's nearest partitions, then its neighbours among their members
        dict(name="probed_300k", kind="probed", n=300000, d=50, k=15, parts=512, probes=48, clusters=100),
        # the router, the size of the benchmark's network: one training step's gradients (forward and backward) and
        # the partitions it picks for a block of cells
        dict(name="router_4096", kind="router", batch=4096, cells=65536, d=50, hidden=256, parts=4096, probes=32, k=15),
        # a perturbation screen: every pair of groups, groups of 50 to 350 cells and one large control
        dict(name="edistance_600", kind="edistance", groups=600, lo=50, hi=351, control=10000, d=50),
        # the embedding itself: sparse log counts over highly variable genes
        dict(name="pca_200k", kind="pca", n=200000, genes=2000, density=0.05, k=50),
        # the layout of a graph
        dict(name="umap_200k", kind="umap", n=200000, k=15, epochs=100, neg=5, dim=2),
        # the communities of a graph
        dict(name="leiden_300k", kind="leiden", n=300000, k=15, gamma=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["graph", "graph", "graph", "query", "query", "precision", "batched", "probed", "router",
                       "edistance", "pca", "umap", "leiden"])
    d = rng.randint(10, 100)
    k = rng.choice([10, 15, 15, 20, 30, 50])
    if kind == "graph":
        return dict(kind=kind, n=_log_int(rng, 500, 400000), d=d, k=k,
                    metric=rng.choice(["euclidean", "euclidean", "cosine"]), clusters=rng.randint(5, 100))
    if kind == "query":
        nq = _log_int(rng, 1, 100000)
        return dict(kind=kind, nq=nq, n=_log_int(rng, 5000, 1000000), d=d, k=k,
                    metric=rng.choice(["euclidean", "euclidean", "cosine"]), clusters=rng.randint(5, 100))
    if kind == "precision":
        form = rng.choice(["bf16", "bf16", "fp8"])
        return dict(kind=kind, n=_log_int(rng, 20000, 500000), d=d, k=rng.choice([10, 15, 15, 20]), form=form,
                    parts=0 if form == "bf16" else 2 ** rng.randint(7, 10), clusters=rng.randint(10, 100))
    if kind == "batched":
        lo = _log_int(rng, 300, 3000)
        return dict(kind=kind, samples=rng.randint(3, 64), lo=lo, hi=lo * rng.randint(2, 25), d=d,
                    k=rng.choice([10, 15, 15, 20]), size_seed=rng.randint(0, 1 << 20))
    if kind == "probed":
        return dict(kind=kind, n=_log_int(rng, 40000, 300000), d=d, k=15, parts=64 * rng.randint(2, 12),
                    probes=rng.choice([16, 24, 32, 48]), clusters=rng.randint(20, 200))
    if kind == "router":
        return dict(kind=kind, batch=_log_int(rng, 500, 16384), cells=_log_int(rng, 1000, 100000), d=d,
                    hidden=rng.choice([128, 256]), parts=64 * rng.randint(4, 64), probes=rng.choice([16, 32, 48]), k=15)
    if kind == "edistance":
        lo = rng.randint(10, 60)
        return dict(kind=kind, groups=_log_int(rng, 20, 600), lo=lo, hi=lo * rng.randint(2, 6),
                    control=_log_int(rng, 500, 10000), d=d)
    if kind == "pca":
        return dict(kind=kind, n=_log_int(rng, 5000, 200000), genes=rng.randint(500, 2000),
                    density=round(rng.uniform(0.02, 0.08), 3), k=rng.choice([30, 50]))
    if kind == "umap":
        return dict(kind=kind, n=_log_int(rng, 2000, 300000), k=rng.choice([10, 15, 15, 30]),
                    epochs=rng.randint(20, 100), neg=rng.choice([3, 5, 5, 8]), dim=rng.choice([2, 2, 3]))
    return dict(kind="leiden", n=_log_int(rng, 2000, 400000), k=rng.choice([10, 15, 15, 30]),
                gamma=rng.choice([0.5, 1.0, 1.0, 2.0]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _mixture(g, n, d, clusters, centres=None):
    """n x d float32 rows around `clusters` centres, cluster sizes by a rank-Zipf law of exponent 1.1."""
    dev = "cuda"
    if centres is None:
        centres = torch.randn((clusters, d), generator=g, device=dev) * 5.0
    p = torch.arange(1, clusters + 1, device=dev, dtype=torch.float64) ** -1.1
    cum = torch.cumsum(p / p.sum(), 0)
    u = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
    label = torch.searchsorted(cum, u).clamp_(max=clusters - 1)
    sd = torch.arange(1, d + 1, device=dev, dtype=torch.float32).rsqrt()
    return centres[label] + torch.randn((n, d), generator=g, device=dev) * sd


def _metric(case):
    return rsc.RSC_COSINE if case["metric"] == "cosine" else rsc.RSC_EUCLIDEAN


def _sample_offsets(case):
    r = np.random.Generator(np.random.PCG64(case["size_seed"]))
    sizes = np.rint(np.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["samples"])))
    return np.concatenate([[0], np.cumsum(sizes.astype(np.int64))])


def _group_sizes(case):
    r = np.random.Generator(np.random.PCG64(9))
    s = np.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["groups"])).astype(np.int64)
    s[0] = case["control"]
    return s


def _sparse_counts(g, n, genes, density):
    """cells x genes CSR of log1p counts; a gene's detection falls off with its rank, 8 latent programs."""
    dev = "cuda"
    det = 1.0 / (1.0 + torch.arange(genes, device=dev, dtype=torch.float32) / 500.0)
    det = (det * (density / det.mean())).clamp_(max=0.9)
    v = torch.randn((8, genes), generator=g, device=dev) * 0.35
    b = torch.randn(genes, generator=g, device=dev) * 0.5 + 0.5
    ptr, cols, vals = [torch.zeros(1, dtype=torch.int64, device=dev)], [], []
    at = 0
    for s in range(0, n, 65536):
        m = min(65536, n - s)
        mask = torch.rand((m, genes), generator=g, device=dev) < det
        u = torch.randn((m, 8), generator=g, device=dev)
        depth = torch.exp(torch.randn((m, 1), generator=g, device=dev) * 0.3)
        x = torch.log1p(depth * torch.exp(b + u @ v))
        counts = mask.sum(1)
        ptr.append(torch.cumsum(counts, 0) + at)
        at += int(counts.sum())
        rows, c = torch.nonzero(mask, as_tuple=True)
        cols.append(c.to(torch.int32))
        vals.append(x[rows, c])
    return torch.cat(ptr), torch.cat(cols), torch.cat(vals)


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case=case, ws=rsc.Workspace("cuda"))
    if kind in ("graph", "precision", "batched"):
        n = int(_sample_offsets(case)[-1]) if kind == "batched" else case["n"]
        cap = 2 * n * (case["k"] - 1)
        s["csr"] = (torch.empty(n + 1, dtype=torch.int64, device="cuda"),
                    torch.zeros(cap, dtype=torch.int32, device="cuda"),
                    torch.zeros(cap, dtype=torch.float32, device="cuda"))
    if kind in ("graph", "precision"):
        s["X"] = _mixture(g, case["n"], case["d"], case["clusters"])
    elif kind == "query":
        centres = torch.randn((case["clusters"], case["d"]), generator=g, device="cuda") * 5.0
        s["X"] = _mixture(g, case["n"], case["d"], case["clusters"], centres)
        s["Q"] = _mixture(g, case["nq"], case["d"], case["clusters"], centres)
    elif kind == "batched":
        s["offsets"] = off = _sample_offsets(case)
        s["X"] = torch.cat([_mixture(g, int(b - a), case["d"], 10 + i % 31) for i, (a, b) in enumerate(zip(off, off[1:]))])
        s["gws"] = rsc.Workspace("cuda")
    elif kind == "probed":
        s["X"] = X = _mixture(g, case["n"], case["d"], case["clusters"])
        init = torch.randperm(case["n"], generator=g, device="cuda")[:case["parts"]].to(torch.int32)
        s["centroids"], _, s["offsets"], s["perm"], _ = rsc.partition_kmeans(X, case["parts"], init, 10)
    elif kind == "router":
        s["X"] = _mixture(g, case["batch"], case["d"], 200)
        s["labels"] = torch.randint(0, case["parts"], (case["batch"], case["k"]), generator=g, device="cuda",
                                    dtype=torch.int32)
        s["cells"] = _mixture(g, case["cells"], case["d"], 200)
        s["router"] = rsc.Router(case["d"], case["hidden"], case["parts"], seed=int(seed))
    elif kind == "edistance":
        sizes = _group_sizes(case)
        n, d = int(sizes.sum()), case["d"]
        label = torch.from_numpy(np.repeat(np.arange(sizes.size), sizes)).cuda()
        label = label[torch.randperm(n, generator=g, device="cuda")]
        sd = torch.arange(1, d + 1, device="cuda", dtype=torch.float32).rsqrt()
        effect = torch.rand(sizes.size, generator=g, device="cuda") < 0.3
        effect[0] = False
        scale = 0.2 * 10.0 ** torch.rand(sizes.size, generator=g, device="cuda") * effect
        shift = torch.randn((sizes.size, d), generator=g, device="cuda") * sd * scale[:, None]
        s["X"] = shift[label] + torch.randn((n, d), generator=g, device="cuda") * sd
        s["offsets"], s["cells"] = rsc.edistance_groups(label.to(torch.int32), sizes.size)
    elif kind == "pca":
        s["csr"] = _sparse_counts(g, case["n"], case["genes"], case["density"])
    else:  # umap, leiden: the graph of an embedding
        X = _mixture(g, case["n"], 50, 60)
        s["graph"] = rsc.knn_graph(X, case["k"])[2]
        if kind == "umap":
            s["Y0"] = torch.rand((case["n"], case["dim"]), generator=g, device="cuda") * 20.0 - 10.0
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------


def _graph_out(s, idx, dist, gr):
    """The lists, the CSR arrays the program keeps (whole: entries past the row pointers' end stay 0), rho and sigma."""
    indptr, indices, data = s["csr"]
    out = dict(idx=idx, dist=dist, indptr=indptr, indices=indices, data=data)
    if gr.rho is not None:
        out.update(rho=gr.rho, sigma=gr.sigma)
    return out


def run(s):
    case, ws = s["case"], s["ws"]
    kind = case["kind"]
    if kind == "graph":
        idx, dist = rsc.knn(s["X"], case["k"], metric=_metric(case), workspace=ws)
        return _graph_out(s, idx, dist, rsc.connectivities(idx, dist, workspace=ws, out=s["csr"]))
    if kind == "query":
        idx, dist = rsc.knn(s["X"], case["k"], Q=s["Q"], metric=_metric(case), workspace=ws)
        return dict(idx=idx, dist=dist)
    if kind == "precision":
        if case["form"] == "bf16":
            idx, dist = rsc.knn(s["X"], case["k"], precision=rsc.RSC_BF16, workspace=ws)
        else:
            idx, dist = rsc.knn(s["X"], case["k"], precision=rsc.RSC_FP8_E4M3, fp8_residual=case["parts"], workspace=ws)
        return _graph_out(s, idx, dist, rsc.connectivities(idx, dist, workspace=ws, out=s["csr"]))
    if kind == "batched":
        idx, dist = rsc.knn_batched(s["X"], s["offsets"], case["k"], workspace=ws)
        gr = rsc.connectivities_batched(idx, dist, s["offsets"], workspace=s["gws"], out=s["csr"])
        return _graph_out(s, idx, dist, gr)
    if kind == "probed":
        probes, _ = rsc.knn(s["centroids"], case["probes"], Q=s["X"], workspace=ws)
        idx, dist, route, _ = rsc.knn_probed(s["X"], case["k"], s["offsets"], s["perm"], probes, workspace=ws)
        return dict(idx=idx, dist=dist, route=route)
    if kind == "router":
        grad, loss = s["router"].gradients(s["X"], s["labels"], workspace=ws)
        parts, mass = s["router"].probe(s["cells"], case["probes"], workspace=ws)
        return dict(grad=grad, loss=loss, parts=parts, mass=mass)
    if kind == "edistance":
        E, D = rsc.edistance_pairwise(s["X"], s["offsets"], s["cells"], want_means=True, workspace=ws)
        return dict(E=E, D=D)
    if kind == "pca":
        mean, evals, loadings, scores = rsc.pca(*s["csr"], case["genes"], case["k"], workspace=ws)
        return dict(mean=mean, evals=evals, loadings=loadings, scores=scores)
    if kind == "umap":
        return rsc.umap_layout(s["graph"], s["Y0"], n_epochs=case["epochs"], neg=case["neg"], seed=7, workspace=ws)
    labels, stats = rsc.leiden(s["graph"], gamma=case["gamma"], workspace=ws)
    return dict(labels=labels, quality=float(stats["quality"]))


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------


def work(case):
    kind = case["kind"]
    if kind in ("graph", "precision"):
        n, d, k = case["n"], case["d"], case["k"]
        # embedding in; lists, row pointers, about 1.6 n (k-1) entries and rho / sigma out
        return dict(bytes=4.0 * n * d + 8.0 * n * k + 24.0 * n + 8 * 1.6 * n * (k - 1), flops=2.0 * d * n * n)
    if kind == "query":
        n, q, d, k = case["n"], case["nq"], case["d"], case["k"]
        return dict(bytes=4.0 * (n + q) * d + 8.0 * q * k, flops=2.0 * d * n * q)
    if kind == "batched":
        sizes = np.diff(_sample_offsets(case)).astype(np.float64)
        n, d, k = float(sizes.sum()), case["d"], case["k"]
        return dict(bytes=4.0 * n * d + 8.0 * n * k + 8.0 * n + 8 * 1.6 * n * (k - 1),
                    flops=2.0 * d * float((sizes ** 2).sum()))
    if kind == "probed":
        n, d, k, P = case["n"], case["d"], case["k"], case["parts"]
        return dict(bytes=4.0 * n * d + 8.0 * n * k, flops=2.0 * d * n * (P + n * case["probes"] / P))
    if kind == "router":
        b, c, d, h, P = case["batch"], case["cells"], case["d"], case["hidden"], case["parts"]
        params = d * h + h * h + h * P
        return dict(bytes=4.0 * (b * (d + case["k"]) + c * (d + case["probes"] + 1) + 2 * (params + 2 * h + P)),
                    flops=(6.0 * b + 2.0 * c) * params)
    if kind == "edistance":
        n, d, G = float(_group_sizes(case).sum()), case["d"], case["groups"]
        return dict(bytes=4.0 * n * (d + 1) + 16.0 * G * G, flops=d * n * (n - 1))
    if kind == "pca":
        n, p, k = case["n"], case["genes"], case["k"]
        nnz = n * p * case["density"]
        # the dense upper-triangle Gram the means and eigenvalues stand on, and the sparse scores
        return dict(bytes=8.0 * nnz + 8.0 * n + 4.0 * n * k + 8.0 * p * (k + 1), flops=1.0 * n * p * p + 2.0 * nnz * k)
    if kind == "umap":
        n, k = case["n"], case["k"]
        edges = 1.6 * n * (k - 1)
        # about 3 of 10 edges are due in an epoch; each with its draws takes two rows in, and a power of some 100 operations
        slots = 0.3 * edges * case["epochs"] * (1 + case["neg"])
        return dict(bytes=8.0 * edges + 8.0 * n * case["dim"], flops=100.0 * slots)
    n, k = case["n"], case["k"]
    edges = 1.6 * n * (k - 1)
    return dict(bytes=8.0 * edges + 12.0 * n, flops=2.0 * edges)


# ---------------------------------------------------------------------------
# the outputs in 64 bits, by plain torch
# ---------------------------------------------------------------------------


def _exact_knn(Q, X, k, cosine, self_first):
    """Distances (float64) and ids of the k nearest rows of X, by (distance, id); itself first in the square problem."""
    X, Q = X.double(), Q.double()
    nx = X.square().sum(1)
    if cosine:
        X, Q = X / nx.sqrt()[:, None], Q / Q.square().sum(1).sqrt()[:, None]
        nx = torch.ones_like(nx)
    m = min(X.shape[0], k + 9)
    Xt = X.t().contiguous()
    step = max(1, int(4e8) // X.shape[0])
    dist, ids = [], []
    for s in range(0, Q.shape[0], step):
        q = Q[s:s + step]
        key = torch.addmm(nx[None, :], q, Xt, alpha=-2.0)
        if self_first:
            r = torch.arange(q.shape[0], device=q.device)
            key[r, r + s] = -math.inf
        cand = key.topk(m, dim=1, largest=False).indices.sort(1).values
        del key
        diff = X[cand] - q[:, None, :]
        d2 = diff.square().sum(2)
        v = 0.5 * d2 if cosine else d2.sqrt()
        if self_first:
            v[cand == torch.arange(s, s + q.shape[0], device=q.device)[:, None]] = -1.0
        v, at = v.sort(dim=1, stable=True)
        dist.append(v[:, :k].clamp(min=0.0))
        ids.append(cand.gather(1, at)[:, :k])
    return torch.cat(dist), torch.cat(ids)


def _exact_graph(dist, ids):
    """rho, sigma and the fuzzy union (row pointers, columns, weights) of float32-rounded distances."""
    dd = dist.float().double()[:, 1:]
    n, m = dd.shape
    target = math.log2(m + 1)
    rho = torch.where(dd > 0, dd, math.inf).amin(1)
    rho = torch.where(torch.isinf(rho), 0.0, rho)
    gap = (dd - rho[:, None]).clamp(min=0.0)
    flat = (gap == 0).sum(1) >= target
    lo, hi = torch.zeros(n, device=dd.device).double(), torch.full((n,), math.inf, device=dd.device).double()
    mid = torch.ones_like(lo)
    for _ in range(120):
        above = torch.exp(-gap / mid[:, None]).sum(1) > target
        hi, lo = torch.where(above, mid, hi), torch.where(above, lo, mid)
        mid = torch.where(torch.isinf(hi), mid * 2, 0.5 * (lo + hi))
    sigma = torch.where(flat, 0.0, mid)
    a = torch.where(flat[:, None], (gap == 0).double(), torch.exp(-gap / mid[:, None]))
    i = torch.arange(n, device=dd.device)[:, None].expand(n, m).reshape(-1)
    j, a = ids[:, 1:].reshape(-1), a.reshape(-1)
    key, order = torch.cat([i * n + j, j * n + i]).sort(stable=True)
    both = torch.cat([a, a])[order]
    first = torch.ones_like(key, dtype=torch.bool)
    first[1:] = key[1:] != key[:-1]
    at = torch.cumsum(first, 0) - 1
    key = key[first]
    total = torch.zeros(key.numel(), device=dd.device).double().index_add_(0, at, both)
    prod = torch.where(torch.bincount(at) == 2, 1.0, 0.0).double()
    second = ~first
    prod[at[second]] = both[second] * both[second.nonzero().squeeze(1) - 1]
    w = total - prod
    keep = w.float() > 0
    key, w = key[keep], w[keep]
    indptr = torch.zeros(n + 1, dtype=torch.int64, device=dd.device)
    indptr[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    data = torch.zeros(2 * n * m, dtype=torch.float64, device=dd.device)
    data[:w.numel()] = w
    return dict(indptr=indptr, indices=None, data=data, rho=rho, sigma=sigma)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("graph", "precision"):
        if float(case["n"]) ** 2 * case["d"] > _EXACT_PAIR_DIMS:
            return None
        s = prepare(case, seed)
        dist, ids = _exact_knn(s["X"], s["X"], case["k"], case.get("metric") == "cosine", True)
        return dict(idx=None, dist=dist, **_exact_graph(dist, ids))
    if kind == "query":
        if float(case["n"]) * case["nq"] * case["d"] > _EXACT_PAIR_DIMS:
            return None
        s = prepare(case, seed)
        dist, ids = _exact_knn(s["Q"], s["X"], case["k"], case["metric"] == "cosine", False)
        return dict(idx=None, dist=dist)
    if kind == "batched":
        off = _sample_offsets(case)
        if float((np.diff(off).astype(np.float64) ** 2).sum()) * case["d"] > _EXACT_PAIR_DIMS:
            return None
        s = prepare(case, seed)
        dist, ids = [], []
        for a, b in zip(off, off[1:]):
            x = s["X"][a:b]
            dk, ik = _exact_knn(x, x, case["k"], False, True)
            dist.append(dk)
            ids.append(ik + int(a))
        dist = torch.cat(dist)
        gr = _exact_graph(dist, torch.cat(ids))
        return dict(idx=None, dist=dist, indptr=None, indices=None, data=gr["data"])
    if kind == "edistance":
        s = prepare(case, seed)
        off = np.asarray(s["offsets"])
        G = off.size - 1
        X = s["X"][s["cells"].long()].double()
        n = X.shape[0]
        grp = torch.from_numpy(np.repeat(np.arange(G), np.diff(off))).cuda()
        nx, Xt = X.square().sum(1), X.t().contiguous()
        S = torch.zeros((G, G), dtype=torch.float64, device="cuda")
        step = max(1, int(2e8) // n)
        for a in range(0, n, step):
            part = torch.addmm(nx[None, :], X[a:a + step], Xt, alpha=-2.0).add_(nx[a:a + step, None])
            part = part.clamp_(min=0.0).sqrt_()
            r = torch.arange(part.shape[0], device="cuda")
            part[r, r + a] = 0.0
            cols = torch.zeros((part.shape[0], G), dtype=torch.float64, device="cuda").index_add_(1, grp, part)
            S.index_add_(0, grp[a:a + step], cols)
        m = torch.from_numpy(np.diff(off)).cuda().double()
        pairs = m[:, None] * m[None, :]
        pairs.diagonal().copy_(m * (m - 1))
        D = S / pairs
        w = D.diagonal()
        return dict(E=2 * D - (w[:, None] + w[None, :]), D=D)
    if kind == "pca":
        s = prepare(case, seed)
        ptr, cols, vals = s["csr"]
        n, p, k = case["n"], case["genes"], case["k"]
        rows = torch.repeat_interleave(torch.arange(n, device="cuda"), ptr[1:] - ptr[:-1])
        S = torch.zeros((p, p), dtype=torch.float64, device="cuda")
        tot = torch.zeros(p, dtype=torch.float64, device="cuda")
        dense = []
        for a in range(0, n, 50000):
            b = min(n, a + 50000)
            lo, hi = int(ptr[a]), int(ptr[b])
            x = torch.zeros((b - a, p), dtype=torch.float64, device="cuda")
            x[rows[lo:hi] - a, cols[lo:hi].long()] = vals[lo:hi].double()
            S += x.t() @ x
            tot += x.sum(0)
            dense.append(x)
        mean = tot / n
        C = (S - n * mean[:, None] * mean[None, :]) / (n - 1)
        ev, V = np.linalg.eigh(C.cpu().numpy())
        ev, V = ev[::-1][:k].copy(), V[:, ::-1][:, :k].copy()
        V *= np.sign(V[np.abs(V).argmax(0), np.arange(k)])[None, :]
        V = torch.from_numpy(V).cuda()
        scores = torch.cat([x @ V for x in dense]) - mean @ V
        return dict(mean=mean, evals=torch.from_numpy(ev), loadings=V, scores=scores)
    # the router's weights live in the library; a layout follows its own rounding and labels are whole numbers
    return None
