"""The pruned exact screen (16384 references and more): rows in a spatial
order, segments skipped by their bounds.  The answer equals the exhaustive
oracle's on data that prunes well (separate clusters), not at all (one
cluster), badly (rows far from every pivot, tiny clusters, duplicates), for
several list lengths, ranges and query shapes, and for flagged rows that
collect their neighbours."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsc():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02402_amd as rsc

    rsc.load()
    return rsc


def rows_of(n, seed, count=150):
    return np.unique(np.concatenate([np.arange(20), np.arange(n - 20, n), synth.sample_rows(n, count, seed=seed)]))


def check(rsc, oracle_mod, X, k, metric="euclidean", extra=()):
    import torch

    n = X.shape[0]
    ws = rsc.Workspace()
    m = rsc.RSC_COSINE if metric == "cosine" else rsc.RSC_EUCLIDEAN
    idx, dist = rsc.knn(torch.from_numpy(X).cuda(), k, metric=m, workspace=ws)
    st = rsc.read_knn_stats(ws)
    assert st["max_err_ratio"] < 1.0
    rows = np.unique(np.concatenate([rows_of(n, seed=k), np.asarray(extra, dtype=np.int64)])).astype(np.int64)
    io, _, do = oracle_mod.knn_rows(X, rows, k, metric=metric)
    np.testing.assert_array_equal(idx.cpu().numpy()[rows], io)
    np.testing.assert_array_equal(dist.cpu().numpy()[rows], np.asarray(do).astype(np.float32))
    return st


@pytest.mark.parametrize("n,d,k,clusters", [
    (16384, 50, 15, 20), (16385, 50, 15, 1), (20011, 2, 10, 8), (20011, 9, 16, 30), (17000, 10, 17, 5),
    (30001, 64, 33, 60), (18000, 128, 50, 40), (16500, 256, 64, 10), (40000, 33, 15, 700), (131072, 20, 15, 100),
    (300007, 12, 15, 50),
])
@pytest.mark.parametrize("metric", ["euclidean", "cosine"])
def test_shapes(rsc, oracle_mod, n, d, k, clusters, metric):
    print(f"[pruned] n={n} d={d} k={k} clusters={clusters} {metric}", flush=True)
    check(rsc, oracle_mod, synth.mixture(n, d=d, n_clusters=clusters, seed=n + d), k, metric)


def test_outliers_duplicates_and_tiny_clusters(rsc, oracle_mod):
    print("[pruned] outliers", flush=True)
    X = synth.mixture(25000, d=50, n_clusters=6, seed=1)
    rng = np.random.default_rng(2)
    far = rng.choice(25000, 60, replace=False)
    X[far[:20]] = rng.standard_normal((20, 50)) * 300.0              # rows alone, far from everything
    X[far[20:40]] = X[far[20]] + rng.standard_normal((20, 50)) * 1e-3  # a cluster of 20
    X[far[40:60]] = X[far[40]]                                         # 20 duplicates
    X[:3] = 0.0
    check(rsc, oracle_mod, X.astype(np.float32), 15, extra=far)


def test_common_offset_collects_or_rescans(rsc, oracle_mod):
    """A large common offset inflates the key error: rows fail the certificate and collect, or are rescanned."""
    print("[pruned] offset", flush=True)
    X = synth.mixture(17000, d=50, n_clusters=300, seed=4) + np.float32(60.0)
    st = check(rsc, oracle_mod, X, 15)
    assert st["escalated_rows"] > 0


def test_norms_far_apart(rsc, oracle_mod):
    """Marked wide: the FP32 chain, its flagged rows collected in float64."""
    print("[pruned] wide", flush=True)
    X = synth.mixture(17000, d=50, n_clusters=30, seed=6)
    X[::2] *= np.float32(2.0 ** -20)
    check(rsc, oracle_mod, X, 15)


@pytest.mark.parametrize("nq,n,d,k", [(20000, 20000, 50, 15), (5003, 60000, 50, 15), (257, 1000003, 16, 10),
                                      (30000, 16384, 20, 40)])
@pytest.mark.parametrize("far", [False, True])
def test_rectangular(rsc, oracle_mod, nq, n, d, k, far):
    import torch

    print(f"[pruned] nq={nq} n={n} d={d} k={k} far={far}", flush=True)
    R = synth.mixture(n, d=d, n_clusters=25, seed=7)
    Q = synth.mixture(nq, d=d, n_clusters=9 if far else 25, seed=8 if far else 7)  # far: other centres
    idx, dist = rsc.knn(torch.from_numpy(R).cuda(), k, Q=torch.from_numpy(Q).cuda())
    rows = rows_of(nq, seed=9, count=80)
    io, _, do = oracle_mod.knn(R, k, Q=Q[rows])
    np.testing.assert_array_equal(idx.cpu().numpy()[rows], io)
    np.testing.assert_array_equal(dist.cpu().numpy()[rows], np.asarray(do).astype(np.float32))
