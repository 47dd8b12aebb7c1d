"""The split FP16 screen of the exact path: every contraction geometry at its
edges, the spatially ordered scan at a ragged row count, and inputs whose norms
spread too far for it (they take the FP32 chain).  The answer is exact
whichever screen ran, so ids and float32 distances equal the oracle's."""

import numpy as np
import pytest

import synth
from tests.parity import compare_knn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rsc():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_02402_amd as rsc

    rsc.load()
    return rsc


def run(rsc, X, k, Q=None, **kw):
    import torch

    ws = rsc.Workspace()
    Qt = None if Q is None else torch.from_numpy(Q).cuda()
    idx, dist = rsc.knn(torch.from_numpy(X).cuda(), k, Q=Qt, workspace=ws, **kw)
    st = rsc.read_knn_stats(ws)
    assert st["max_err_ratio"] < 1.0, "screen error exceeded its certified bound"
    return idx.cpu().numpy(), dist.cpu().numpy(), st


def check(rsc, oracle_mod, X, k, rows=None):
    rows = np.arange(X.shape[0]) if rows is None else rows
    idx, dist, st = run(rsc, X, k)
    io, _, do = oracle_mod.knn_rows(X, rows, k)
    res = compare_knn(X, rows, idx[rows], dist[rows], io, do, oracle_mod, k)
    assert res["exact_rows"] + res["near_tie_rows"] == len(rows)
    return st


# both sides of every geometry's widest d (16 q + 4, 16 q + 9), the plain multiples of 16 and the largest d
@pytest.mark.parametrize("d", [1, 4, 5, 9, 10, 16, 20, 21, 25, 26, 36, 37, 41, 42, 52, 53, 57, 58, 68, 69, 84, 85, 100,
                               116, 117, 132, 133, 164, 165, 196, 197, 228, 229, 256])
@pytest.mark.parametrize("n,k", [(321, 7), (577, 33)])
def test_geometries(rsc, oracle_mod, d, n, k):
    print(f"[split] d={d} n={n} k={k}", flush=True)
    check(rsc, oracle_mod, synth.mixture(n, d=d, n_clusters=4, seed=d * 7 + n), k)


# from 16384 rows on they are screened in a spatial order: ragged last block and last query tile, one and two ranges
@pytest.mark.parametrize("n", [16384, 16385, 33001, 70017])
def test_ordered_rows(rsc, oracle_mod, n):
    print(f"[split] ordered n={n}", flush=True)
    X = synth.mixture(n, d=50, n_clusters=12, seed=n)
    check(rsc, oracle_mod, X, 15, np.unique(np.concatenate([np.arange(40), np.arange(n - 40, n),
                                                            synth.sample_rows(n, 200, seed=3)])))


@pytest.mark.parametrize("spread", [2.0 ** -20, 2.0 ** -15, 2.0 ** -10])
def test_norms_far_apart(rsc, oracle_mod, spread):
    """Half of the rows `spread` times as long as the others: below 2^-16 of the largest norm the FP32 chain runs,
    above it the split screen; either way few rows may need the exhaustive scan."""
    print(f"[split] spread={spread}", flush=True)
    X = synth.mixture(1500, d=50, n_clusters=6, seed=5)
    X[750:] *= np.float32(spread)
    st = check(rsc, oracle_mod, X, 15)
    assert st["rescanned_rows"] <= 15


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -45, 2.0 ** 40, 2.0 ** 62])
def test_scales(rsc, oracle_mod, scale):
    print(f"[split] scale={scale}", flush=True)
    check(rsc, oracle_mod, synth.mixture(900, d=20, n_clusters=5, seed=8) * np.float32(scale), 10)


@pytest.mark.parametrize("factor", [1e-6, 1e-3, 1e3, 1e6])
def test_queries_of_another_size(rsc, oracle_mod, factor):
    print(f"[split] query factor={factor}", flush=True)
    R = synth.mixture(2001, d=50, n_clusters=8, seed=11)
    Q = synth.mixture(333, d=50, n_clusters=8, seed=12) * np.float32(factor)
    idx, dist, _ = run(rsc, R, 15, Q=Q)
    io, _, do = oracle_mod.knn(R, 15, Q=Q)
    res = compare_knn(None, np.arange(333), idx, dist, io, do, oracle_mod, 15, self_mode=False,
                      pair_dist=lambda _, i, j: np.sqrt(((Q[i].astype(np.float64) - R[j]) ** 2).sum(1)))
    assert res["exact_rows"] + res["near_tie_rows"] == 333


@pytest.mark.parametrize("spread", [1.0, 2.0 ** -20])
def test_batched_samples(rsc, oracle_mod, spread):
    """Ragged samples around the tile sizes; with one sample 2^-20 as long as the others the FP32 chain answers."""
    import torch

    print(f"[split] batched spread={spread}", flush=True)
    sizes = [15, 16, 31, 33, 255, 256, 257, 700, 2049]
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = np.concatenate([synth.mixture(n, d=50, n_clusters=3, seed=n) for n in sizes])
    X[off[5]:off[7]] *= np.float32(spread)
    idx, dist = rsc.knn_batched(torch.from_numpy(X).cuda(), off, 15)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    for s in range(len(sizes)):
        io, _, do = oracle_mod.knn(X[off[s]:off[s + 1]], 15)
        np.testing.assert_array_equal(idx[off[s]:off[s + 1]] - off[s], io)
        np.testing.assert_array_equal(dist[off[s]:off[s + 1]], np.asarray(do).astype(np.float32))


@pytest.mark.parametrize("spread", [1.0, 2.0 ** -20])
@pytest.mark.parametrize("d,k", [(50, 15), (9, 5), (64, 20), (100, 40), (128, 15)])
def test_probed_partitions(rsc, oracle_mod, d, k, spread):
    import torch
    from oracle import partition

    print(f"[split] probed d={d} k={k} spread={spread}", flush=True)
    n, P = 2500, 37
    X = synth.mixture(n, d=d, n_clusters=5, seed=d)
    X[::2] *= np.float32(spread)
    labels = synth.random_labels(n, P, 3)
    off, perm = partition.inverted_lists(labels, P)
    pr = synth.random_probes(n, P, 9, 4, own=labels)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, off, perm.astype(np.int32), pr)]
    idx, dist, route, _ = rsc.knn_probed(dev[0], k, *dev[1:])
    route = route.cpu().numpy()
    io, _, do = partition.routed_knn(X, k, off, perm, pr, exact_rows=route != 0)
    np.testing.assert_array_equal(idx.cpu().numpy(), io)
    np.testing.assert_array_equal(dist.cpu().numpy(), np.asarray(do).astype(np.float32))
