"""The rerank of short answers at the edges of its variants: answers of 31 to
65 neighbours, few and many candidates per row, odd and even row lengths and
bases, ties beyond a wave, zero rows.  Ids and float32 distances equal the
oracle's (both are exact)."""

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


def same(rsc, oracle_mod, X, k, metric="euclidean", shift=0, Q=None):
    import torch

    def dev(A):
        flat = torch.zeros(A.size + shift, dtype=torch.float32, device="cuda")
        flat[shift:] = torch.from_numpy(A).reshape(-1)
        return flat[shift:].view(A.shape)  # base 4 * shift bytes past an allocation

    ws = rsc.Workspace()
    m = rsc.RSC_COSINE if metric == "cosine" else rsc.RSC_EUCLIDEAN
    idx, dist = rsc.knn(dev(X), k, Q=None if Q is None else dev(Q), metric=m, workspace=ws)
    assert rsc.read_knn_stats(ws)["max_err_ratio"] < 1.0
    if Q is None:
        io, _, do = oracle_mod.knn_rows(X, np.arange(X.shape[0]), k, metric=metric)
    else:
        io, _, do = oracle_mod.knn(X, k, Q=Q)
    np.testing.assert_array_equal(idx.cpu().numpy(), io)
    np.testing.assert_array_equal(dist.cpu().numpy(), np.asarray(do).astype(np.float32))


@pytest.mark.parametrize("d", [1, 31, 32, 33, 50, 63, 64, 66])
@pytest.mark.parametrize("n,k", [(40, 15), (700, 2), (700, 16), (700, 17), (900, 32), (900, 33), (900, 34), (900, 64),
                                 (900, 65), (900, 66), (3000, 15), (3000, 50)])
def test_answer_and_list_sizes(rsc, oracle_mod, n, d, k):
    print(f"[rerank] n={n} d={d} k={k}", flush=True)
    same(rsc, oracle_mod, synth.mixture(n, d=d, n_clusters=4, seed=n + d + k), k)


# 600 rows: two ranges, 128 candidates in lists of 32; 257: one range, 64
@pytest.mark.parametrize("n", [257, 600])
@pytest.mark.parametrize("k", [17, 32, 33, 34, 40, 64])
@pytest.mark.parametrize("metric", ["euclidean", "cosine"])
def test_candidates_per_lane(rsc, oracle_mod, n, k, metric):
    print(f"[rerank] n={n} k={k} {metric}", flush=True)
    same(rsc, oracle_mod, synth.mixture(n, d=50, n_clusters=4, seed=n + k), k, metric=metric)


@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("d", [49, 50])
def test_unaligned_rows(rsc, oracle_mod, d, shift):
    print(f"[rerank] d={d} shift={shift}", flush=True)
    same(rsc, oracle_mod, synth.mixture(600, d=d, n_clusters=4, seed=d + shift), 15, shift=shift)


@pytest.mark.parametrize("metric", ["euclidean", "cosine"])
@pytest.mark.parametrize("copies", [20, 70, 300])
def test_ties_and_zero_rows(rsc, oracle_mod, metric, copies):
    print(f"[rerank] {metric} copies={copies}", flush=True)
    X = synth.mixture(1200, d=50, n_clusters=4, seed=copies)
    X[100:100 + copies] = X[99]
    X[700:703] = 0.0
    same(rsc, oracle_mod, X, 15, metric=metric)


@pytest.mark.parametrize("nq", [1, 7, 8, 9, 257])
def test_rectangular(rsc, oracle_mod, nq):
    print(f"[rerank] nq={nq}", flush=True)
    same(rsc, oracle_mod, synth.mixture(1500, d=50, n_clusters=4, seed=1), 20,
         Q=synth.mixture(nq, d=50, n_clusters=4, seed=2))
