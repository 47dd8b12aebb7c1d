"""The exact search with lists of 32 where bounds do not help: the unpruned screen answers in the pruned one's place.

Tiles spread over the queries tell how much of the references the bounds leave to
visit.  Either screen's answer is exact: it is compared with the oracle on
sampled rows, for rows without clusters (unpruned), well separated ones (pruned)
and near the line; one range and several, square and foreign queries, both
metrics, ragged last tiles, and widths at both ends of the rule.
"""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc
from tests.parity import compare_knn
from tests.test_gpu_rounded_plain import plain_answered

pytestmark = pytest.mark.gpu


def rows(n, d, clusters, spread, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    X = torch.randn((n, d), generator=gen, device="cuda")
    if clusters:
        at = torch.randint(0, clusters, (n,), generator=gen, device="cuda")
        X += spread * torch.randn((clusters, d), generator=torch.Generator("cuda").manual_seed(d), device="cuda")[at]
    return X


def check(oracle_mod, X, k, Q=None):
    """Compares sampled rows with the oracle and a second call with the first; whether the unpruned screen answered."""
    ws = rsc.Workspace("cuda")
    idx, dist = rsc.knn(X, k, Q=Q, workspace=ws)
    plain = plain_answered(ws)
    st = rsc.read_knn_stats(ws)
    print(f"[plain] n={len(X)} d={X.shape[1]} k={k} nq={0 if Q is None else len(Q)} plain={plain} {st}", flush=True)
    assert st["max_err_ratio"] < 1.0
    again = rsc.knn(X, k, Q=Q, workspace=ws)
    assert torch.equal(idx, again[0]) and torch.equal(dist, again[1])
    Xn = X.cpu().numpy()
    if Q is None:
        at = np.unique(np.concatenate([np.arange(0, len(X), len(X) // 60), [len(X) - 1]]))
        io, _, do = oracle_mod.knn_rows(Xn, at, k)
        res = compare_knn(Xn, at, idx.cpu().numpy()[at], dist.cpu().numpy()[at], io, do, oracle_mod, k)
        assert res["exact_rows"] + res["near_tie_rows"] == at.size
    else:
        at = np.unique(np.concatenate([np.arange(0, len(Q), len(Q) // 60), [len(Q) - 1]]))
        got = dist.cpu().numpy()[at].astype(np.float64)
        far = np.stack([((Xn - q) ** 2).sum(-1) for q in Q.cpu().numpy()[at].astype(np.float64)])
        want = np.sqrt(np.partition(far, k - 1, axis=1)[:, :k])
        want.sort(axis=1)
        np.testing.assert_allclose(got, want, rtol=3e-7)  # distances rounded to float32
        found = np.sqrt(np.take_along_axis(far, idx.cpu().numpy()[at].astype(np.int64), 1))
        np.testing.assert_allclose(found, want, rtol=3e-7)
        assert all(len(set(r)) == k for r in idx.cpu().numpy()[at])
    return plain


@pytest.mark.parametrize("n,d,k", [(40003, 25, 30), (40003, 26, 17), (36001, 50, 30), (40000, 50, 100), (33001, 96, 64),
                                   (20000, 128, 17), (34000, 50, 255), (24001, 190, 30), (66000, 35, 20)])
def test_square(oracle_mod, n, d, k):
    assert check(oracle_mod, rows(n, d, 0, 0, 1), k) == (d > 25)
    assert not check(oracle_mod, rows(n, d, 30, 20, 2), k)
    for spread in (1.5, 2.0, 2.5):
        check(oracle_mod, rows(n, d, 20, spread, 3), k)


@pytest.mark.parametrize("nq,n,k", [(20001, 70000, 30), (60000, 20001, 50), (100000, 16500, 17)])
def test_foreign(oracle_mod, nq, n, k):
    assert check(oracle_mod, rows(n, 50, 0, 0, 4), k, rows(nq, 50, 0, 0, 5))
    check(oracle_mod, rows(n, 50, 30, 3, 6), k, rows(nq, 50, 30, 3, 7))


def test_short_lists_are_not_sampled():
    X = rows(60000, 50, 0, 0, 8)
    ws = rsc.Workspace("cuda")
    rsc.knn(X, 16, workspace=ws)
    assert not plain_answered(ws)


def test_cosine():
    X = rows(40000, 50, 0, 0, 9)
    ws = rsc.Workspace("cuda")
    idx, dist = rsc.knn(X, 30, metric=rsc.RSC_COSINE, workspace=ws)
    assert plain_answered(ws)
    at = torch.arange(0, 40000, 500, device="cuda")
    U = X.double() / X.double().norm(dim=1, keepdim=True)
    want = (1 - (U[at] @ U.T)).topk(30, dim=1, largest=False).values
    # (the row itself: 0)
    assert torch.allclose(dist[at].double(), want.clamp(min=0), rtol=3e-7, atol=3e-7)
