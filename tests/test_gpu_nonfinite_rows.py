"""Rows with NaN or infinite values are in no answer and hide no other row.

The embedding has to be finite; a row that is not costs its own entry and
nothing else.  One cluster of rows, so that the neighbours of a query lie in
many segments of the spatial order: the finite rows' answers are those of the
finite rows alone, in every form that the split screen serves.
"""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu

NEGATIVE_NAN = np.array([0xFFC00000], np.uint32).view(np.float32)[0]


def rows(n, d, bad, seed):
    """n rows, about one in 100 of them not finite; the finite ones' positions."""
    gen = torch.Generator().manual_seed(seed)
    X = torch.randn((n, d), generator=gen).numpy()
    at = np.unique(torch.randint(0, n, (n // 100,), generator=gen).numpy())
    X[at, at % d] = bad
    return torch.from_numpy(X).cuda(), torch.from_numpy(np.setdiff1d(np.arange(n), at)).cuda()


def compare(idx, dist, want, wdist, keep, square=True):
    if square:
        idx, dist = idx[keep], dist[keep]
    assert torch.equal(dist, wdist)
    assert torch.equal(idx.long(), keep[want.long()])


BAD = [float("nan"), NEGATIVE_NAN, float("inf"), -float("inf")]


@pytest.mark.parametrize("bad", BAD, ids=["nan", "negative nan", "inf", "negative inf"])
@pytest.mark.parametrize("n,precision", [(3000, rsc.RSC_FP32), (20000, rsc.RSC_FP32), (20000, rsc.RSC_BF16)])
def test_search(n, precision, bad):
    X, keep = rows(n, 8, bad, seed=n)
    if precision == rsc.RSC_BF16:
        X = X.bfloat16().float()
    ws = rsc.Workspace("cuda")
    idx, dist = rsc.knn(X, 15, precision=precision, workspace=ws)
    want, wdist = rsc.knn(X[keep].contiguous(), 15, precision=precision)
    compare(idx, dist, want, wdist, keep)
    assert rsc.read_knn_stats(ws)["rescanned_rows"] < n // 50  # the others are not scanned exhaustively


@pytest.mark.parametrize("bad", BAD, ids=["nan", "negative nan", "inf", "negative inf"])
def test_foreign_queries(bad):
    X, keep = rows(60000, 8, bad, seed=1)
    Q, kept = rows(5003, 8, bad, seed=2)
    idx, dist = rsc.knn(X, 15, Q=Q)
    want, wdist = rsc.knn(X[keep].contiguous(), 15, Q=Q[kept].contiguous())
    compare(idx[kept], dist[kept], want, wdist, keep, square=False)


@pytest.mark.parametrize("bad", BAD[:2], ids=["nan", "negative nan"])
def test_batched_samples(bad):
    sizes = [300, 1000, 2049]
    off = np.concatenate([[0], np.cumsum(sizes)])
    X, keep = rows(int(off[-1]), 8, bad, seed=3)
    kept = np.searchsorted(keep.cpu().numpy(), off)
    idx, dist = rsc.knn_batched(X, off, 15)
    want, wdist = rsc.knn_batched(X[keep].contiguous(), kept, 15)
    compare(idx, dist, want, wdist, keep)
