"""The BF16 form where bounds do not help: the plain BF16 screen answers in the pruned one's place.

Tiles spread over the queries tell how much of the references the bounds leave to
visit, and the verdict goes to one screen or the other.  Rows that BF16 holds
exactly give the exact search's answer whichever screen ran, so
ids and distances are compared bit for bit: rows without clusters (plain), well
separated ones (pruned), and one large cluster among small ones, near the line;
one range and several, square and rectangular, ragged last tiles, widths at the
edges of both packings, and a second call in the same workspace.
"""

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


def rows(n, d, clusters, seed, mixed=False):
    """Rows around far centres (none: one cluster); mixed: around the first of them lie as many as around all others."""
    gen = torch.Generator("cuda").manual_seed(seed)
    X = torch.randn((n, d), generator=gen, device="cuda")
    if clusters:
        at = torch.randint(0, clusters, (n,), generator=gen, device="cuda")
        if mixed:
            at[torch.rand((n,), generator=gen, device="cuda") < 0.7] = 0
        X += 20 * torch.randn((clusters, d), generator=torch.Generator("cuda").manual_seed(d), device="cuda")[at]
    return X.bfloat16().float()


def plain_answered(ws):
    """KnnCounters.verdict, the eighth word of the workspace, is kPlain."""
    return int(ws.buf[:64].view(torch.int32)[7]) == 2


def same(X, k, **kw):
    """Compares the BF16 form with the exact one; whether the plain screen answered."""
    ws = rsc.Workspace("cuda")
    idx, dist = rsc.knn(X, k, precision=rsc.RSC_BF16, workspace=ws, **kw)
    plain = plain_answered(ws)
    assert rsc.read_knn_stats(ws)["max_err_ratio"] < 1e-3
    again, _ = rsc.knn(X, k, precision=rsc.RSC_BF16, workspace=ws, **kw)
    want, wdist = rsc.knn(X, k, **kw)
    assert torch.equal(idx, want)
    assert torch.equal(dist, wdist)
    assert torch.equal(again, want)
    return plain


@pytest.mark.parametrize("n,d,k", [(25000, 50, 15), (40003, 13, 30), (66000, 29, 10), (140001, 50, 15), (33000, 126, 5)])
def test_square(n, d, k):
    assert same(rows(n, d, 0, 1), k)
    assert not same(rows(n, d, 30, 2), k)
    same(rows(n, d, 30, 3, mixed=True), k)


@pytest.mark.parametrize("nq,n", [(16000, 120000), (70000, 30000), (300001, 20000)])
@pytest.mark.parametrize("clusters,mixed", [(0, False), (30, False), (30, True)])
def test_rectangular(nq, n, clusters, mixed):
    same(rows(n, 50, clusters, 3, mixed), 15, Q=rows(nq, 50, clusters, 4, mixed))


@pytest.mark.parametrize("nq,n", [(2999, 100000), (3000, 100000), (4499, 400000), (4500, 400000)])
def test_few_queries(nq, n):
    same(rows(n, 50, 30, 5), 15, Q=rows(nq, 50, 30, 6))


@pytest.mark.parametrize("n,d", [(16500, 50), (40000, 128)])
def test_not_sampled(n, d):
    """Short ranges and the widest rows stay with the pruned screen."""
    assert not same(rows(n, d, 0, 7), 15)


def test_repeats_itself():
    """Which screen answers, and hence an answer that is not exact, is the same in every call."""
    X = torch.randn((60000, 50), generator=torch.Generator("cuda").manual_seed(8), device="cuda")
    first = rsc.knn(X, 30, precision=rsc.RSC_BF16)
    for _ in range(3):
        again = rsc.knn(X, 30, precision=rsc.RSC_BF16)
        assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])
