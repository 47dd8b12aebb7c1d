"""The BF16 form on the pruned screen (16384 references and more).

Rows that BF16 holds exactly lose nothing to the rounding, so every list of 32
keys contains the true neighbours up to k = 31 and the answer is the exact
search's, bit for bit: for widths at the edges of the 16-slot chunks, ranges,
rectangular queries, and norms so far apart that the FP32 chain takes over.
"""

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


def rows(n, d, clusters, seed, centres=None):
    gen = torch.Generator("cuda").manual_seed(seed)
    c = torch.randn((clusters, d), generator=gen, device="cuda") * 5 if centres is None else centres
    at = torch.randint(0, clusters, (n,), generator=gen, device="cuda")
    return (c[at] + torch.randn((n, d), generator=gen, device="cuda")).bfloat16().float(), c


def same(X, k, **kw):
    idx, dist = rsc.knn(X, k, precision=rsc.RSC_BF16, **kw)
    want, wdist = rsc.knn(X, k, **kw)
    assert torch.equal(idx, want)
    assert torch.equal(dist, wdist)


@pytest.mark.parametrize("d", [3, 12, 13, 28, 29, 50, 60, 61, 77, 92, 108, 124, 125, 128])
@pytest.mark.parametrize("n,k,clusters", [(16384, 15, 20), (40003, 30, 7), (20000, 1, 1)])
def test_exact_rows(n, k, clusters, d):
    X, _ = rows(n, d, clusters, seed=d)
    same(X, k)


@pytest.mark.parametrize("nq,n", [(20000, 20000), (5003, 60000), (257, 1000003)])
def test_rectangular(nq, n):
    X, c = rows(n, 50, 30, seed=1)
    Q, _ = rows(nq, 50, 30, seed=2, centres=c)
    same(X, 15, Q=Q)


def test_norms_far_apart():
    X, _ = rows(20000, 50, 20, seed=3)
    X[::7] *= 2.0 ** -20
    X[5] *= 2.0 ** 10
    same(X, 15)


@pytest.mark.parametrize("k", [10, 50])
def test_recall(k):
    X = rows(60000, 50, 20, seed=4)[0]
    X = X + 0.01 * torch.randn(X.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    for metric in (rsc.RSC_EUCLIDEAN, rsc.RSC_COSINE):
        idx, _ = rsc.knn(X, k, precision=rsc.RSC_BF16, metric=metric)
        want, _ = rsc.knn(X, k, metric=metric)
        hit = (idx[:, :, None] == want[:, None, :]).any(2).double().mean().item()
        assert hit > 0.999


@pytest.mark.parametrize("metric", [rsc.RSC_EUCLIDEAN, rsc.RSC_COSINE])
@pytest.mark.parametrize("spread", [1.0, 2.0 ** -20])
def test_error_statistic(metric, spread):
    """The statistic is the relative error of a screened key, |key - d^2 + x^2| over 2 |x| |y| + |y|^2 (cosine: the
    error itself).  Rounding both rows to BF16 moves a key by at most 2^-9 of each term: 2 (2^-9 + 2^-9) |x| |y| and
    2 2^-9 |y|^2, so it stays below 2^-7 (cosine: below twice that of 3 terms), and it is not zero."""
    X = rows(20000, 50, 20, seed=6)[0]
    X = 40 * (X + 0.01 * torch.randn(X.shape, generator=torch.Generator("cuda").manual_seed(7), device="cuda"))
    X[::7] *= spread
    ws = rsc.Workspace("cuda")
    rsc.knn(X, 15, precision=rsc.RSC_BF16, metric=metric, workspace=ws)
    ratio = rsc.read_knn_stats(ws)["max_err_ratio"]
    assert 2.0 ** -16 < ratio < (2.0 ** -7 if metric == rsc.RSC_EUCLIDEAN else 2.0 ** -5)
