"""Few foreign queries, and long answers over few rows: the plain scan, without an order of the references."""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


def ordered(f):
    """Whether a call sorts the references."""
    f()
    rsc.profile_enable(True)
    rsc.profile_reset()
    try:
        f()
        torch.cuda.synchronize()
        return rsc.profile_get("query_order")[1] > 0
    finally:
        rsc.profile_enable(False)


def rows(n, d, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    X = torch.randn((n, d), generator=gen, device="cuda")
    return X + 3 * torch.randn((30, d), generator=torch.Generator("cuda").manual_seed(d), device="cuda")[
        torch.randint(0, 30, (n,), generator=gen, device="cuda")]


@pytest.mark.parametrize("nq,n,d,k", [(300, 1000000, 20, 15), (2000, 500000, 50, 15), (3999, 70000, 50, 30),
                                      (4000, 70000, 50, 30), (3999, 70001, 9, 100)])
def test_queries(nq, n, d, k):
    X, Q = rows(n, d, 1), rows(nq, d, 2)
    ws = rsc.Workspace("cuda")
    assert ordered(lambda: rsc.knn(X, k, Q=Q, workspace=ws)) == (nq >= 4000)
    idx, dist = rsc.knn(X, k, Q=Q, workspace=ws)
    Xn = X.cpu().numpy()
    for i in (0, 1, nq // 2, nq - 1):
        far = ((Xn - Q[i].cpu().numpy().astype(np.float64)) ** 2).sum(1)
        at = idx[i].cpu().numpy()
        assert len(set(at.tolist())) == k
        want = np.sqrt(np.sort(np.partition(far, k)[:k]))
        np.testing.assert_allclose(dist[i].cpu().numpy(), want, rtol=3e-7)  # rounded to float32
        np.testing.assert_allclose(np.sqrt(far[at]), want, rtol=3e-7)
