"""The pairs that the benchmark reports for the pruned search: all of them without clusters, few with."""

import pytest
import torch

import bench
import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,precision", [(15, rsc.RSC_FP32), (30, rsc.RSC_FP32), (15, rsc.RSC_BF16)])
def test_pairs(k, precision):
    n, d = 40000, 50
    gen = torch.Generator("cuda").manual_seed(1)
    X = torch.randn((n, d), generator=gen, device="cuda")
    ws = rsc.Workspace("cuda")
    rsc.knn(X, k, precision=precision, workspace=ws)
    assert n * n <= bench.screened_pairs(ws, n) < 1.05 * n * n  # (whole tiles and segments)
    X += 20 * torch.randn((20, d), generator=gen, device="cuda")[torch.randint(0, 20, (n,), generator=gen, device="cuda")]
    rsc.knn(X, k, precision=precision, workspace=ws)
    # a tile's rows lie in one cluster of 20, or two; segments of 32 rows and more at the clusters' edges
    assert 0 < bench.screened_pairs(ws, n) < 0.2 * n * n
