"""A batch of few query tiles splits its references, as one matrix of that size does."""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


def rows(n, d, seed):
    return torch.randn((n, d), generator=torch.Generator("cuda").manual_seed(seed), device="cuda")


# one range to four: the largest batch that splits by each number, and one tile more; samples that keep one range
@pytest.mark.parametrize("sizes", [[32 * 256], [63 * 256, 41], [41, 65 * 256], [85 * 256 - 7], [86 * 256], [128 * 256 - 31],
                                   [129 * 256], [31 * 32, 64 * 32, 63 * 32, 96 * 32, 45, 128 * 32 + 1], [700, 40, 9000]])
@pytest.mark.parametrize("d,k", [(50, 15), (20, 40)])
def test_answers(sizes, d, k):
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = rows(int(off[-1]), d, len(sizes))
    idx, dist = rsc.knn_batched(X, off, k)
    for s, n in enumerate(sizes):
        one, odist = rsc.knn(X[off[s]:off[s + 1]].contiguous(), k)
        assert torch.equal(idx[off[s]:off[s + 1]] - int(off[s]), one)
        assert torch.equal(dist[off[s]:off[s + 1]], odist)


def test_time():
    """12000 rows: 47 tiles of 375 blocks.  The plain search takes 3 ranges of 125; a single range takes 3 times as long."""
    n, took = 12000, []
    X = rows(n, 50, 1)
    ws = rsc.Workspace("cuda")
    for f, name in ((lambda: rsc.knn(X, 30, workspace=ws), "screen_fp32"),
                    (lambda: rsc.knn_batched(X, np.array([0, n]), 30, workspace=ws), "screen_batched")):
        f()
        rsc.profile_enable(True)
        try:
            best = np.inf
            for _ in range(9):
                rsc.profile_reset()
                f()
                torch.cuda.synchronize()
                best = min(best, rsc.profile_get(name)[0])
        finally:
            rsc.profile_enable(False)
        took.append(best)
    print(f"[batched] one matrix {took[0]:.3f} ms, as a batch {took[1]:.3f}", flush=True)
    assert took[1] < 1.5 * took[0]
