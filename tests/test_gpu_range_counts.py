"""Reference ranges of the pruned search over few query tiles: the last round of workgroups is not nearly empty."""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc
from tests.parity import compare_knn

pytestmark = pytest.mark.gpu


def rows(n, d):
    return torch.randn((n, d), generator=torch.Generator("cuda").manual_seed(n), device="cuda")


def test_rounds():
    """Rows without clusters, one workgroup a CU.  16384 rows: 64 tiles, 4 ranges of 4096 rows, one round.  20000: 79
    tiles, and 3 ranges take one round of 6667 rows (1.63 times as long), 4 take two of 5000 (2.44 times)."""
    took = []
    for n in (16384, 20000):
        X, ws = rows(n, 50), rsc.Workspace("cuda")
        rsc.knn(X, 15, workspace=ws)
        rsc.profile_enable(True)
        try:
            best = np.inf
            for _ in range(9):
                rsc.profile_reset()
                rsc.knn(X, 15, workspace=ws)
                torch.cuda.synchronize()
                best = min(best, rsc.profile_get("screen_fp32")[0])
        finally:
            rsc.profile_enable(False)
        took.append(best)
    print(f"[ranges] 16384 rows {took[0]:.3f} ms, 20000 {took[1]:.3f}", flush=True)
    assert took[1] < 2.0 * took[0]


# tiles of 256 queries around the sizes where the ranges change: 64, 65, 85, 86, 128, 129, 170, 171, 256, 257
@pytest.mark.parametrize("n", [16384, 16385, 21760, 21761, 32768, 32769, 43520, 43521, 65536, 65537])
@pytest.mark.parametrize("d,k", [(10, 15), (50, 60)])
def test_answers(oracle_mod, n, d, k):
    X = rows(n, d)
    idx, dist = rsc.knn(X, k)
    Xn, at = X.cpu().numpy(), np.unique(np.concatenate([np.arange(0, n, n // 25), [n - 1]]))
    io, _, do = oracle_mod.knn_rows(Xn, at, k)
    res = compare_knn(Xn, at, idx.cpu().numpy()[at], dist.cpu().numpy()[at], io, do, oracle_mod, k)
    assert res["exact_rows"] + res["near_tie_rows"] == at.size
