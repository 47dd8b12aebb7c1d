"""Rows that no list certifies, where the norms spread too far for the split screen.

One near-zero row sends the call to the FP32 chain; an offset common to the other
rows makes their distances small beside the keys' error bound, so that many rows
are searched again, in that chain's keys.  The answers are the oracle's, at both
kinds of packing (norm folded into the chain or added after it) and at ragged
block counts, and the second search stays cheaper than the first.
"""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc
from tests.parity import compare_knn

pytestmark = pytest.mark.gpu


def rows(n, d, offset, scale=1.0):
    X = np.random.default_rng(n + d).standard_normal((n, d)).astype(np.float32) + np.float32(offset)
    X[7] *= np.float32(2.0 ** -25)
    return (X * np.float32(scale)).astype(np.float32)


# (in all but the last, whose keys cannot be bounded, most rows searched again are answered without the exhaustive scan)
@pytest.mark.parametrize("n,d,offset,scale", [(3001, 50, 130, 1.0), (20000, 50, 90, 1.0), (3001, 7, 300, 1.0),
                                              (3001, 64, 110, 1.0), (3001, 96, 82, 1.0), (2003, 256, 43, 1.0),
                                              (1503, 50, 140, 2.0 ** -40), (1503, 50, 130, 2.0 ** 54)])
def test_answers(oracle_mod, n, d, offset, scale):
    X = rows(n, d, offset, scale)
    ws = rsc.Workspace("cuda")
    idx, dist = rsc.knn(torch.from_numpy(X).cuda(), 15, workspace=ws)
    st = rsc.read_knn_stats(ws)
    again = rsc.read_knn_escalated(ws, n, n, d, 15)
    print(f"[wide] n={n} d={d} {st}", flush=True)
    assert again.size > 32  # the case is about them
    assert scale > 1 or st["rescanned_rows"] < max(again.size / 2, again.size - 8192 / 2)
    assert st["max_err_ratio"] < 1.0
    at = np.unique(np.concatenate([again[:150], again[-50:], np.arange(20)]))
    io, _, do = oracle_mod.knn_rows(X, at, 15)
    res = compare_knn(X, at, idx.cpu().numpy()[at], dist.cpu().numpy()[at], io, do, oracle_mod, 15)
    assert res["exact_rows"] + res["near_tie_rows"] == at.size


def test_cost():
    n = 60000
    X = torch.from_numpy(rows(n, 50, 80)).cuda()
    ws = rsc.Workspace("cuda")
    rsc.knn(X, 15, workspace=ws)
    assert rsc.read_knn_stats(ws)["escalated_rows"] > 8192
    rsc.profile_enable(True)
    rsc.profile_reset()
    try:
        rsc.knn(X, 15, workspace=ws)
        torch.cuda.synchronize()
        first, again = rsc.profile_get("screen_wide")[0], rsc.profile_get("screen_escalate")[0]
    finally:
        rsc.profile_enable(False)
    print(f"[wide] first {first:.2f} ms, again {again:.2f} ms", flush=True)
    assert again < first
