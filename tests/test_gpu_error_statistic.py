"""The error statistic's own arithmetic is in 64 bits.

One query at the origin and one reference: the BF16 screen's key is the rounded
row's norm in two BF16 parts, and the statistic |key - ||y||^2| / ||y||^2, known
here to the last bit before it is rounded to float32.
"""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


def bf16(x):
    return torch.tensor(x, dtype=torch.float32).bfloat16().double().numpy()


@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_norm_of_the_reference(seed):
    y = np.random.default_rng(seed).uniform(0.5, 2.0, (1, 128)).astype(np.float32)
    norm = np.float32((bf16(y) ** 2).sum())
    high = np.float32(bf16(norm))
    key = np.float32(high + np.float32(bf16(np.float32(norm - high))))
    exact = (y.astype(np.float64) ** 2).sum()
    want = abs(float(key) - exact) / exact
    ws = rsc.Workspace("cuda")
    _, dist = rsc.knn(torch.from_numpy(y).cuda(), 1, Q=torch.zeros((1, 128), device="cuda"), precision=rsc.RSC_BF16,
                      workspace=ws)
    assert float(dist[0, 0]) == np.float32(np.sqrt(exact))
    # float32 rounds the result once (2^-24), and its terms in 64 bits round it by less than that again
    assert rsc.read_knn_stats(ws)["max_err_ratio"] == pytest.approx(want, rel=2.0 ** -23, abs=0)
