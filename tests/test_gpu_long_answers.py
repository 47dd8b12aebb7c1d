"""Answers longer than 64: enough lists that they hold the nearest rows, and no spatial order over few rows."""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc
from tests.parity import compare_knn
from tests.test_gpu_few_queries import ordered, rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,k", [(4000, 10, 255), (10000, 10, 255), (4000, 50, 255), (5000, 20, 129), (20000, 20, 200)])
def test_lists_suffice(oracle_mod, n, d, k):
    """m nearest in 2 P lists of 32, P >= m / 25: a list is to hold 12.5 of them on average, and more than 32 in one of
    1e6 (Poisson).  20000 rows of 22 lists at most: 0.4 rows expected, none here."""
    X = rows(n, d, n)
    ws = rsc.Workspace("cuda")
    idx, dist = rsc.knn(X, k, workspace=ws)
    assert rsc.read_knn_stats(ws)["escalated_rows"] <= 3
    Xn, at = X.cpu().numpy(), np.arange(0, n, n // 40)
    io, _, do = oracle_mod.knn_rows(Xn, at, k)
    res = compare_knn(Xn, at, idx.cpu().numpy()[at], dist.cpu().numpy()[at], io, do, oracle_mod, k)
    assert res["exact_rows"] + res["near_tie_rows"] == at.size


@pytest.mark.parametrize("n,k,order", [(20000, 65, True), (20000, 66, False), (20479, 66, False), (20480, 66, True)])
def test_order(oracle_mod, n, k, order):
    X = rows(n, 50, 3)
    ws = rsc.Workspace("cuda")
    assert ordered(lambda: rsc.knn(X, k, workspace=ws)) == order
    idx, dist = rsc.knn(X, k, workspace=ws)
    Xn, at = X.cpu().numpy(), np.arange(0, n, n // 40)
    io, _, do = oracle_mod.knn_rows(Xn, at, k)
    res = compare_knn(Xn, at, idx.cpu().numpy()[at], dist.cpu().numpy()[at], io, do, oracle_mod, k)
    assert res["exact_rows"] + res["near_tie_rows"] == at.size
