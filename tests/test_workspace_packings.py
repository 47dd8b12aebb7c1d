"""A workspace holds one packing of the references: the split screen's, or the FP32 chain's in its place.

Inputs of either kind, one after the other in the same workspace, and the answers
of longer lists, which read both packings.
"""

import ctypes

import pytest

import paper_2603_02402_amd as rsc


def need(n, d, k, precision=0):
    o = rsc._opts(precision)
    return rsc.load().rsc_knn_workspace_bytes(n, n, d, k, ctypes.byref(o))


@pytest.mark.parametrize("d", [16, 50, 128])
def test_one_packing(d):
    """Bytes a row beside the candidates (two ranges at most: 2 x 32 x 8) and the order (below 64): norms, flags and the
    larger packing, whose rows hold at most 9 values of 4 bytes to 8 dimensions, and 64 bytes of norms and rest."""
    n = 1000000
    assert need(n, d, 15) / n < 2 * 32 * 8 + 64 + 32 + (4 * d * 9 / 8 + 64) + 8192 * 1024 * 8 / n + 8
    # the BF16 form: rounded rows, and one packing of half that size
    assert need(n, d, 15, rsc.RSC_BF16) / n < 2 * 64 * 8 + 64 + 32 + 2 * 4 * d + (2 * d * 9 / 8 + 64) + 8


@pytest.mark.gpu
@pytest.mark.parametrize("n,k", [(900, 15), (900, 200), (20000, 15), (20000, 80), (20000, 65)])
def test_either_kind_in_turn(oracle_mod, n, k):
    import numpy as np
    import torch

    import synth
    from tests.parity import compare_knn

    ws = rsc.Workspace("cuda")
    at = np.arange(0, n, n // 100)
    for spread in (1.0, 2.0 ** -20, 1.0):
        X = synth.mixture(n, d=50, n_clusters=6, seed=n + k)
        X[::3] *= np.float32(spread)
        idx, dist = rsc.knn(torch.from_numpy(X).cuda(), k, workspace=ws)
        io, _, do = oracle_mod.knn_rows(X, at, k)
        res = compare_knn(X, at, idx.cpu().numpy()[at], dist.cpu().numpy()[at], io, do, oracle_mod, k)
        assert res["exact_rows"] + res["near_tie_rows"] == at.size


@pytest.mark.gpu
def test_batched_flagged_rows(oracle_mod):
    """Samples with an offset flag rows, whose second search packs for the FP32 chain."""
    import numpy as np
    import torch

    from tests.parity import compare_knn

    sizes = [700, 3000, 1500]
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = np.random.default_rng(1).standard_normal((int(off[-1]), 50)).astype(np.float32)
    X[off[1]:off[2]] += np.float32(150)
    ws = rsc.Workspace("cuda")
    for _ in range(2):
        idx, dist = rsc.knn_batched(torch.from_numpy(X).cuda(), off, 15, workspace=ws)
        assert rsc.read_knn_stats(ws)["escalated_rows"] > 100
        idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
        for s in range(len(sizes)):
            Xs = X[off[s]:off[s + 1]]
            rows = np.arange(0, sizes[s], 7)
            io, _, do = oracle_mod.knn_rows(Xs, rows, 15)
            res = compare_knn(Xs, rows, idx[off[s]:off[s + 1]][rows] - off[s], dist[off[s]:off[s + 1]][rows], io, do,
                              oracle_mod, 15)
            assert res["exact_rows"] + res["near_tie_rows"] == rows.size
