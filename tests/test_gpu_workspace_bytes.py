"""A workspace of exactly the queried size serves the square and the rectangular call, at the sizes where plans change."""

import ctypes

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [500, 16383, 16384, 17000, 20000, 20479, 20480, 21761, 32769, 43521, 66000, 131073])
@pytest.mark.parametrize("precision", [rsc.RSC_FP32, rsc.RSC_BF16])
def test_square_and_rectangular(n, precision):
    lib, d = rsc.load(), 20
    X = torch.randn((n, d), generator=torch.Generator("cuda").manual_seed(n), device="cuda")
    o = rsc._opts(precision)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    for k in (1, 15, 33, 34, 63) + ((64, 65, 66, 67, 129, 255) if precision == rsc.RSC_FP32 else ()):
        need = lib.rsc_knn_workspace_bytes(n, n, d, k, ctypes.byref(o))
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        idx, dist = torch.empty((n, k), dtype=torch.int32, device="cuda"), torch.empty((n, k), device="cuda")
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert lib.rsc_knn_opt(ptr(X), n, d, k, ctypes.byref(o), ptr(idx), ptr(dist), ptr(ws), need, stream) == 0, (k, need)
        assert lib.rsc_knn_ex(ptr(X), n, ptr(X), n, d, k, ctypes.byref(o), ptr(idx), ptr(dist), ptr(ws), need, stream) == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,listed", [(300000, 900), (300000, 20000), (20000, 15000)])
def test_listed_rows(n, listed):
    """The exact rows of a probed search, few of many: the answers are the exact search's."""
    import numpy as np

    gen = torch.Generator().manual_seed(n)
    X = torch.randn((n, 20), generator=gen).cuda()
    label = torch.randint(0, 64, (n,), generator=gen).numpy()
    perm = np.argsort(label, kind="stable").astype(np.int32)
    off = np.concatenate([[0], np.cumsum(np.bincount(label, minlength=64))]).astype(np.int64)
    probes = np.stack([label, (label + 1) % 64], 1).astype(np.int32)
    mark = torch.zeros((n,), dtype=torch.uint8)
    mark[torch.randperm(n, generator=gen)[:listed]] = 1
    idx, dist, route, _ = rsc.knn_probed(X, 15, *[torch.from_numpy(a).cuda() for a in (off, perm, probes)],
                                         exact_rows=mark.cuda())
    want, wdist = rsc.knn(X, 15)
    rows = route != 0
    assert int(rows.sum()) >= listed
    assert torch.equal(idx[rows], want[rows]) and torch.equal(dist[rows], wdist[rows])
