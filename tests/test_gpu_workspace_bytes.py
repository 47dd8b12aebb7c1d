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
