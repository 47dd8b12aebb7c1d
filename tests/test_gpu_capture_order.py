"""Recorded reduced-precision searches: kernels alone, and replays equal the eager call.

The rows' order comes from a library sort that clears counters by memset above
2^20 rows; memset nodes have given wrong results on replays, so a recorded call
sorts in pieces.
"""

import ctypes

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu

KERNEL = 0  # hipGraphNodeTypeKernel


def node_types(call):
    """Types of the nodes that `call` records on a stream."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    graph, count, stream = ctypes.c_void_p(), ctypes.c_size_t(0), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        handle = ctypes.c_void_p(stream.cuda_stream)
        assert hip.hipStreamBeginCapture(handle, 2) == 0
        try:
            call()
        finally:
            assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    types = set()
    for node in nodes:
        t = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(t)) == 0
        types.add(t.value)
    assert hip.hipGraphDestroy(graph) == 0
    return types


def rows(n, d, gen, centres):
    """Rows that BF16 holds exactly: the BF16 answer then does not depend on the order."""
    at = torch.randint(0, centres.shape[0], (n,), generator=gen, device="cuda")
    return (centres[at] + torch.randn((n, d), generator=gen, device="cuda")).bfloat16().float()


def buffers(n, k):
    return (torch.empty((n, k), dtype=torch.int32, device="cuda"),
            torch.empty((n, k), dtype=torch.float32, device="cuda"))


# (queries, references): one side or both above 2^20 rows, and a square problem
@pytest.mark.parametrize("precision", [rsc.RSC_BF16, rsc.RSC_FP8_E4M3])
@pytest.mark.parametrize("nq,n", [(2 ** 20 + 1, 300), (1000, 2 ** 20 + 1), (2 ** 20 + 33, 2 ** 20 + 7), (0, 2 ** 20 + 1)])
def test_records_kernels_alone(precision, nq, n):
    X = torch.randn((n, 4), device="cuda")
    Q = torch.randn((nq, 4), device="cuda") if nq else None
    ws, out = rsc.Workspace("cuda"), buffers(nq or n, 5)
    o = rsc.KnnOpts(precision, 0, 0, 0)
    ws.get(rsc.load().rsc_knn_workspace_bytes(nq or n, n, 4, 5, ctypes.byref(o)))
    torch.cuda.synchronize()
    assert node_types(lambda: rsc.knn(X, 5, Q=Q, precision=precision, out=out, workspace=ws)) == {KERNEL}


@pytest.mark.parametrize("precision", [rsc.RSC_BF16, rsc.RSC_FP8_E4M3])
@pytest.mark.parametrize("n,nq", [(3000, 0), (20000, 0), (60000, 5003), (2 ** 20 + 1000, 0), (2 ** 20 + 1000, 5003)])
def test_replays_equal_the_eager_call(n, nq, precision):
    if n > 2 ** 20 and precision == rsc.RSC_FP8_E4M3:
        pytest.skip("FP8 answers depend on the order, which differs above 2^20 rows")
    gen = torch.Generator("cuda").manual_seed(n + nq)
    centres = torch.randn((100, 50), generator=gen, device="cuda") * 5
    X = rows(n, 50, gen, centres)
    Q = rows(nq, 50, gen, centres) if nq else None
    ws, out = rsc.Workspace("cuda"), buffers(nq or n, 15)
    rsc.knn(X, 15, Q=Q, precision=precision, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rsc.knn(X, 15, Q=Q, precision=precision, out=out, workspace=ws)
    for _ in range(4):
        X.copy_(rows(n, 50, gen, centres))
        out[0].fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        idx, dist = rsc.knn(X, 15, Q=Q, precision=precision)
        assert torch.equal(out[0], idx)
        assert torch.equal(out[1], dist)
