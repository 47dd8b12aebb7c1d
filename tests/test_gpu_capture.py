"""The exact search recorded into a graph: every replay equals the eager call.

20,000 rows take the pruned screen when called eagerly and the unpruned one when
recorded; 3,000 rows the unpruned one both times.  Replays are mixed with the
program's own work and synchronisations, and read new inputs.
"""

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3000, 20000])
@pytest.mark.parametrize("metric", ["euclidean", "cosine"])
def test_replays_equal_the_eager_call(n, metric):
    m = rsc.RSC_COSINE if metric == "cosine" else rsc.RSC_EUCLIDEAN
    gen = torch.Generator("cuda").manual_seed(n)
    centres = torch.randn((20, 50), generator=gen, device="cuda") * 5

    def rows():
        at = torch.randint(0, 20, (n,), generator=gen, device="cuda")
        return centres[at] + torch.randn((n, 50), generator=gen, device="cuda")

    X = rows()
    ws = rsc.Workspace("cuda")
    out = (torch.empty((n, 15), dtype=torch.int32, device="cuda"),
           torch.empty((n, 15), dtype=torch.float32, device="cuda"))
    rsc.knn(X, 15, metric=m, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rsc.knn(X, 15, metric=m, out=out, workspace=ws)
    for _ in range(4):
        X.copy_(rows())
        out[0].fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        idx, dist = rsc.knn(X, 15, metric=m)
        assert torch.equal(out[0], idx)
        assert torch.equal(out[1], dist)
