"""The probed search's workspace: its bound for the exact fallback, whatever rows go there."""

import numpy as np
import pytest

import paper_2603_02402_amd as rsc


def test_small_problem_stays_small():
    """3000 rows: up to 131072 rows of 32 candidates (8 bytes) for the fallback's ranges, 1024 candidates for each row
    searched again, and the packings and lists of the rows themselves (below 2 KiB a row)."""
    need = rsc.load().rsc_knn_probed_workspace_bytes(3000, 50, 15, 512, 48)
    assert need < (131072 + 3000) * 32 * 8 + 3000 * 1024 * 8 + 3000 * 2048 + 512 * 32 * 2048 + (1 << 20)


# rows that all go to the exact search, and a part of them, around the sizes where its ranges change
@pytest.mark.gpu
@pytest.mark.parametrize("n,k", [(2000, 15), (16384, 15), (16500, 40), (40000, 63), (66000, 16), (132000, 40), (140000, 63)])
def test_fallback_fits(n, k):
    import torch

    gen = torch.Generator().manual_seed(n)
    centres = 4 * torch.randn((20, 20), generator=gen)
    at = torch.randint(0, 20, (n,), generator=gen)
    X = (centres[at] + torch.randn((n, 20), generator=gen)).cuda()
    parts = 64
    label = torch.randint(0, parts, (n,), generator=gen).numpy()
    perm = np.argsort(label, kind="stable").astype(np.int32)
    off = np.concatenate([[0], np.cumsum(np.bincount(label, minlength=parts))]).astype(np.int64)
    probes = np.stack([label, (label + 1) % parts, (label + 2) % parts, (label + 3) % parts], 1).astype(np.int32)
    dev = [torch.from_numpy(a).cuda() for a in (off, perm, probes)]
    want, wdist = rsc.knn(X, k)
    for share in (1.0, 0.5, 0.1):
        exact = torch.rand((n,), generator=gen) < share
        idx, dist, route, _ = rsc.knn_probed(X, k, *dev, exact_rows=exact.to(torch.uint8).cuda())
        rows = route != 0
        assert int(rows.sum()) >= int(exact.sum())
        assert torch.equal(idx[rows], want[rows])
        assert torch.equal(dist[rows], wdist[rows])
