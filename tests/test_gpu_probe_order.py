"""Probed search: partitions are taken from the queries' own around.

Probe lists are random: with and without the row's own partition, with repeats
and gaps (-1), over partition counts at the edges of the bitmap's words and with
empty partitions.  A certified row's neighbours are the nearest rows of its
probed partitions, by float64 distances, with -1 where there are fewer.
"""

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts", [1, 31, 32, 33, 64, 97, 300])
@pytest.mark.parametrize("d,probes,k", [(50, 1, 8), (17, 7, 15), (70, 40, 20)])
def test_neighbours_lie_in_the_probed_partitions(parts, d, probes, k):
    n = 3001
    probes = min(probes, parts)
    gen = torch.Generator("cuda").manual_seed(parts * 7 + d)
    centres = torch.randn((12, d), generator=gen, device="cuda") * 4
    X = centres[torch.randint(0, 12, (n,), generator=gen, device="cuda")]
    X = X + torch.randn((n, d), generator=gen, device="cuda")
    part = torch.randint(0, parts, (n,), generator=gen, device="cuda")
    if parts > 32:
        part[(part >= 5) & (part < 9)] = 4  # empty partitions
    perm = torch.argsort(part, stable=True).int()
    offsets = torch.zeros(parts + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.bincount(part, minlength=parts).cumsum(0)
    lists = torch.randint(0, parts, (n, probes), generator=gen, device="cuda", dtype=torch.int32)
    lists[::3, 0] = part[::3].int()
    if probes > 2:
        lists[1::5, 1] = -1
    idx, dist, route, _ = rsc.knn_probed(X, k, offsets, perm, lists)

    # the oracle on the host
    X, part, lists, idx, rows = X.cpu(), part.cpu(), lists.cpu().long(), idx.cpu().long(), route.cpu() == 0
    D = torch.cdist(X.double(), X.double(), compute_mode="donot_use_mm_for_euclid_dist")
    probed = torch.zeros((n, parts + 1), dtype=torch.bool)  # (the last column takes the gaps)
    probed[torch.arange(n)[:, None], torch.where(lists < 0, parts, lists)] = True
    D.masked_fill_(~probed[:, part], float("inf"))
    D.fill_diagonal_(-1.0)  # the row itself comes first
    best = torch.sort(D, dim=1).values[:, :k]
    got = torch.where(idx < 0, float("inf"), torch.gather(D, 1, idx.clamp_min(0)))
    assert torch.equal(idx[:, 0], torch.arange(n))
    assert torch.equal(got[rows].isinf(), best[rows].isinf())  # fewer rows probed than asked for
    assert float((got[rows] - best[rows]).nan_to_num(0.0).abs().max()) <= 1e-9
