"""Top probes of the router: the gathered and sorted columns, and the rows that
take the winner-by-winner path (every logit equal: all columns tie at the bound).

The partitions are the first `probes` of a stable descending sort of the logits
the same network returns; their mass is the float32 softmax sum, within its
rounding (probes + 8 units of 2^-24 of a sum below one, and the exponential's).
"""

import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts,probes", [(64, 1), (64, 64), (128, 64), (192, 63), (1024, 32), (4096, 1), (4096, 32),
                                          (4096, 64)])
@pytest.mark.parametrize("n,tied", [(1, False), (130, False), (515, True)])
def test_probes_are_the_largest_logits(parts, probes, n, tied):
    router = rsc.Router(17, 64, parts, seed=parts + probes)
    gen = torch.Generator("cuda").manual_seed(n)
    X = torch.randn((n, 17), generator=gen, device="cuda")
    if tied:
        X[::3] = 0.0  # no biases yet: every logit of these rows is zero
    z = router.logits(X)
    want = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :probes]
    got, mass = router.probe(X, probes)
    assert torch.equal(got.long(), want)
    share = torch.softmax(z.double(), 1).gather(1, want).sum(1)
    assert float((mass.double() - share).abs().max()) <= (probes + 8) * 2.0**-23
