"""Community sums gathered per block: few and many communities per table slot.

Each graph is a set of disjoint cliques, so the number of communities is known:
one, as many as the block's table has slots, one more, and far more (where most
sums go to memory directly); the clique sizes reach rows on both sides of the
lanes that share a row, of the entries that a wave takes at once (256) and of the
rows that it takes.  Vertices without edges lie between them.  Labels and
modularity equal the oracle's.
"""

import numpy as np
import pytest
import torch

import paper_2603_02402_amd as rsc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,size", [(1, 40), (2, 17), (127, 5), (128, 16), (129, 9), (700, 3), (3000, 2), (40, 70),
                                        (5, 256), (3, 257), (2, 258), (300, 17)])
def test_cliques_match_the_oracle(count, size):
    from oracle import leiden as ol

    rng = np.random.default_rng(count)
    n = count * size + count // 2
    place = rng.permutation(n)  # a clique's vertices lie anywhere in the order
    w = rng.uniform(0.5, 1.0, (count, size, size)).astype(np.float32)
    w = np.maximum(w, w.transpose(0, 2, 1))
    rows, cols, vals = [], [], []
    for c in range(count):
        ids = place[c * size:(c + 1) * size]
        i, j = np.nonzero(~np.eye(size, dtype=bool))
        rows.append(ids[i])
        cols.append(ids[j])
        vals.append(w[c][i, j])
    rows, cols, vals = map(np.concatenate, (rows, cols, vals))
    order = np.lexsort((cols, rows))
    rows, cols, vals = rows[order], cols[order], vals[order]
    indptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    indices = cols.astype(np.int32)

    want, quality, levels = ol.leiden(indptr, indices, vals, 1.0)
    graph = tuple(torch.from_numpy(a).cuda() for a in (indptr, indices, vals))
    labels, st = rsc.leiden(graph, gamma=1.0)
    assert np.array_equal(labels.cpu().numpy(), want)
    assert st["quality"] == quality
    assert st["levels"] == levels
    assert st["n_communities"] == want.max() + 1
