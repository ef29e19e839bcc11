"""Long lists with one wave per query: every wave takes many queries one
after the other through the same hash table, lists of all lengths in turn, so
that an entry of one query met by the next would give a wrong distance."""
import numpy as np
import pytest

import pins
from gpu_util import gpu_labels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clique", [240, 300, 700])
@pytest.mark.parametrize("q", [16385, 300007, 1000003])
def test_queries_one_after_the_other(clique, q):
    """A clique: the list of the vertex at rank position r holds r + 1 hubs,
    and a pair's distance is the weight of its edge."""
    print("queries in turn", clique, q, flush=True)
    g = np.random.default_rng(clique)
    w = np.triu(g.integers(1000, 2000, (clique, clique)), 1)
    w = w + w.T
    e = [(i, j, int(w[i, j])) for i in range(clique) for j in range(i)]
    row, col, ww = pins.csr_from_edges(clique, e)
    order = g.permutation(clique).astype(np.int32)
    L, _, _, _ = gpu_labels(row, col, ww, order, autotune=False, prune_hubs=-1)
    # long and short lists in turn
    by_len = order                       # rank order: lists of 1, 2, 3, ... hubs
    k = np.arange(q) // 7 % 2
    pairs = np.stack([np.where(k == 1, by_len[g.integers(clique // 2, clique, q)], by_len[g.integers(0, 20, q)]),
                      g.integers(0, clique, q)], 1).astype(np.int32)
    for _ in range(2):
        got = L.query(pairs).cpu().numpy()
        assert np.array_equal(got, w[pairs[:, 0], pairs[:, 1]])
    L.free()
