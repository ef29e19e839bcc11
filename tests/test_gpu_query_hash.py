"""Queries over long lists (hash table in LDS): lists around the table's
capacity and beyond it, a single entry against a long list, empty
intersections, batches on both sides of the small-batch rule."""
import numpy as np
import pytest

import pins
from gpu_util import gpu_labels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clique,lonely", [(300, 0), (700, 900), (700, 300), (1100, 100)])
def test_long_lists(clique, lonely):
    """A clique (every vertex holds a label of each vertex above it, so the
    lists have every length up to the clique's size) and isolated vertices."""
    g = np.random.default_rng(clique)
    w = g.integers(1000, 2000, (clique, clique))
    e = [(i, j, int(w[i, j])) for i in range(clique) for j in range(i)]
    n = clique + lonely
    row, col, ww = pins.csr_from_edges(n, e)
    order = g.permutation(n).astype(np.int32)
    L, off, hub, dist = gpu_labels(row, col, ww, order, autotune=False, prune_hubs=-1)
    assert off[n] == clique * (clique + 1) // 2 + lonely
    want = np.full((n, n), -1, np.int64)
    want[:clique, :clique] = np.where(np.arange(clique)[:, None] > np.arange(clique), w, w.T)
    np.fill_diagonal(want, 0)
    for q in (1, 7, 1000, 16384, 16385, 60001):
        print("long lists", clique, lonely, q, flush=True)
        pairs = g.integers(0, n, (q, 2)).astype(np.int32)
        got = L.query(pairs).cpu().numpy()
        assert np.array_equal(got, want[pairs[:, 0], pairs[:, 1]])
    L.free()
