"""Frontier expansion at the sizes where it changes path: near lists of one
vertex, around a wave, around the workgroup (the part of a list held in LDS
and the rest), arcs and candidates around multiples of the batch; far lists
that empty a bucket. Bit-exact against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import pins
from gpu_util import assert_same_labels, gpu_labels

pytestmark = pytest.mark.gpu


def _fan(width, tail, seed):
    """Hub - `width` middle vertices - `width` ends - a second hub, equal and
    unequal weights mixed (ties, in-round improvements), and a weighted path
    of `tail` vertices behind it (sparse buckets)."""
    g = np.random.default_rng(seed)
    n = 2 + 2 * width + tail
    e = []
    for i in range(width):
        e.append((0, 2 + i, int(g.integers(1, 3))))
        e.append((2 + i, 2 + width + i, int(g.integers(1, 4))))
        e.append((2 + i, 2 + width + (i + 1) % width, int(g.integers(1, 4))))
        e.append((2 + width + i, 1, int(g.integers(1, 3))))
    last = 1
    for i in range(tail):
        e.append((last, 2 + 2 * width + i, int(g.integers(1, 200))))
        last = 2 + 2 * width + i
    return n, e


@pytest.mark.parametrize("wg", [64, 128, 256, 512, 1024])
@pytest.mark.parametrize("width", [1, 31, 63, 64, 65, 255, 256, 257, 1023, 1025])
def test_near_list_sizes(wg, width):
    print("near list", wg, width, flush=True)
    n, e = _fan(width, 20, width)
    row, col, w = pins.csr_from_edges(n, e)
    order = gg.degree_rank(row, 1) if width % 2 else gg.random_rank(n, width)
    ref = oracle.chl(row, col, w, order)
    for kw in (dict(delta=1, prune_hubs=-1), dict(delta=1000, prune_hubs=-1, early_term=False),
               dict(delta=3, prune_hubs=min(16, n // 2), team_wgs=1)):
        L, off, hub, dist = gpu_labels(row, col, w, order, wg_size=wg, roots_in_flight=7, autotune=False, **kw)
        assert_same_labels(off, hub, dist, ref, str((wg, width, kw)))
        L.free()


@pytest.mark.parametrize("rows,cols", [(1, 2047), (2, 1024), (45, 46), (53, 61), (128, 17)])
@pytest.mark.parametrize("directed", [False, True])
def test_input_numbering(rows, cols, directed):
    """Unpruned trees of a graph stored row by row grow in input numbering
    (from 2048 vertices on, half the arcs within 4 sqrt(n) ids); the same
    graph with scrambled ids grows by rank position. Complete builds and root
    subsets, in both forms, against the oracle."""
    print("input numbering", rows, cols, directed, flush=True)
    n, u, v, w = gg.grid_edges(rows, cols, 1, 4, 5, diag_prob=0.3)
    g = np.random.default_rng(rows)
    for ids in (np.arange(n), g.permutation(n)):
        e = list(zip(ids[u].tolist(), ids[v].tolist(), w.tolist()))
        row, col, ww = pins.csr_from_edges(n, e)
        order = gg.random_rank(n, 3)
        if directed:
            refs = oracle.chl_directed(row, col, ww, order)
        else:
            refs = [oracle.chl(row, col, ww, order)]
        for kw in (dict(delta=1), dict(delta=7, wg_size=64, roots_in_flight=300), dict(early_term=False, delta=50)):
            L, off, hub, dist = gpu_labels(row, col, ww, order, autotune=False, prune_hubs=-1, directed=directed, **kw)
            assert_same_labels(off, hub, dist, refs[0], str((rows, cols, kw)))
            if directed:
                off, hub, dist = (x.numpy() for x in L.export_in("cpu"))
                assert_same_labels(off, hub, dist, refs[1], str((rows, cols, kw)))
            L.free()
        if not directed:
            roots = (5, 40, n // 41)
            L, off, hub, dist = gpu_labels(row, col, ww, order, autotune=False, prune_hubs=-1, roots=roots)
            want = np.isin(refs[0].hub_pos, roots[0] + roots[2] * np.arange(roots[1]))
            assert np.array_equal(hub, refs[0].hub_pos[want])
            assert np.array_equal(dist.astype(np.int64), refs[0].dist[want])
            L.free()


@pytest.mark.parametrize("hubs", [1, 2, 3, 4, 5, 6, 12, 13, 100])
@pytest.mark.parametrize("wmax", [2, 1 << 22])
def test_prefix_label_counts(hubs, wmax):
    """Pruning with prefixes whose per-vertex label lists end before, at and
    just behind the labels tested first and the batches read after them, with
    32- and 64-bit keys, in the batched, team, group and small-tree kernels."""
    print("prefix labels", hubs, wmax, flush=True)
    n, u, v, w = gg.random_edges(700, 1500, 1, wmax, hubs)
    row, col, ww = gg.to_csr(n, u, v, w)
    order = gg.random_rank(n, hubs)
    ref = oracle.chl(row, col, ww, order)
    for kw in (dict(team_wgs=1, wg_size=64), dict(team_wgs=3), dict(), dict(groups=False, small=True)):
        L, off, hub, dist = gpu_labels(row, col, ww, order, autotune=False, prune_hubs=hubs, delta=1 + wmax // 2, **kw)
        assert_same_labels(off, hub, dist, ref, str((hubs, wmax, kw)))
        L.free()
