"""Prefix sums at the sizes where their launches change (one tile of 2048
items, one tile more, the last size whose tile sums each block adds up
itself, and beyond), and pruning levels whose label lists cross the sort's
tiers. Exact equality."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import pins
from gpu_util import assert_same_labels, gpu_labels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [1, 7, 2047, 2048, 2049, 4096, 300 * 2048 + 5, 512 * 2048, 512 * 2048 + 1,
                               513 * 2048 + 1])
def test_path_offsets(q):
    """The offsets of q paths are the exclusive sums of their lengths."""
    import torch
    from paper_1907_00140_amd import chl
    print("path offsets", q, flush=True)
    n, u, v, w = gg.grid_edges(8, 8, 1, 4, 5)
    row, col, ww = pins.csr_from_edges(n, list(zip(u.tolist(), v.tolist(), w.tolist())))
    L = chl.build(row, col, ww, gg.random_rank(n, 3), autotune=False)
    par, slot = L.parents(row, col, ww)
    pairs = torch.from_numpy(np.random.default_rng(q).integers(0, n, (q, 2)).astype(np.int32))
    hops, off = L.path_hops(pairs, par, slot)
    hops, off = hops.cpu().numpy(), off.cpu().numpy()
    assert hops.min() >= 0                       # connected
    assert off[0] == 0 and np.array_equal(off[1:], np.cumsum(hops + 1))
    L.free()


@pytest.mark.parametrize("hubs", [16, 255, 256, 257, 600])
def test_level_list_lengths(hubs):
    """A row of vertices under a ranking by position: every vertex keeps a
    label of every outranking hub nearer the end, so the levels' lists are as
    long as there are hubs."""
    print("level lists", hubs, flush=True)
    n = 1300
    e = [(i, i + 1, 1 + i % 5) for i in range(n - 1)]
    row, col, w = pins.csr_from_edges(n, e)
    for order in (np.arange(n, dtype=np.int32), gg.random_rank(n, 2)):
        ref = oracle.chl(row, col, w, order)
        L, off, hub, dist = gpu_labels(row, col, w, order, autotune=False, prune_hubs=hubs)
        assert_same_labels(off, hub, dist, ref, str(hubs))
        L.free()
