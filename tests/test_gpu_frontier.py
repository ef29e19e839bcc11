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
