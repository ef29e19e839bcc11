"""Rows of the graph given to the parents call: malformed ones of every kind
are flagged whatever their claimed length, on graphs of fewer and of more arcs
than make a row a heavy one; heavy vertices with more labels than one pass
holds match the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import pins

pytestmark = pytest.mark.gpu


def _bad_rows(row, m):
    """(what, row offsets) with one malformed row each, first, inner or last."""
    n = len(row) - 1
    for at in (1, n // 2, n):
        for beyond in (1, 255, 256, 257, 1000, 1 << 40):
            r = row.copy()
            r[at] = m + beyond
            yield "row %d ends %d beyond the arcs" % (at - 1, beyond), r
        r = row.copy()
        r[at] = -1 - m
        yield "row %d ends below 0" % (at - 1), r
    r = row.copy()
    r[0] = -1000
    yield "row 0 starts below 0", r


@pytest.mark.parametrize("leaves", [5, 127, 128, 129, 400])
def test_malformed_rows_are_flagged(leaves):
    from paper_1907_00140_amd import chl
    row, col, w = pins.csr_from_edges(leaves + 1, [(0, 1 + i, 1 + i % 3) for i in range(leaves)])
    L = chl.build(row, col, w, gg.degree_rank(row, 1), autotune=False)
    L.parents(row, col, w)                            # well-formed: accepted
    for what, r in _bad_rows(np.asarray(row, np.int64), len(col)):
        print("malformed rows", leaves, what, flush=True)
        with pytest.raises(chl.ChlError) as e:
            L.parents(r, col, w)
        assert e.value.code == -1, what
    L.free()


@pytest.mark.parametrize("clique", [258, 300, 600])
def test_heavy_vertices_of_many_labels(clique):
    """A clique: its vertices are heavy and hold up to `clique` labels."""
    from paper_1907_00140_amd import chl
    print("clique", clique, flush=True)
    g = np.random.default_rng(clique)
    e = [(i, j, int(g.integers(1000, 2000))) for i in range(clique) for j in range(i)]
    row, col, w = pins.csr_from_edges(clique, e)
    order = g.permutation(clique).astype(np.int32)
    L = chl.build(row, col, w, order, autotune=False)
    par, slot = L.parents(row, col, w)
    rpar, rslot = oracle.parents(oracle.chl(row, col, w, order), row, col, w)
    assert np.array_equal(par.cpu().numpy(), rpar) and np.array_equal(slot.cpu().numpy(), rslot)
    L.free()
