"""Shortest paths from the labeling on the GPU (chl_labels_parents,
chl_query_path_hops, chl_query_paths) against the oracle, bit for bit.

The parent of a label is unique (the smallest-id shortest-path neighbour
towards its hub), and so is the path of a pair (through the most important
hub among those giving d(u, v)), so every comparison is an exact equality.
"""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle
import pins

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a device"
    from paper_1907_00140_amd import chl
    chl.load()


def _gpu(row, col, w, order, pairs, **kw):
    from paper_1907_00140_amd import chl
    L = chl.build(row, col, w, order, **kw)
    par, slot = L.parents(row, col, w)
    hops, off, path = L.paths(pairs, par, slot)
    return L, par.cpu().numpy(), slot.cpu().numpy(), (hops.cpu().numpy(), off.cpu().numpy(), path.cpu().numpy())


def _same(got, ref, where):
    (par, slot, (hops, off, path)), (rpar, rslot, (rhops, roff, rpath)) = got, ref
    assert np.array_equal(par, rpar), where + ": parents differ"
    assert np.array_equal(slot, rslot), where + ": slots differ"
    assert np.array_equal(hops, rhops), where + ": hop counts differ"
    assert np.array_equal(off, roff), where + ": path offsets differ"
    assert np.array_equal(path, rpath), where + ": path vertices differ"


def _all_pairs(n):
    uu, vv = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    return np.stack([uu.ravel(), vv.ravel()], 1).astype(np.int32)


def _check(row, col, w, order, pairs, where, **kw):
    ref_lab = oracle.chl(row, col, w, order)
    rpar, rslot = oracle.parents(ref_lab, row, col, w)
    ref = (rpar, rslot, oracle.paths(ref_lab, rpar, rslot, pairs))
    L, par, slot, paths = _gpu(row, col, w, order, pairs, **kw)
    _same((par, slot, paths), ref, where)
    return L, ref_lab, par, slot, paths


@pytest.mark.parametrize("name", ["fig1_example.txt", "reading1_counterexample.txt"])
def test_golden_paths(name):
    _say("golden paths", name)
    n, order, edges, _ = pins.load_golden(name)
    row, col, w = pins.csr_from_edges(n, edges)
    _check(row, col, w, order, _all_pairs(n), name, delta=1, autotune=False)


@pytest.mark.parametrize("seed", range(12))
def test_random_small_paths(seed):
    """Random multigraphs (parallel arcs, self-loops, several components) with
    few distinct weights, all pairs; the paths also pass the Floyd-Warshall
    checks of the oracle's pins."""
    g = np.random.default_rng(1000 + seed)
    n = int(g.integers(2, 90))
    m = int(g.integers(n // 2, 3 * n))
    wmax = int(g.integers(1, 5))
    e = [(int(a), int(b), int(c)) for a, b, c in
         zip(g.integers(0, n, m), g.integers(0, n, m), g.integers(1, wmax + 1, m))]
    row, col, w = pins.csr_from_edges(n, e)
    order = gg.random_rank(n, seed) if seed % 2 else gg.degree_rank(row, seed)
    _say("random_small_paths", seed, n, m, wmax)
    _, lab, par, slot, paths = _check(row, col, w, order, _all_pairs(n), "seed %d" % seed,
                                      delta=1 + seed % 3, autotune=False)
    D = pins.floyd_warshall(n, row, col, w)
    pins.check_parent_labels(lab, par, slot, D, row, col, w, order)
    pins.check_path_walks(paths, D, row, col, w, order)


@pytest.mark.parametrize("name", ["grid64", "rmat12s9"])
def test_config_paths(name):
    c = gg.make_config(name)
    _say("config paths", name)
    pairs = c["pairs"][:20000]
    _check(c["row_ptr"], c["col"], c["w"], c["order"], pairs, name)


def test_rmat16_paths():
    """The benchmark's graph: every label's parent, 2*10^4 paths."""
    c = gg.make_config("rmat16")
    _say("rmat16 paths")
    _check(c["row_ptr"], c["col"], c["w"], c["order"], c["pairs"][:20000], "rmat16")


def test_grid1024d_sampled_paths():
    """Full-size road-like grid (1.28e9 labels): sampled labels' parents
    against Dijkstra from their hub, sampled paths as walks of the queried
    length that follow the parent rule towards their most important vertex."""
    import torch
    from paper_1907_00140_amd import chl
    c = gg.make_config("grid1024d")
    row, col, w, order = c["row_ptr"], c["col"], c["w"], c["order"]
    n = len(row) - 1
    _say("grid1024d build")
    L = chl.build(row, col, w, order)
    _say("grid1024d parents")
    par_d, slot_d = L.parents(row, col, w)
    off = L.offsets()
    pos = pins.pos_of(order)
    rng = np.random.default_rng(7)
    _, hub_d, _ = L.export("cuda")
    for hp in (0, 3, 1000, 200000, 900000):
        h = int(order[hp])
        dh = oracle.sssp(row, col, w, h)
        vs = rng.integers(0, n, 1500)
        # the label of hub hp in each sampled L_v
        for v in vs.tolist():
            a, b = int(off[v]), int(off[v + 1])
            hs = hub_d[a:b].cpu().numpy()
            i = np.searchsorted(hs, hp)
            if i == len(hs) or hs[i] != hp:
                continue
            p = int(par_d[a + i].item())
            nb = [(int(col[e]), int(w[e])) for e in range(row[v], row[v + 1])]
            want = min((x for x, y in nb if dh[x] + y == dh[v]), default=-1)
            assert p == want, (hp, v, p, want)
    del hub_d
    _say("grid1024d paths")
    pairs = c["pairs"][:200]
    hops, poff, path = L.paths(pairs, par_d, slot_d)
    hops, poff, path = hops.cpu().numpy(), poff.cpu().numpy(), path.cpu().numpy()
    d = L.query(torch.from_numpy(pairs).cuda()).cpu().numpy()
    for k, (u, v) in enumerate(pairs.tolist()):
        P = path[poff[k]:poff[k + 1]].tolist()
        assert P[0] == u and P[-1] == v and len(P) == hops[k] + 1
        s = 0
        for a, b in zip(P[:-1], P[1:]):
            seg = range(row[a], row[a + 1])
            s += min(int(w[e]) for e in seg if col[e] == b)
        assert s == d[k], (u, v, s, d[k])
    for k in range(5):
        u, v = pairs[k].tolist()
        P = path[poff[k]:poff[k + 1]].tolist()
        hm = min(P, key=lambda x: pos[x])
        dh = oracle.sssp(row, col, w, hm)
        a = P.index(hm)
        for half in (P[:a + 1], P[a:][::-1]):
            for x, y in zip(half[:-1], half[1:]):
                nb = [(int(col[e]), int(w[e])) for e in range(row[x], row[x + 1])]
                assert y == min(p for p, z in nb if dh[p] + z == dh[x])


def test_path_edge_cases():
    import torch
    from paper_1907_00140_amd import chl
    # two components plus an isolated vertex; a self-loop and a parallel arc
    edges = [(0, 1, 2), (1, 2, 2), (0, 2, 5), (0, 2, 4), (3, 4, 1), (4, 4, 3)]
    n = 6
    row, col, w = pins.csr_from_edges(n, edges)
    order = np.array([2, 0, 4, 1, 3, 5], np.int32)
    pairs = np.array([[0, 2], [2, 0], [0, 0], [5, 5], [0, 3], [3, 4], [1, 5]], np.int32)
    L, lab, par, slot, (hops, off, path) = _check(row, col, w, order, pairs, "edge cases", autotune=False)
    assert hops.tolist() == [2, 2, 0, 0, -1, 1, -1]
    assert path[off[0]:off[1]].tolist() == [0, 1, 2] and path[off[2]:off[3]].tolist() == [0]
    par_d, slot_d = L.parents(row, col, w)
    # q = 0
    h0, o0, p0 = L.paths(np.zeros((0, 2), np.int32), par_d, slot_d)
    assert h0.numel() == 0 and o0.cpu().tolist() == [0] and p0.numel() == 0
    # an id out of range
    with pytest.raises(chl.ChlError):
        L.path_hops(np.array([[0, 6]], np.int32), par_d, slot_d)
    # a graph of another size, and a weight below 1
    r2, c2, w2 = pins.csr_from_edges(n + 1, edges)
    with pytest.raises(chl.ChlError):
        L.parents(r2, c2, w2)
    w0 = w.copy()
    w0[0] = 0
    with pytest.raises(chl.ChlError):
        L.parents(row, col, w0)
    # parent arrays that do not fit the labeling
    bad = slot_d.clone()
    bad[bad >= 0] += 1000
    with pytest.raises(chl.ChlError):
        L.path_hops(pairs, par_d, bad)
    # path offsets that do not match the hop counts: error, nothing written
    # outside the pairs' ranges
    p = torch.from_numpy(pairs[:2]).cuda()
    _, o = L.path_hops(p, par_d, slot_d)
    o2 = o.clone()
    o2[2] -= 1
    buf = torch.full((int(o[2].item()) + 4,), -7, dtype=torch.int32, device="cuda")
    lib = chl.load()
    import ctypes as C
    rc = lib.chl_query_paths(L.handle, par_d.data_ptr(), slot_d.data_ptr(), p.data_ptr(), 2, o2.data_ptr(),
                             buf.data_ptr(), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == -1
    assert (buf[int(o2[2].item()):].cpu() == -7).all()


def test_paths_after_pruned_and_team_builds():
    """Parents depend only on the labels: builds with other schedules give
    the same arrays."""
    c = gg.make_config("rmat12s9")
    row, col, w, order = c["row_ptr"], c["col"], c["w"], c["order"]
    pairs = c["pairs"][:5000]
    ref = None
    for kw in (dict(), dict(prune_hubs=-1), dict(prune_hubs=64, team_wgs=4), dict(mode="batched", wg_size=64)):
        _, par, slot, paths = _gpu(row, col, w, order, pairs, **kw)
        if ref is None:
            ref = (par, slot, paths)
        else:
            _same((par, slot, paths), ref, str(kw))


@pytest.mark.parametrize("leaves", [255, 256, 257, 1025, 3000])
def test_parents_heavy_vertices(leaves):
    """Vertices around and far beyond the arc count from which several waves
    share a vertex, important and unimportant ones, with ties."""
    print("heavy vertices", leaves, flush=True)
    g = np.random.default_rng(leaves)
    e = [(0, 3 + i, int(g.integers(1, 4))) for i in range(leaves)]
    e += [(1, 3 + i, int(g.integers(1, 4))) for i in range(0, leaves, 2)]
    e += [(2, 3 + i, int(g.integers(1, 4))) for i in range(0, leaves, 3)]
    row, col, w = pins.csr_from_edges(leaves + 3, e)
    for order in (gg.degree_rank(row, 1), gg.random_rank(leaves + 3, 2)):
        from paper_1907_00140_amd import chl
        L = chl.build(row, col, w, order, autotune=False)
        ref = oracle.chl(row, col, w, order)
        par, slot = L.parents(row, col, w)
        rpar, rslot = oracle.parents(ref, row, col, w)
        assert np.array_equal(par.cpu().numpy(), rpar) and np.array_equal(slot.cpu().numpy(), rslot)
        L.free()
