"""What a user of this library has it do, as timed cases: complete builds of
the canonical labeling (scale-free, road-like and directed graphs, from the
size of a serving request to a million vertices; the Hybrid construction),
distance queries from one pair to a million, shortest paths, and the
continuous-batching server under a full queue.

Graphs are drawn on the device from the seed: R-MAT graphs (quadrants
0.57, 0.19, 0.19, 0.05; 8 samples per vertex; vertices beyond n dropped, so
that n need not be a power of two) and 4-neighbour grids (5% diagonal
shortcuts from 128 rows on), integer weights uniform in [1, wmax], ranked by
degree with random ties (as scale-free graphs are in the paper), or at random
for the Hybrid.
"""
import math

import numpy as np
import torch

from paper_1907_00140_amd import chl, serve

DEV = "cuda"
RMAT_A, RMAT_AB, RMAT_ABC = 0.57, 0.76, 0.95


def listed():
    return [
        # a build request of the serving workload: launches and latency
        {"name": "build-rmat10", "kind": "build", "graph": "rmat", "n": 1024, "wmax": 1000},
        # the small grid of the tests and the benchmark
        {"name": "build-grid64", "kind": "build", "graph": "grid", "rows": 64, "cols": 64, "wmax": 100},
        # a scale-free graph of 65,536 vertices, the benchmark's middle size
        {"name": "build-rmat16", "kind": "build", "graph": "rmat", "n": 65536, "wmax": 1000},
        # the benchmark's headline: a million vertices, 64-bit keys
        {"name": "build-rmat20", "kind": "build", "graph": "rmat", "n": 1 << 20, "wmax": 65536},
        # a road-like graph: long paths, long label lists, pruning does not pay
        {"name": "build-grid512", "kind": "build", "graph": "grid", "rows": 512, "cols": 512, "wmax": 10000},
        # a directed social graph: out- and in-labels in one build
        {"name": "build-directed16", "kind": "build", "graph": "rmat", "n": 65536, "wmax": 1000, "directed": True},
        # the Hybrid under a ranking that covers few shortest paths
        {"name": "build-hybrid15", "kind": "build", "graph": "rmat", "n": 32768, "wmax": 1000, "psi": 100},
        # one interactive query: latency
        {"name": "query-one", "kind": "query", "graph": "rmat", "n": 65536, "wmax": 1000, "q": 1},
        # a batch over short label lists
        {"name": "query-rmat16", "kind": "query", "graph": "rmat", "n": 65536, "wmax": 1000, "q": 1000000},
        # a batch over long label lists
        {"name": "query-grid512", "kind": "query", "graph": "grid", "rows": 512, "cols": 512, "wmax": 10000,
         "q": 1000000},
        # a labeling made ready for path queries (a parent per label), then a
        # batch of shortest paths
        {"name": "paths-rmat16", "kind": "paths", "graph": "rmat", "n": 65536, "wmax": 1000, "q": 100000},
        # the server with its queue full: host memory in, host memory out
        {"name": "serve-rmat16", "kind": "serve", "graph": "rmat", "n": 65536, "wmax": 1000, "q": 200000},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["build", "build", "build", "query", "query", "query", "paths", "serve"])
    graph = "rmat" if kind == "serve" else rng.choice(["rmat", "rmat", "grid"])
    case = {"kind": kind, "graph": graph}
    if graph == "grid":
        top = 500 if kind in ("build", "query") else 250
        case["rows"], case["cols"] = _log(rng, 24, top), _log(rng, 24, top)
        case["wmax"] = rng.choice([100, 1000, 10000])
    else:
        case["n"] = _log(rng, 1000, 600000 if kind == "build" else 150000)
        case["wmax"] = rng.choice([100, 1000, 65536])
        if kind in ("build", "query") and rng.random() < 0.25:
            case["directed"] = True
            case["n"] = min(case["n"], 100003)
        elif kind == "build" and rng.random() < 0.15:
            case["psi"] = rng.choice([50, 100, 500])
            case["n"] = _log(rng, 1000, 30000)
    if kind == "query":
        case["q"] = _log(rng, 1, 1000000)
    elif kind == "paths":
        case["q"] = _log(rng, 100, 100000)
    elif kind == "serve":
        case["q"] = _log(rng, 1000, 200000)
    return case


# ------------------------------------------------------------------ inputs
def _size(case):
    return case["rows"] * case["cols"] if case["graph"] == "grid" else case["n"]


def _edges(case, gen):
    """Distinct edges (u < v), or distinct arcs u -> v of a directed graph,
    sorted, as one int64 key u * n + v each."""
    n = _size(case)
    if case["graph"] == "grid":
        rows, cols = case["rows"], case["cols"]
        ids = torch.arange(n, dtype=torch.int64, device=DEV)
        r, c = ids // cols, ids % cols
        right, down = ids[c < cols - 1], ids[r < rows - 1]
        keys = [right * n + right + 1, down * n + down + cols]
        if rows >= 128:
            hit = torch.rand(n, generator=gen, device=DEV) < 0.05
            to = c + 2 * torch.randint(0, 2, (n,), generator=gen, device=DEV) - 1
            src = ids[hit & (r < rows - 1) & (to >= 0) & (to < cols)]
            keys.append(src * n + (src // cols + 1) * cols + to[src])
        return torch.unique(torch.cat(keys))
    scale = max(1, (n - 1).bit_length())
    u = torch.zeros(8 * n, dtype=torch.int64, device=DEV)
    v = torch.zeros_like(u)
    for _ in range(scale):
        x = torch.rand(8 * n, generator=gen, device=DEV)
        v = 2 * v + (((x >= RMAT_A) & (x < RMAT_AB)) | (x >= RMAT_ABC)).to(torch.int64)
        u = 2 * u + (x >= RMAT_AB).to(torch.int64)
    keep = (u != v) & (u < n) & (v < n)
    u, v = u[keep], v[keep]
    if not case.get("directed"):
        u, v = torch.minimum(u, v), torch.maximum(u, v)
    return torch.unique(u * n + v)


def _graph(case, seed):
    """(row_ptr, col, w, order) on the device, and the generator."""
    n = _size(case)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    key = _edges(case, gen)
    w = torch.randint(1, case["wmax"] + 1, (key.numel(),), generator=gen, device=DEV, dtype=torch.int32)
    u, v = key // n, key % n
    if not case.get("directed"):
        key, at = torch.sort(torch.cat([u * n + v, v * n + u]))
        w = torch.cat([w, w])[at]
    src, col = key // n, (key % n).to(torch.int32)
    deg = torch.bincount(src, minlength=n)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cumsum(deg, 0)
    order = torch.randperm(n, generator=gen, device=DEV)
    if "psi" not in case:
        rank = deg + torch.bincount(col.to(torch.int64), minlength=n)
        order = order[torch.argsort(rank[order], descending=True, stable=True)]
    return row_ptr, col, w, order.to(torch.int32), gen


def _labels(case, graph):
    """The labeling that a querying program holds (built without tuning)."""
    return chl.build(*graph[:4], directed=bool(case.get("directed")), autotune=False, stats=False,
                     prune_hubs=-1 if case["graph"] == "grid" else 0)


def _pairs(case, graph):
    """Uniform pairs, as the benchmark's batches; the few pairs of an
    interactive caller are vertices with arcs."""
    n, q, (_, col, _, _, gen) = _size(case), case["q"], graph
    if q > 64:
        return torch.randint(0, n, (q, 2), generator=gen, device=DEV, dtype=torch.int32)
    return col[torch.randint(0, col.numel(), (q, 2), generator=gen, device=DEV)]


def _rooms(*sizes):
    """The caller's result arrays: fixed room, -1 behind what a pass fills."""
    return [torch.full((n,), -1, dtype=t, device=DEV) for n, t in sizes]


def _fill(room, x):
    room[:x.numel()].copy_(x)
    return room


def prepare(case, seed):
    graph = _graph(case, seed)
    state = {"case": dict(case), "graph": graph[:4]}
    if case["kind"] == "build":
        cap = _label_cap(case)
        state["out"] = _rooms(*[(cap, torch.int32)] * (4 if case.get("directed") else 2))
        return state
    state["labels"] = _labels(case, graph)
    pairs = _pairs(case, graph)
    if case["kind"] == "paths":
        cap = _label_cap(case)
        state["out"] = _rooms((cap, torch.int32), (cap, torch.int32), (_path_cap(case), torch.int32))
    if case["kind"] != "serve":
        state["pairs"] = pairs
        return state
    state["pairs"] = pairs.cpu().numpy()
    state["arrival"] = np.zeros(case["q"], np.float64)
    state["server"] = serve.Server()
    state["gid"] = state["server"].add_labels(state["labels"])
    return state


# ------------------------------------------------------------------ a pass
def run(state):
    case = state["case"]
    if case["kind"] == "build":
        L = chl.build(*state["graph"], directed=bool(case.get("directed")), hybrid_psi=case.get("psi", 0))
        off, hub, dist = L.export("cuda")
        out = [off, _fill(state["out"][0], hub), _fill(state["out"][1], dist)]
        if case.get("directed"):
            off, hub, dist = L.export_in("cuda")
            out += [off, _fill(state["out"][2], hub), _fill(state["out"][3], dist)]
        L.free()
        return out
    if case["kind"] == "query":
        return state["labels"].query(state["pairs"])
    if case["kind"] == "paths":
        L = state["labels"]
        parent, slot = L.parents(*state["graph"][:3])
        hops, off, path = L.paths(state["pairs"], parent, slot)
        return [hops, off] + [_fill(a, b) for a, b in zip(state["out"], (parent, slot, path))]
    ticket = state["server"].submit_queries(state["gid"], state["pairs"], state["arrival"])
    state["server"].start()
    state["server"].wait()
    return ticket.out


# ------------------------------------------------------------------ work
def _label_count(case):
    """About how many labels the (out-)labeling holds, from builds of these
    generators: average list length against n."""
    n = _size(case)
    if case["graph"] == "grid":
        return n * max(8.0, 118.0 * (n / 4096.0) ** 0.42)
    if "psi" in case:
        return n * max(8.0, 2800.0 * (n / 65536.0) ** 0.8)
    return n * 26.0 * (n / 65536.0) ** 0.2


def _label_cap(case):
    return int(1.6 * _label_count(case)) + 4096


def _path_vertices(case):
    """About how many vertices the paths of a case's pairs hold."""
    if case["graph"] == "grid":
        return case["q"] * 0.45 * (case["rows"] + case["cols"])
    return case["q"] * 0.4 * 9.0


def _path_cap(case):
    return int(1.6 * _path_vertices(case)) + 4096


def work(case):
    """Each input read once, each output written once; for queries the two
    lists' hubs, for paths one lookup per (arc, label) as well."""
    n, labels = _size(case), _label_count(case)
    arcs = (4.2 if case["graph"] == "grid" else 14.5) * n
    lists = labels / n
    if case["kind"] == "build":
        sets = 2 if case.get("directed") else 1
        return {"bytes": 12.0 * n + 8.0 * arcs / sets + sets * (8.0 * n + 8.0 * labels), "flops": 0}
    q = case["q"]
    merge = q * (16.0 + 32.0 + 2 * 4.0 * lists)
    if case["kind"] == "paths":
        return {"bytes": 16.0 * labels + 12.0 * n + 8.0 * arcs + 2 * merge + 4.0 * _path_vertices(case), "flops": 0}
    return {"bytes": merge, "flops": 0}


# ------------------------------------------------------------------ oracle
def _all_distances(n, row_ptr, col, w):
    """All-pairs distances by Floyd's recurrence, int64 (INF: no path)."""
    inf = 1 << 40
    src = torch.repeat_interleave(torch.arange(n, device=DEV), row_ptr[1:] - row_ptr[:-1])
    d = torch.full((n * n,), inf, dtype=torch.int64, device=DEV)
    d.scatter_reduce_(0, src * n + col.to(torch.int64), w.to(torch.int64), "amin")
    d = d.view(n, n)
    d.fill_diagonal_(0)
    for x in range(n):
        torch.minimum(d, d[:, x:x + 1] + d[x:x + 1, :], out=d)
    return d, inf


def _some_distances(n, row_ptr, col, w, pairs):
    """Distances of a few pairs: Bellman-Ford from their distinct sources."""
    inf = 1 << 40
    src = torch.repeat_interleave(torch.arange(n, device=DEV), row_ptr[1:] - row_ptr[:-1])
    starts, at = torch.unique(pairs[:, 0].to(torch.int64), return_inverse=True)
    d = torch.full((starts.numel(), n), inf, dtype=torch.int64, device=DEV)
    d.scatter_(1, starts[:, None], 0)
    dst = col.to(torch.int64)[None, :].expand(starts.numel(), -1)
    for _ in range(n):
        nd = d.scatter_reduce(1, dst, d[:, src] + w.to(torch.int64), "amin")
        if torch.equal(nd, d):
            break
        d = nd
    got = d[at, pairs[:, 1].to(torch.int64)]
    return torch.where(got >= inf, -1, got)


def _canonical(n, d, inf, order):
    """Both label sets by the definition: the highest-ranked vertex x of all
    shortest a-b paths, for all a, b in rank order."""
    o = order.to(torch.int64)
    d = d[o][:, o].contiguous()
    top = torch.full((n, n), n, dtype=torch.int32, device=DEV)
    for x in range(n - 1, -1, -1):
        top.masked_fill_(d[:, x:x + 1] + d[x:x + 1, :] == d, x)
    ids = torch.arange(n, device=DEV, dtype=torch.int32)
    reach = d < inf
    back = torch.empty_like(o)
    back[o] = torch.arange(n, device=DEV)

    def lists(is_label, dist):       # [vertex position, hub position]
        is_label, dist = is_label[back], dist[back]
        off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(is_label.sum(1), 0)
        at = is_label.nonzero()
        return off, at[:, 1].to(torch.int32), dist[at[:, 0], at[:, 1]].to(torch.int32)

    out = lists((top == ids[None, :]) & reach, d)
    inn = lists(((top == ids[:, None]) & reach).t().contiguous(), d.t().contiguous())
    return out, inn


def exact(case, seed):
    n = _size(case)
    if case["kind"] == "build" and n <= 4096:
        row_ptr, col, w, order, _ = _graph(case, seed)
        d, inf = _all_distances(n, row_ptr, col, w)
        room = _rooms(*[(_label_cap(case), torch.int32)] * 4)
        out, inn = _canonical(n, d, inf, order)
        return [out[0], _fill(room[0], out[1]), _fill(room[1], out[2])] + (
            [inn[0], _fill(room[2], inn[1]), _fill(room[3], inn[2])] if case.get("directed") else [])
    if case["kind"] == "query" and (n <= 4096 or case["q"] <= 16):
        graph = _graph(case, seed)
        pairs, (row_ptr, col, w) = _pairs(case, graph), graph[:3]
        if case["q"] <= 16 and case["graph"] == "rmat":
            return _some_distances(n, row_ptr, col, w, pairs)
        if n <= 4096:
            d, inf = _all_distances(n, row_ptr, col, w)
            got = d[pairs[:, 0].to(torch.int64), pairs[:, 1].to(torch.int64)]
            return torch.where(got >= inf, -1, got)
    return None
