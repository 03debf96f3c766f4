"""Timed cases of the shortest-path framework: what its users call, over the sizes they call it with.

A case names a network (grid, road, oneway, rmat), a call (single queries in turn, one batch, all distances from a
source, a burst of requests to the server) and the options of that call. The network of a case is fixed, as the one
that a routing service holds resident; the queries come from the seed. Distances are returned as int64, -1 where
there is no path.
"""
import json
import math
import random

import numpy as np
import torch

import paper_2506_16488_amd as P

FRAC_BITS = 8          # coordinates: fixed point with 8 fractional bits, unit cells
W_SCALE = 1000         # road weight: ceil(1000 * Euclidean length)


def listed():
    return [
        # the smallest call: one route question on a city-sized grid (256 x 256, weights U[1, 1000])
        {"name": "grid256_query", "net": "grid", "rows": 256, "cols": 256, "wmax": 1000, "call": "query", "pairs": 1,
         "algo": "bids"},
        # a route planner answering one question after another on a road network with coordinates
        {"name": "road1024_queries", "net": "road", "rows": 1024, "cols": 1024, "call": "query", "pairs": 8,
         "algo": "bidastar"},
        # turn-by-turn routes: a small batch that asks for the paths too; odd sizes, wide weights (unique paths)
        {"name": "grid_routes16", "net": "grid", "rows": 333, "cols": 517, "wmax": 1 << 20, "call": "batch",
         "pairs": 16, "algo": "bids", "batch": "plainstar", "paths": True},
        # the small batch: 64 pairs on the 256 x 256 grid
        {"name": "grid256_batch64", "net": "grid", "rows": 256, "cols": 256, "wmax": 1000, "call": "batch",
         "pairs": 64, "algo": "bids", "batch": "plainstar"},
        # the road batch: bidirectional A* on the 2048 x 2048 jittered lattice
        {"name": "road2048_batch256", "net": "road", "rows": 2048, "cols": 2048, "call": "batch", "pairs": 256,
         "algo": "bidastar", "batch": "plainstar"},
        # one-sided A*, on a lattice whose sides are no round numbers
        {"name": "road_odd_astar100", "net": "road", "rows": 769, "cols": 1023, "call": "batch", "pairs": 100,
         "algo": "astar", "batch": "plainstar"},
        # a depot batch: half of the pairs share a few sources, answered by shared searches
        {"name": "road1024_depots192", "net": "road", "rows": 1024, "cols": 1024, "call": "batch", "pairs": 192,
         "algo": "bids", "batch": "multi", "hubs": 8},
        # a directed road network (each direction its own weight): the backward searches walk the transpose
        {"name": "oneway_batch48", "net": "oneway", "rows": 700, "cols": 901, "call": "batch", "pairs": 48,
         "algo": "bids", "batch": "plainstar"},
        # one question after another on a power-law network, with the library's defaults
        {"name": "rmat20_queries", "net": "rmat", "scale": 20, "call": "query", "pairs": 4, "algo": "bids"},
        # the power-law batch with the setting the autotuner picks there (bucketed steps, dense frontiers): the largest
        {"name": "rmat22_batch128", "net": "rmat", "scale": 22, "call": "batch", "pairs": 128, "algo": "bids",
         "batch": "plainstar", "delta": 1433, "tuned": True},
        # all distances from one source
        {"name": "road1024_sssp", "net": "road", "rows": 1024, "cols": 1024, "call": "sssp", "pairs": 1,
         "algo": "sssp"},
        # a burst of mixed-size requests to the server, a road and a power-law network resident together
        {"name": "serve_burst", "net": "road", "rows": 1024, "cols": 1024, "call": "serve", "scale": 17,
         "requests": 16, "pairs": 32, "algo": "bidastar"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ranges: any network, call and algorithm, sizes over their logarithm."""
    kind = rng.choice(["query", "query", "batch", "batch", "batch", "routes", "multi", "rmat", "rmat", "sssp", "serve"])
    side = lambda: _log_int(rng, 64, 2048)  # noqa: E731
    if kind == "rmat":
        scale = rng.randint(14, 21)
        tuned = rng.random() < 0.5
        single = rng.random() < 0.3
        c = {"net": "rmat", "scale": scale, "call": "query" if single else "batch",
             "pairs": rng.randint(1, 8) if single else _log_int(rng, 2, 128), "algo": "bids",
             "delta": _log_int(rng, 1000, 6000) if tuned else 0, "tuned": tuned}
        return c if single else dict(c, batch="plainstar")
    if kind == "serve":
        return {"net": "road", "rows": _log_int(rng, 128, 1024), "cols": _log_int(rng, 128, 1024), "call": "serve",
                "scale": rng.randint(13, 17), "requests": rng.randint(2, 16), "pairs": _log_int(rng, 2, 32),
                "algo": rng.choice(["bids", "bidastar"])}
    net = rng.choice(["grid", "road", "road", "oneway"])
    c = {"net": net, "rows": side(), "cols": side()}
    n = c["rows"] * c["cols"]
    if net == "grid":
        c["wmax"] = rng.choice([1000, 65535, 1 << 20])
    algos = ["bids", "et"] if net == "grid" else ["bids", "bidastar", "bidastar", "astar", "et"]
    if kind == "sssp":
        return dict(c, call="sssp", pairs=1, algo="sssp")
    if kind == "query":
        return dict(c, call="query", pairs=rng.randint(1, 8), algo=rng.choice(algos))
    if kind == "routes":
        return dict(c, net="grid", wmax=1 << 20, call="batch", pairs=_log_int(rng, 2, 64), algo="bids",
                    batch="plainstar", paths=True)
    most = max(2, min(256, (1 << 28) // n))
    if kind == "multi":
        return dict(c, call="batch", pairs=_log_int(rng, 2, most), algo="bids", batch="multi", hubs=rng.randint(1, 16))
    return dict(c, call="batch", pairs=_log_int(rng, 2, most), algo=rng.choice(algos), batch="plainstar")


# ---- networks, made on the GPU -------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _csr(n, src, dst, w):
    """Host CSR arrays of the arcs, each row by head."""
    order = torch.sort(src * n + dst).indices
    src, dst, w = src[order], dst[order], w[order]
    row = torch.zeros(n + 1, dtype=torch.int64, device=src.device)
    row[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return (row.cpu().numpy().astype(np.uint64), dst.to(torch.int32).cpu().numpy().view(np.uint32),
            w.to(torch.int32).cpu().numpy().view(np.uint32))


def _lattice(case):
    """grid: a 4-neighbour grid, weights U[1, wmax] per edge. road: one vertex jittered in each unit cell, 5% short
    diagonals, weight ceil(1000 * length). oneway: the road network, each direction up to twice as long."""
    R, C, dev = case["rows"], case["cols"], _device()
    g = torch.Generator(device=dev).manual_seed(1000003 * R + C)
    ids = torch.arange(R * C, device=dev).reshape(R, C)
    a = [ids[:, :-1].reshape(-1), ids[:-1, :].reshape(-1)]
    b = [ids[:, 1:].reshape(-1), ids[1:, :].reshape(-1)]
    if case["net"] == "grid":
        a, b = torch.cat(a), torch.cat(b)
        w = torch.randint(1, case["wmax"] + 1, a.shape, generator=g, device=dev)
        return (R * C, *_csr(R * C, torch.cat([a, b]), torch.cat([b, a]), torch.cat([w, w])), None)
    diag = torch.rand((R - 1, C - 1), generator=g, device=dev) < 0.05
    a.append(ids[:-1, :-1][diag])
    b.append(ids[1:, 1:][diag])
    a, b = torch.cat(a), torch.cat(b)
    unit = 1 << FRAC_BITS
    jitter = torch.randint(0, unit, (R * C, 2), generator=g, device=dev)
    xy = torch.stack([(ids % C).reshape(-1), (ids // C).reshape(-1)], 1) * unit + jitter
    d2 = (xy[a] - xy[b]).square().sum(1)
    # ceil(W_SCALE * sqrt(d2) / unit) in whole numbers: the smallest w with (w * unit)^2 >= W_SCALE^2 * d2
    w = torch.ceil(W_SCALE * torch.sqrt(d2.double()) / unit).long()
    w = torch.where(((w - 1) * unit).square() >= W_SCALE * W_SCALE * d2, w - 1, w)
    w = torch.where((w * unit).square() < W_SCALE * W_SCALE * d2, w + 1, w).clamp_(min=1)
    w2 = torch.cat([w, w])
    if case["net"] == "oneway":
        w2 = w2 + (torch.rand(w2.shape, generator=g, device=dev) * w2).long()
    return (R * C, *_csr(R * C, torch.cat([a, b]), torch.cat([b, a]), w2), xy.to(torch.int32).cpu().numpy())


def _rmat(scale):
    """R-MAT (0.57, 0.19, 0.19, 0.05), edge factor 16, symmetrised and deduplicated, weights U[1, 65535]."""
    n, e, dev = 1 << scale, 16 << scale, _device()
    g = torch.Generator(device=dev).manual_seed(77 + scale)
    u = torch.zeros(e, dtype=torch.int64, device=dev)
    v = torch.zeros(e, dtype=torch.int64, device=dev)
    for _ in range(scale):
        r = torch.rand(e, generator=g, device=dev)
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    relabel = torch.randperm(n, generator=g, device=dev)
    u, v = relabel[u], relabel[v]
    key = torch.unique((torch.minimum(u, v) * n + torch.maximum(u, v))[u != v])
    u, v = key // n, key % n
    w = torch.randint(1, 65536, u.shape, generator=g, device=dev)
    return (n, *_csr(n, torch.cat([u, v]), torch.cat([v, u]), torch.cat([w, w])), None)


_arrays, _handle = {}, {}


def _kept(cache, key, make):
    """The last network (or its handle) stays, as in a program that holds one."""
    if key not in cache:
        cache.clear()
        cache[key] = make()
    return cache[key]


def _host(case):
    key = json.dumps([case["net"], case.get("rows"), case.get("cols"), case.get("wmax"),
                      case["scale"] if case["net"] == "rmat" else None])

    def make():
        a = _rmat(case["scale"]) if case["net"] == "rmat" else _lattice(case)
        if torch.cuda.is_available():
            torch.cuda.empty_cache()
        return a
    return _kept(_arrays, key, make)


def _graph(case):
    n, row, col, w, xy = _host(case)
    g = P.Graph(n, row, col, w, xy, FRAC_BITS, W_SCALE, symmetric=case["net"] != "oneway",
                reorder=case["net"] in ("road", "rmat"))
    if case.get("tuned"):
        g.set_option("theta_mode", 1)
        g.set_option("dense_min", 1 << 16)
        g.set_option("dense_ring", 32)
    return g


def _make_handle(case):
    if case["call"] != "serve":
        return _graph(case)
    power = {"net": "rmat", "scale": case["scale"]}
    road = _graph(case)
    return P.Server([road, _graph(power)], algo=[case["algo"], "bids"], state_budget_bytes=4 << 30)


def _pairs(case, seed):
    """The queries of a seed: uniform pairs among the vertices that have an arc; with hubs, the first half from them."""
    rng = np.random.default_rng([seed, case["pairs"]])
    k = case["pairs"]
    if case["net"] == "rmat":
        row = _host(case)[1]
        some = np.nonzero(row[1:] != row[:-1])[0]
        p = some[rng.integers(0, some.size, (k, 2))]
    else:
        p = rng.integers(0, case["rows"] * case["cols"], (k, 2))
    if case.get("hubs"):
        hub = rng.integers(0, case["rows"] * case["cols"], case["hubs"])
        p[: k // 2, 0] = hub[rng.integers(0, case["hubs"], k // 2)]
    return np.ascontiguousarray(p, np.uint32)


def _requests(case, seed):
    """A burst of requests: graph by graph in turn, sizes (the case's own) over their logarithm up to `pairs`."""
    rng = random.Random(case["requests"] * 1000 + case["pairs"])
    out = []
    for j in range(case["requests"]):
        size = _log_int(rng, 1, case["pairs"])
        c = dict(case, pairs=size) if j % 2 == 0 else {"net": "rmat", "scale": case["scale"], "pairs": size}
        out.append((j % 2, c, seed * 1009 + j))
    pairs = [None] * len(out)
    for graph in (1, 0):          # one network at a time
        for j, (g, c, s) in enumerate(out):
            if g == graph:
                pairs[j] = _pairs(c, s)
    return [(g, p) for (g, _, _), p in zip(out, pairs)]


# ---- one pass --------------------------------------------------------------------

def prepare(case, seed):
    key = json.dumps({k: v for k, v in case.items() if k in
                      ("net", "rows", "cols", "wmax", "scale", "tuned") or (k == "call" and v == "serve")
                      or (k == "algo" and case["call"] == "serve")}, sort_keys=True)
    handle = _kept(_handle, key, lambda: _make_handle(case))
    if case["call"] == "serve":
        return {"case": case, "handle": handle, "requests": _requests(case, seed)}
    return {"case": case, "handle": handle, "pairs": _pairs(case, seed)}


def run(state):
    case, h = state["case"], state["handle"]
    call = case["call"]
    if call == "serve":
        ids = [h.submit(g, p) for g, p in state["requests"]]
        return [h.wait(i)[0].view(np.int64) for i in ids]
    pairs = state["pairs"]
    if call == "query":
        d = np.array([h.query(int(s), int(t), algo=case["algo"], delta=case.get("delta", 0)) for s, t in pairs],
                     np.uint64)
        return d.view(np.int64)
    if call == "sssp":
        return h.sssp(int(pairs[0, 0])).view(np.int64)
    out = h.batch_query(pairs, algo=case["algo"], batch=case["batch"], delta=case.get("delta", 0),
                        want_path=case.get("paths", False))
    if case.get("paths"):
        d, (off, vtx) = out
        routes = np.full(4 * len(pairs) * (case["rows"] + case["cols"]), -1, np.int32)   # one length for every seed
        routes[: vtx.size] = vtx.view(np.int32)
        return [d.view(np.int64), off.view(np.int64), routes]
    return out.view(np.int64)


# ---- what a pass cannot do without -------------------------------------------------

# Share of the network's vertices that a search for a uniform pair has to settle: two discs of half the distance
# (bidirectional), one disc of the whole distance (early termination), and what the heuristic leaves of them.
SHARE = {"bids": 0.4, "et": 0.6, "sssp": 1.0, "astar": 0.25, "bidastar": 0.12}
DEGREE = {"grid": 4.0, "road": 4.1, "oneway": 4.1, "rmat": 30.0}


def _search_bytes(net, n, share, queries):
    """Per settled vertex its row bounds (8) and distance (8 written); per arc of it the arc (8) and the head's
    distance (8); the network's arrays are read once for the whole batch."""
    settled = share * n * queries
    d = DEGREE[net]
    return min(settled, n) * (8 + 8 * d) + settled * (8 + 8 * d)


def work(case):
    if case["call"] == "serve":
        half = case["requests"] * case["pairs"] / 5.0     # mean size of a request whose size is drawn over its logarithm
        road = _search_bytes("road", case["rows"] * case["cols"], SHARE[case["algo"]], half)
        return {"bytes": road + _search_bytes("rmat", 1 << case["scale"], 0.3, half), "flops": 0}
    n = 1 << case["scale"] if case["net"] == "rmat" else case["rows"] * case["cols"]
    share = 0.3 if case["net"] == "rmat" else SHARE[case["algo"]]
    b = _search_bytes(case["net"], n, share, case["pairs"])
    if case["call"] == "sssp":
        b += 8 * n
    return {"bytes": b + 16 * case["pairs"], "flops": 0}


# ---- the same distances from plain torch -------------------------------------------

def _distances(case, sources):
    """Distances from each source to every vertex: rounds of relaxing all arcs until nothing changes, in int64."""
    n, row, col, w, _ = _host(case)
    dev = _device()
    row = torch.from_numpy(row.astype(np.int64)).to(dev)
    dst = torch.from_numpy(col.astype(np.int64)).to(dev)
    w = torch.from_numpy(w.astype(np.int64)).to(dev)
    src = torch.repeat_interleave(torch.arange(n, device=dev), row[1:] - row[:-1])
    far = 1 << 60
    d = torch.full((n, len(sources)), far, dtype=torch.int64, device=dev)
    d[torch.tensor(sources, device=dev), torch.arange(len(sources), device=dev)] = 0
    while True:
        before = d.clone()
        for _ in range(16):
            d.index_reduce_(0, dst, d[src] + w[:, None], "amin")
        if torch.equal(before, d):
            break
    d[d >= far] = -1
    return d


def exact(case, seed):
    """None where it would take long: many sources on a large network."""
    if case["call"] == "serve":
        return None
    pairs = _pairs(case, seed).astype(np.int64)
    sources = sorted(set(pairs[:, 0].tolist()))
    n = 1 << case["scale"] if case["net"] == "rmat" else case["rows"] * case["cols"]
    rounds = 40 if case["net"] == "rmat" else 2.5 * (case["rows"] + case["cols"])
    if n * DEGREE[case["net"]] * len(sources) * rounds > 4e10:
        return None
    d = _distances(case, sources)
    if case["call"] == "sssp":
        return d[:, 0].cpu().numpy()
    col = {s: j for j, s in enumerate(sources)}
    got = d[torch.from_numpy(pairs[:, 1]).to(d.device), torch.tensor([col[s] for s in pairs[:, 0].tolist()], device=d.device)]
    got = got.cpu().numpy()
    return [got, None, None] if case.get("paths") else got
