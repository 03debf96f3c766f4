"""Resident searches (option "resident": one workgroup per query) against the
oracle at the sizes where they can go wrong: ties and zero weights, the
degrees on both sides of the limit, more bids in a round than fit, more
queries than compute units (both workgroup sizes), frontiers beyond the LDS
queue, directed graphs, unreachable pairs, paths, all distances, the time
limit, and the calls that keep to rounds. Distances are integers: equality."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
INF = (1 << 64) - 1


@pytest.fixture(scope="module")
def P():
    import paper_2506_16488_amd as P
    P.lib()
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return P


def _open(P, g, **kw):
    G = P.Graph.from_host(g, **kw)
    G.set_option("timeout_ms", 60000)
    return G


def _check(G, g, pairs, algos, want_resident=True):
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    for algo in algos:
        print("resident", g.n, algo, len(pairs), flush=True)
        assert np.array_equal(G.batch_query(pairs, algo=algo), exp), algo
        assert (G.stats()["relax_launches"] == 1) == want_resident
        G.set_option("resident", 0)
        assert np.array_equal(G.batch_query(pairs, algo=algo), exp), algo
        assert G.stats()["relax_launches"] > 1
        G.set_option("resident", 1)
    return exp


@pytest.mark.parametrize("wlo,whi", [(1, 1), (0, 1), (0, 3), (1, 1 << 24)])
def test_ties_and_zero_weights(P, wlo, whi):
    """Many equal distances in a round: one entry each; zero-weight arcs."""
    g = gen.grid(61, 67, wlo, whi, seed=3)
    _check(_open(P, g), g, gen.pairs_uniform(g.n, 40, seed=4), ["bids", "et", "sssp"])


@pytest.mark.parametrize("shape", [(1, 2), (1, 4000), (2, 3), (640, 3), (97, 131)])
def test_narrow_grids(P, shape):
    g = gen.grid(*shape, 1, 1000, seed=5)
    _check(_open(P, g), g, gen.pairs_uniform(g.n, 33, seed=6, distinct=g.n > 40), ["bids", "et"])


@pytest.mark.parametrize("deg,resident", [(63, True), (64, True), (65, False)])
def test_degree_limit(P, deg, resident):
    """Stars joined in a chain, inner hubs of that degree; 65 goes in rounds."""
    k, leaves = 48, deg - 2
    rng = np.random.default_rng(deg)
    hub = np.arange(k) * (leaves + 1)
    leaf = np.setdiff1d(np.arange(k * (leaves + 1)), hub)
    src = np.concatenate([np.repeat(hub, leaves), hub[:-1]])
    dst = np.concatenate([leaf, hub[1:]])
    g = gen.csr_from_edges(k * (leaves + 1), src, dst, rng.integers(1, 50, src.size))
    assert np.diff(g.row_ptr.astype(np.int64)).max() == deg
    _check(_open(P, g), g, gen.pairs_uniform(g.n, 30, seed=deg), ["bids", "et", "sssp"], resident)


def test_more_bids_than_fit(P):
    """A block of mean degree 49 (thousands of bids in a round) on a long path, which keeps the mean degree low."""
    rng = np.random.default_rng(8)
    n, tail = 3000, 12000
    src = np.repeat(np.arange(n), 25)
    dst = (src + rng.integers(1, 400, src.size)) % n
    deg = np.bincount(src, minlength=n) + np.bincount(dst, minlength=n)
    big = np.nonzero(deg > 63)[0]
    keep = (src != dst) & ~np.isin(src, big) & ~np.isin(dst, big)
    src = np.concatenate([src[keep], [0], np.arange(n, n + tail - 1)])
    dst = np.concatenate([dst[keep], [n], np.arange(n + 1, n + tail)])
    g = gen.csr_from_edges(n + tail, src, dst, rng.integers(1, 3, src.size))
    deg = np.diff(g.row_ptr.astype(np.int64))
    assert deg.max() <= 64 and deg[:n].mean() > 40 and g.m <= 16 * g.n
    _check(_open(P, g), g, gen.pairs_uniform(n, 60, seed=9), ["bids", "et", "sssp"])


@pytest.mark.parametrize("k", [255, 257, 512, 513, 700])
def test_more_queries_than_units(P, k):
    """512 queries run 1,024 threads each, 513 on a small graph 512 threads."""
    g = gen.lattice(70, 0.1, seed=10)
    _check(_open(P, g, reorder=True), g, gen.pairs_uniform(g.n, k, seed=11), ["bidastar", "bids", "astar"])


def test_frontier_beyond_lds(P):
    """A lattice whose frontiers pass the LDS queue (and, at step 2^40, hold every vertex reached)."""
    g = gen.lattice(400, 0.05, seed=12)
    pairs = np.concatenate([gen.pairs_uniform(g.n, 12, seed=13), [[0, g.n - 1], [399, g.n - 400]]]).astype(np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = _open(P, g)
    for algo in ["bids", "bidastar", "et", "astar"]:
        for delta in [1, 300, 0, 20000, 1 << 40]:
            if delta == 1 and algo in ("et", "bids"):
                continue                       # one distance a round: thousands of rounds
            print("beyond lds", algo, delta, flush=True)
            assert np.array_equal(G.batch_query(pairs, algo=algo, delta=delta), exp), (algo, delta)
    for mode in (0, 1, 3):
        G.set_option("theta_mode", mode)
        for algo in ["bids", "bidastar", "et"]:
            assert np.array_equal(G.batch_query(pairs, algo=algo), exp), (mode, algo)


def test_frontier_beyond_the_queue_runs_in_rounds(P):
    """A random part between two grids whose frontier outgrows every queue: the queries there
    run again in rounds, those on the grids keep their answers and paths."""
    rng = np.random.default_rng(14)
    a, b = gen.grid(20, 20, 1, 9, seed=15), gen.grid(240, 300, 1, 9, seed=16)
    mid, n = 60000, 400 + 60000 + 72000
    arcs = [(np.repeat(np.arange(x.n), np.diff(x.row_ptr.astype(np.int64))) + base, x.col + base, x.w)
            for x, base in ((a, 0), (b, 400 + mid))]
    arcs.append((rng.integers(400, 400 + mid, 6 * mid), rng.integers(400, 400 + mid, 6 * mid),
                 rng.integers(1, 1 << 20, 6 * mid)))
    g = gen.csr_from_edges(n, *(np.concatenate(x) for x in zip(*arcs)))
    pairs = np.concatenate([gen.pairs_uniform(400, 5, seed=16), gen.pairs_uniform(mid, 6, seed=17) + 400,
                            gen.pairs_uniform(72000, 5, seed=18) + 400 + mid, [[3, 900]]]).astype(np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = _open(P, g)
    for algo in ["bids", "et", "sssp"]:
        dist, (off, vtx) = G.batch_query(pairs, algo=algo, want_path=True, delta=1 << 30)
        assert np.array_equal(dist, exp), algo
        if algo != "bids":
            assert G.stats()["relax_launches"] > 1
        for q in range(len(pairs)):
            if exp[q] != INF:
                assert oracle.check_path(g.n, g.row_ptr, g.col, g.w, vtx[off[q]:off[q + 1]], int(pairs[q, 0]),
                                         int(pairs[q, 1]), int(exp[q])) == (0, 0), (algo, q)
    assert np.array_equal(G.batch_query(pairs, algo="sssp", batch="vc", delta=1 << 30), exp)


@pytest.mark.parametrize("symmetric", [True, False])
@pytest.mark.parametrize("verts,k,resident", [(2, 1, True), (9, 36, True), (33, 528, True), (36, 630, False), (300, 200, True)])
def test_shared_batches(P, symmetric, verts, k, resident):
    """Multi-BiDS: every query on its own searches up to 16 pairs a query-graph vertex, shared beyond; with paths."""
    g = gen.lattice(60, 0.1, seed=30)
    rng = np.random.default_rng(31)
    if not symmetric:
        g.w = (g.w + rng.integers(0, 800, g.w.size)).astype(np.uint32)
        g.symmetric = False
    v = rng.choice(g.n, verts, replace=False)
    pairs = np.array([(v[i], v[j]) for i in range(verts) for j in range(i)])
    pairs = pairs[rng.choice(len(pairs), k, replace=False)].astype(np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = _open(P, g)
    dist, (off, vtx) = G.batch_query(pairs, algo="bids", batch="multi", want_path=True)
    assert np.array_equal(dist, exp)
    if symmetric:      # on a directed graph a vertex is two of the query graph: a source and a target
        assert (G.stats()["relax_launches"] == 1) == resident
        assert G.stats()["searches"] == len(np.unique(pairs))
    for q in range(k):
        assert oracle.check_path(g.n, g.row_ptr, g.col, g.w, vtx[off[q]:off[q + 1]], int(pairs[q, 0]),
                                 int(pairs[q, 1]), int(exp[q])) == (0, 0), q


def test_directed_paths_and_all_distances(P):
    g = gen.lattice(90, 0.1, seed=18)
    rng = np.random.default_rng(19)
    g.w = (g.w + rng.integers(0, 800, g.w.size)).astype(np.uint32)
    g.symmetric = False
    pairs = gen.pairs_uniform(g.n, 40, seed=20)
    G = _open(P, g)
    exp = _check(G, g, pairs, ["bids", "bidastar", "et", "astar"])
    for algo in ["bids", "bidastar", "et", "astar"]:
        dist, (off, vtx) = G.batch_query(pairs, algo=algo, want_path=True)
        assert np.array_equal(dist, exp)
        for q in range(40):
            assert oracle.check_path(g.n, g.row_ptr, g.col, g.w, vtx[off[q]:off[q + 1]], int(pairs[q, 0]),
                                     int(pairs[q, 1]), int(exp[q])) == (0, 0), (algo, q)
    every = np.stack([np.full(g.n, 7), np.arange(g.n)], 1).astype(np.uint32)
    for reorder in (False, True):
        H = _open(P, g, reorder=reorder)
        assert np.array_equal(H.sssp(7), oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, every))


def test_time_limit(P):
    """The limit ends a launch with PPSP_E_TIMEOUT (or the call finished first), and the handle stays usable."""
    g = gen.grid(300, 300, 1, 1000, seed=21)
    pairs = np.array([[0, g.n - 1], [299, g.n - 300]], np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = _open(P, g)
    G.set_option("timeout_ms", 1)
    try:
        assert np.array_equal(G.batch_query(pairs, algo="et", delta=1), exp)
    except P.PPSPError as e:
        assert e.code == P.E_TIMEOUT
    G.set_option("timeout_ms", 60000)
    assert np.array_equal(G.batch_query(pairs, algo="et"), exp)


def _islands(g, isles, size, seed):
    """g with `isles` paths of `size` vertices spread through its numbering, the first and the last number among them."""
    n = g.n + isles * size
    at = np.unique(np.linspace(0, n - 1, isles * size).astype(np.int64))
    assert at.size == isles * size
    land = np.setdiff1d(np.arange(n), at)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr.astype(np.int64)))
    path = at.reshape(isles, size)
    return gen.csr_from_edges(n, np.concatenate([land[src], path[:, :-1].ravel()]),
                              np.concatenate([land[g.col], path[:, 1:].ravel()]),
                              np.concatenate([g.w, np.full(isles * (size - 1), 7, g.w.dtype)])), land


@pytest.mark.parametrize("isles,size", [(3, 1), (3, 7), (700, 2)])
def test_small_components_do_not_decide(P, isles, size):
    """Islands at the ends, in the middle and all over the numbering say nothing about the graph
    beside them: a random one (its balls grow fast) goes in rounds at once, a grid stays resident."""
    rng = np.random.default_rng(40)
    n = 40000
    fast = gen.csr_from_edges(n, np.repeat(np.arange(n), 4), rng.integers(0, n, 4 * n), rng.integers(1, 1000, 4 * n))
    for base, resident in ((fast, False), (gen.grid(150, 200, 1, 1000, seed=41), True)):
        g, land = _islands(base, isles, size, 42)
        assert np.diff(g.row_ptr.astype(np.int64)).max() <= 64
        pairs = land[gen.pairs_uniform(base.n, 40, seed=43)].astype(np.uint32)
        exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
        G = _open(P, g)
        for algo in ("bids", "et"):
            assert np.array_equal(G.batch_query(pairs, algo=algo), exp)
            launches = G.stats()["relax_launches"]
            assert launches == 1 if resident else launches > 1 and launches % 16 == 0, (isles, size, algo, launches)


def test_distances_near_the_limit(P):
    """Keys beyond 32 bits lose their order in a resident search, so a tentative distance can
    pass 2^32 where none does in rounds: an answer, not PPSP_E_OVERFLOW. Distances that do not
    fit are an error either way."""
    hops, tail = 30, 400
    a, v, x = 1, 2, 3
    chain = 4 + np.arange(hops)
    end = 4 + hops + np.arange(tail)
    src = [0, a, v] + [a, *chain] + list(end[:-1])
    dst = [a, v, x] + [*chain, v] + list(end[1:])
    w = [2147500000, 100000000, 2100000000] + [1000000] * (hops + 1) + [2000000] * (tail - 1)
    g = gen.csr_from_edges(int(end[-1]) + 1, np.array(src), np.array(dst), np.array(w, np.uint32), symmetric=False)
    G = _open(P, g)
    pairs = np.array([[0, end[-1]], [0, v], [a, x]], np.uint32)
    exp = [INF, 2147500000 + 31000000, 31000000 + 2100000000]
    for resident in (0, 1):
        G.set_option("resident", resident)
        for k in (1, 3):
            assert G.batch_query(pairs[:k], algo="bids", delta=1000000).tolist() == exp[:k], (resident, k)
    w[2] = 4000000000
    g = gen.csr_from_edges(int(end[-1]) + 1, np.array(src), np.array(dst), np.array(w, np.uint32), symmetric=False)
    G = _open(P, g)
    for resident in (0, 1):
        G.set_option("resident", resident)
        for algo in ("et", "sssp"):
            with pytest.raises(P.PPSPError) as e:
                G.batch_query(pairs[:1], algo=algo, delta=1000000)
            assert e.value.code == P.E_OVERFLOW


def test_time_limit_is_kept(P):
    """A search of many rounds, and a launch of many short ones, end with PPSP_E_TIMEOUT; the handle stays usable."""
    g = gen.grid(300, 300, 1, 1000, seed=44)
    pairs = np.array([[0, g.n - 1]], np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    s = gen.grid(20, 20, 1, 1000, seed=45)
    many = gen.pairs_uniform(s.n, 40000, seed=46, distinct=False)
    for h, p, delta in ((g, pairs, 1), (s, many, 0)):
        want = oracle.pp_batch(h.n, h.row_ptr, h.col, h.w, p[:500])
        G = _open(P, h)
        for algo in ("et", "sssp"):
            G.set_option("timeout_ms", 1)
            with pytest.raises(P.PPSPError) as e:
                G.batch_query(p, algo=algo, delta=delta)
            assert e.value.code == P.E_TIMEOUT
            G.set_option("timeout_ms", 60000)
            assert np.array_equal(G.batch_query(p[:500], algo=algo), want)
            assert G.stats()["relax_launches"] == 1
    # a limit whose clock ticks do not fit 64 bits is a long one (this one's product ends in 0.5 ms)
    G = _open(P, g)
    G.set_option("timeout_ms", 184467440737096)
    assert np.array_equal(G.batch_query(pairs, algo="et", delta=1), exp)
    assert G.stats()["relax_launches"] == 1


def _neighbours(side, seed):
    """A jittered lattice of `side` x `side` with 16 neighbours a vertex and coordinates."""
    rng = np.random.default_rng(seed)
    ids = np.arange(side * side).reshape(side, side)
    xy = np.stack([ids % side, ids // side], -1).reshape(-1, 2) * 256 + rng.integers(0, 256, (side * side, 2))
    a, b = [], []
    for dr, dc in ((0, 1), (1, 0), (1, 1), (1, -1), (0, 2), (2, 0), (1, 2), (2, -1)):
        a.append(ids[:side - dr, max(0, -dc):side - max(0, dc)].ravel())
        b.append(ids[dr:, max(0, dc):side + min(0, dc)].ravel())
    a, b = np.concatenate(a), np.concatenate(b)
    w = np.ceil(1000 * np.sqrt(((xy[a] - xy[b]) ** 2).sum(1)) / 256 * rng.uniform(1, 1.3, a.size)).astype(np.int64) + 1
    return gen.csr_from_edges(side * side, a, b, w, coords=xy.astype(np.int32))


@pytest.mark.parametrize("side,algo,few,many", [(400, "bidastar", 4, 16), (400, "astar", 0, 1), (400, "bids", 0, 1),
                                                (640, "bidastar", 24, 72), (640, "astar", 16, 40), (700, "bids", 1, 4)])
def test_few_queries_on_many_arcs(P, side, algo, few, many):
    """The arcs of a round decide from how many queries on a unit each does more than the whole chip on all of them."""
    g = _neighbours(side, side)
    pairs = gen.pairs_uniform(g.n, many, seed=50)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs[:4])
    G = _open(P, g, reorder=True)
    for k, resident in ((few, False), (many, True)):
        if k:
            d = G.batch_query(pairs[:k], algo=algo)
            launches = G.stats()["relax_launches"]
            assert launches == 1 if resident else launches % 16 == 0, (k, launches)
            assert np.array_equal(d[:4], exp[:k])
            G.set_option("resident", 0)
            assert np.array_equal(G.batch_query(pairs[:k], algo=algo), d)
            G.set_option("resident", 1)


def test_wide_steps_go_in_rounds(P):
    """The step decides too: a wide one has rounds of many arcs and a large frontier, a narrow one small rounds."""
    g = _neighbours(640, 51)
    pairs = gen.pairs_uniform(g.n, 4, seed=52)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = _open(P, g, reorder=True)
    d = G.get_option("default_delta")
    for algo, mode, delta, resident in (("bids", 2, 0, True), ("bids", 2, 64 * d, False), ("bids", 3, 0, False),
                                        ("sssp", 2, 4 * d, True), ("sssp", 2, 256 * d, False),
                                        ("bidastar", 2, d, False), ("bidastar", 2, d // 8, True)):
        G.set_option("theta_mode", mode)
        assert np.array_equal(G.batch_query(pairs, algo=algo, delta=delta), exp), (algo, mode, delta)
        launches = G.stats()["relax_launches"]
        assert launches == 1 if resident else launches % 16 == 0, (algo, mode, delta, launches)
