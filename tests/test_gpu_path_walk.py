"""The path walks (a wave per half) where they can go wrong: walks around the
64 vertices that a wave writes at once and beyond the room kept for them,
rows of more arcs than lanes, directed graphs. The paths are checked arc by arc."""
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


def _check(P, g, pairs, algos, resident=(0, 1)):
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    for algo in algos:
        for r in resident:
            print("paths", g.n, algo, len(pairs), r, flush=True)
            G.set_option("resident", r)
            dist, (off, vtx) = G.batch_query(pairs, algo=algo, want_path=True)
            assert np.array_equal(dist, exp)
            for q in range(len(pairs)):
                if exp[q] == INF:
                    assert off[q] == off[q + 1]
                else:
                    assert oracle.check_path(g.n, g.row_ptr, g.col, g.w, vtx[off[q]:off[q + 1]], int(pairs[q, 0]),
                                             int(pairs[q, 1]), int(exp[q])) == (0, 0), (algo, q)


def test_walk_lengths(P):
    """On a path graph, halves of 1 to 257 vertices."""
    g = gen.grid(1, 600, 1, 1000, seed=1)
    ends = [1, 2, 62, 63, 64, 65, 66, 126, 127, 128, 129, 130, 255, 256, 257, 512]
    _check(P, g, np.array([[20, 20 + e] for e in ends] + [[560, 560 - e] for e in ends], np.uint32), ["bids", "et"])


def test_walks_beyond_their_room(P):
    """2,000 queries leave 2,097 vertices to a walk: those of up to 3,999 are walked twice."""
    g = gen.grid(1, 4000, 1, 1000, seed=2)
    pairs = gen.pairs_uniform(g.n, 1998, seed=3)
    _check(P, g, np.concatenate([pairs, [[0, 3999], [3999, 0]]]).astype(np.uint32), ["et", "bids"], resident=(1,))


@pytest.mark.parametrize("deg", [63, 64, 65, 129, 1000])
def test_rows_wider_than_a_wave(P, deg):
    """Hubs in a chain, the way on at the end of a row of `deg` arcs."""
    k = 20
    hub = np.arange(k)
    leaf = k + np.arange(k * (deg - 2))
    src = np.concatenate([np.repeat(hub, deg - 2), hub[:-1], [k]])
    dst = np.concatenate([leaf, hub[1:], [k + k * (deg - 2)]])
    n = k + k * (deg - 2) + 1
    perm = n - 1 - np.arange(n)            # chain neighbours get the largest ids: last in their rows
    g = gen.csr_from_edges(n, perm[src], perm[dst], np.random.default_rng(deg).integers(1, 9, src.size))
    pairs = np.concatenate([gen.pairs_uniform(n, 20, seed=deg), [[n - 1, 0], [n - 1, n - k]]]).astype(np.uint32)
    _check(P, g, pairs, ["bids", "et"])
