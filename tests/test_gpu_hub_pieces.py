"""The hub-list kernel's pieces of records: lists from one record to more than
the grid takes in parts, hubs of every length around a part, a chunk and their
multiples, directed graphs and dense frontiers, against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2506_16488_amd as P
    P.lib()
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return P


def _hubs(seed):
    """Hubs of 513 to 8,193 leaves (parts are 128 to 2,048 arcs) in a chain, the leaves shared between neighbours."""
    rng = np.random.default_rng(seed)
    degs = [513, 514, 639, 640, 641, 767, 768, 769, 1023, 1024, 1025, 2047, 2048, 2049, 2175, 2176, 2177, 4095, 4096,
            4097, 6143, 6145, 8191, 8192, 8193]
    leaves, k = 20000, len(degs)
    src = [np.arange(k - 1)]
    dst = [np.arange(1, k)]
    for h, d in enumerate(degs):
        src.append(np.full(d, h))
        dst.append(k + rng.choice(leaves, d, replace=False))
    src, dst = np.concatenate(src), np.concatenate(dst)
    return gen.csr_from_edges(k + leaves, src, dst, rng.integers(1, 1000, src.size))


@pytest.mark.parametrize("waves", [1, 24, 32])
@pytest.mark.parametrize("symmetric", [True, False])
def test_hub_pieces(P, symmetric, waves):
    g = _hubs(1)
    if not symmetric:
        g.w = (g.w + np.random.default_rng(2).integers(0, 50, g.w.size)).astype(np.uint32)
        g.symmetric = False
    pairs = gen.pairs_uniform(g.n, 600, seed=3)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    G.set_option("heavy_waves", waves)
    G.set_option("heavy_window", 1)
    for k in (1, 40, 600):          # few records (16 parts each) to several thousand a round
        for algo in ("bids", "et", "sssp"):
            print("hub pieces", symmetric, waves, k, algo, flush=True)
            assert np.array_equal(G.batch_query(pairs[:k], algo=algo), exp[:k]), (k, algo)
    assert G.stats()["heavy_arcs"] > 0
    if symmetric:
        G.set_option("dense_min", 64)
        assert np.array_equal(G.batch_query(pairs, algo="bids", delta=3000), exp)


@pytest.mark.parametrize("k", [15, 16, 17, 100, 300])
def test_hub_bins(P, k):
    """The hub list in bins by pair: below and above 16 pairs, more pairs than bins, with few and
    with many waves, whole records claimed and pieces dealt out."""
    g = _hubs(5)
    pairs = gen.pairs_uniform(g.n, k, seed=k)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    for window in (1, 64):
        G.set_option("heavy_window", window)
        for waves, claim in ((24, 4), (1, 1), (0, 64)):
            G.set_option("heavy_waves", waves)
            G.set_option("heavy_claim", claim)
            for algo in ("bids", "et"):
                print("hub bins", k, window, waves, algo, flush=True)
                assert np.array_equal(G.batch_query(pairs, algo=algo), exp), (window, waves, algo)


@pytest.mark.parametrize("grid", [4, 8, 20, 100, 301])
def test_hub_bins_any_grid(P, grid):
    """Grids of the hub-list kernel that the chip's 8 dies do not share evenly, and one that leaves dies empty."""
    g = _hubs(6)
    pairs = gen.pairs_uniform(g.n, 40, seed=60)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    G.set_option("heavy_waves", 0)
    G.set_option("grid_blocks", grid)
    for window in (1, 64):
        G.set_option("heavy_window", window)
        for algo in ("bids", "et", "sssp"):
            print("hub bins, grid", grid, window, algo, flush=True)
            assert np.array_equal(G.batch_query(pairs, algo=algo), exp), (window, algo)
    assert G.stats()["heavy_arcs"] > 0


def test_hub_bins_of_uneven_pairs(P):
    """24 pairs of searches in 16 bins: a bin of two pairs has room for all the hubs of both, so the wave runs once."""
    rng = np.random.default_rng(7)
    n, d = 40000, 30
    src = np.concatenate([np.repeat(np.arange(n), d), np.zeros(600, np.int64)])
    dst = np.concatenate([rng.integers(0, n, n * d), 1 + np.arange(600)])
    g = gen.csr_from_edges(n, src, dst, np.ones(src.size, np.uint32))
    pairs = rng.permutation(n)[:96].reshape(-1, 2).astype(np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    G.set_option("list_deg", 16)
    G.set_option("queue_cap", 1 << 23)
    G.set_option("heavy_window", 1)
    for _ in range(2):
        assert np.array_equal(G.batch_query(pairs, algo="sssp", delta=1 << 20), exp)
        assert G.stats()["retries"] == 0 and G.stats()["heavy_chunks"] > 0


@pytest.mark.parametrize("real", [1, 2, 5])
def test_hub_bins_of_few_pairs(P, real):
    """Most pairs end at once, so the list lies in the bins of a few dies, at changing places."""
    g = _hubs(9)
    n = g.n + 200
    rp = np.concatenate([g.row_ptr, np.full(200, g.row_ptr[-1], g.row_ptr.dtype)])
    idle = g.n + np.arange(200).reshape(-1, 2)
    G = P.Graph(n, rp, g.col, g.w, symmetric=True)
    G.set_option("timeout_ms", 60000)
    for k, at in ((16, 0), (16, 9), (40, 30), (100, 93)):
        pairs = idle[:k].copy()
        pairs[at:at + real] = gen.pairs_uniform(g.n, real, seed=70 + real)
        pairs = pairs.astype(np.uint32)
        exp = oracle.pp_batch(n, rp, g.col, g.w, pairs)
        for waves, grid in ((24, 0), (0, 20)):
            G.set_option("heavy_waves", waves)
            G.set_option("grid_blocks", grid)
            for algo in ("bids", "et"):
                assert np.array_equal(G.batch_query(pairs, algo=algo), exp), (k, at, waves, algo)
    assert G.stats()["heavy_arcs"] > 0
