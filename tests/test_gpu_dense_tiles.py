"""Dense bitmaps are read in tiles of runs from all over them: sizes around a
word, a run (512 vertices), two runs, a tile (2,048) and several, with one and
with many dense searches, against the oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [31, 32, 33, 1023, 1025, 2047, 2048, 2049, 4095, 4097, 6145, 10240])
def test_dense_tiles(n):
    import paper_2506_16488_amd as P
    rng = np.random.default_rng(n)
    m = 6 * n
    g = gen.csr_from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(1, 200, m))
    pairs = gen.pairs_uniform(n, 70, seed=n)
    pairs = np.concatenate([pairs, [[0, n - 1], [n - 1, n // 2]]]).astype(np.uint32)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    G.set_option("dense_force", 1)
    for k in (1, 72):
        for algo in ("bids", "et"):
            print("dense tiles", n, k, algo, flush=True)
            assert np.array_equal(G.batch_query(pairs[-k:], algo=algo, delta=100), exp[-k:]), (k, algo)


@pytest.mark.parametrize("grid", [1, 2, 3, 5])
@pytest.mark.parametrize("n", [4097, 6145, 10240, 16385])
def test_dense_tiles_on_a_small_grid(n, grid):
    """A bitmap of at least as many tiles as the grid has workgroups is read in tiles on end."""
    import paper_2506_16488_amd as P
    rng = np.random.default_rng(n)
    m = 6 * n
    g = gen.csr_from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(1, 200, m))
    pairs = gen.pairs_uniform(n, 12, seed=n + grid)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    G.set_option("dense_force", 1)
    G.set_option("grid_blocks", grid)
    for k in (1, 12):
        for algo in ("bids", "et"):
            print("dense tiles", n, grid, k, algo, flush=True)
            assert np.array_equal(G.batch_query(pairs[-k:], algo=algo, delta=100), exp[-k:]), (k, algo)
