"""The tuning cache across versions of the library: an entry written by an
older one, whose launch shape keeps a road graph from resident searches, is
not loaded."""
import re

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


def test_older_entries_are_tuned_again(tmp_path):
    import paper_2506_16488_amd as P
    g = gen.lattice(64, 0.05, seed=3)
    pairs = gen.pairs_uniform(g.n, 24, seed=4)
    exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
    cache = tmp_path / "tune.txt"
    G = P.Graph.from_host(g)
    G.set_option("timeout_ms", 60000)
    assert G.tune(pairs, algo="bids", cache_path=str(cache))["from_cache"] == 0
    line = cache.read_text()
    key, val = re.match(r"(ppsp-tune-v\d+ \w+ \d+ \d+) (.*)", line).groups()
    val = val.split()
    val[2] = "3072"                                     # a grid that the version before could choose
    cache.write_text(re.sub(r"-v\d+ ", "-v5 ", key) + " " + " ".join(val) + "\n")
    H = P.Graph.from_host(g)
    H.set_option("timeout_ms", 60000)
    assert H.tune(pairs, algo="bids", cache_path=str(cache))["from_cache"] == 0
    assert np.array_equal(H.batch_query(pairs, algo="bids", sched="autotuned"), exp)
    # what this version writes is loaded
    K = P.Graph.from_host(g)
    assert K.tune(pairs, algo="bids", cache_path=str(cache))["from_cache"] == 1
