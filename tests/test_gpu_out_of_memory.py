"""Device memory that does not hold the larger buffers of a faster way: the
call answers the slower way. A small library in front of hipMalloc (in a
process of its own, loaded before the search library) refuses sizes in a range,
or whatever goes beyond a total."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <stddef.h>
static int (*real_malloc)(void **, size_t);
static int (*real_free)(void *);
static size_t lo = ~(size_t)0, hi = ~(size_t)0, most = ~(size_t)0, live, refused;
static struct { void *p; size_t n; } held[4096];
void shim_real(void *m, void *f) { real_malloc = m; real_free = f; }
void shim_range(size_t a, size_t b) { lo = a; hi = b; }
void shim_most(size_t extra) { most = extra == ~(size_t)0 ? extra : live + extra; }
size_t shim_refused(void) { return refused; }
int hipMalloc(void **p, size_t n) {
    if ((n >= lo && n < hi) || (most != ~(size_t)0 && live + n > most)) { refused++; return 2; }
    int rc = real_malloc(p, n);
    if (rc == 0) {
        live += n;
        for (int i = 0; i < 4096; i++) if (!held[i].p) { held[i].p = *p; held[i].n = n; break; }
    }
    return rc;
}
int hipFree(void *p) {
    for (int i = 0; p && i < 4096; i++) if (held[i].p == p) { live -= held[i].n; held[i].p = 0; break; }
    return real_free(p);
}
"""

PRELUDE = r"""
import ctypes, os, sys
import numpy as np
import torch
assert torch.cuda.is_available()
torch.cuda.init()
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
path = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
assert len(path) == 1, path
hip = ctypes.CDLL(path.pop())
shim.shim_real(ctypes.cast(hip.hipMalloc, ctypes.c_void_p), ctypes.cast(hip.hipFree, ctypes.c_void_p))
shim.shim_refused.restype = ctypes.c_size_t
def refuse(a, b=1 << 62): shim.shim_range(ctypes.c_size_t(a), ctypes.c_size_t(b))
def most(extra): shim.shim_most(ctypes.c_size_t(extra))
def refused(): return int(shim.shim_refused())
import gen, oracle
import paper_2506_16488_amd as P
"""


def _run(tmp_path, body):
    c, so, py = tmp_path / "shim.c", tmp_path / "libshim.so", tmp_path / "case.py"
    c.write_text(SHIM)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", str(c), "-o", str(so)])
    py.write_text(PRELUDE + body + "\nprint('case done', flush=True)\n")
    r = subprocess.run([sys.executable, str(py), str(so)], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, PYTHONPATH=os.pathsep.join(
                           [ROOT] + os.environ.get("PYTHONPATH", "").split(os.pathsep)).rstrip(os.pathsep)))
    assert r.returncode == 0 and "case done" in r.stdout, r.stdout[-1000:] + r.stderr[-2000:]


HUBS = r"""
g = gen.rmat(16, 16, seed=5)
pairs = np.random.default_rng(6).permutation(g.n)[:256].reshape(-1, 2).astype(np.uint32)
exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
deg = np.diff(g.row_ptr.astype(np.int64))
room = 256 * int(((deg[deg > 16] + 2047) // 2048).sum())      # records of every hub of 256 searches
assert deg.max() > 512 and room > 1 << 21
G = P.Graph.from_host(g)
G.set_option("timeout_ms", 60000)
G.set_option("list_deg", 16)
G.set_option("queue_cap", 1 << 21)
state = 256 * g.n * 8
"""


def test_hub_bins_fall_back_to_one_list(tmp_path):
    _run(tmp_path, HUBS + r"""
refuse(room * 32, room * 32 + 1)
for _ in range(2):
    assert np.array_equal(G.batch_query(pairs, algo="bids"), exp)
    assert G.get_option("heavy_cap") < room and refused()
refuse(1 << 62)
assert np.array_equal(G.batch_query(pairs, algo="bids"), exp) and G.get_option("heavy_cap") >= room
""")


def test_hub_bins_keep_within_the_budget(tmp_path):
    _run(tmp_path, HUBS + r"""
G.set_option("mem_budget_mb", (state >> 20) + 8)
assert np.array_equal(G.batch_query(pairs, algo="bids"), exp)
assert G.get_option("heavy_cap") < room and G.stats()["waves"] == 1
""")


ROADS = r"""
g = gen.grid(64, 64, 1, 1000, seed=7)
pairs = np.random.default_rng(8).permutation(g.n)[:128].reshape(-1, 2).astype(np.uint32)
exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
G = P.Graph.from_host(g)
G.set_option("timeout_ms", 60000)
spill = 64 * 4 * 4096 * 16                                    # four areas of 4,096 entries a query
"""


def test_resident_falls_back_to_rounds(tmp_path):
    _run(tmp_path, ROADS + r"""
refuse(spill)
for algo in ("bids", "et"):
    assert np.array_equal(G.batch_query(pairs, algo=algo), exp) and G.stats()["relax_launches"] > 1
refuse(1 << 62)
assert np.array_equal(G.batch_query(pairs, algo="bids"), exp) and G.stats()["relax_launches"] == 1
""")


def test_rounds_take_back_the_spill_area(tmp_path):
    _run(tmp_path, ROADS + r"""
assert np.array_equal(G.batch_query(pairs, algo="bids"), exp) and G.stats()["relax_launches"] == 1
most(spill // 2)              # rounds need more than that, and less than the spill area
G.set_option("resident", 0)
G.set_option("queue_cap", 300000)
for _ in range(2):
    assert np.array_equal(G.batch_query(pairs, algo="bids"), exp)
""")


def test_paths_without_room_for_the_walks(tmp_path):
    """No room to keep the walks as they are found: each is walked again into its place."""
    _run(tmp_path, r"""
g = gen.lattice(64, 0.1, seed=9)
pairs = np.random.default_rng(10).permutation(g.n)[:96].reshape(-1, 2).astype(np.uint32)
exp = oracle.pp_batch(g.n, g.row_ptr, g.col, g.w, pairs)
G = P.Graph.from_host(g)
G.set_option("timeout_ms", 60000)
for resident in (0, 1):
    G.set_option("resident", resident)
    assert np.array_equal(G.batch_query(pairs, algo="bids"), exp)
    walks = 48 * 2 * g.n * 4
    refuse(walks, walks + 1)
    for algo in ("bids", "et"):
        before = refused()
        dist, (off, vtx) = G.batch_query(pairs, algo=algo, want_path=True)
        assert refused() > before and np.array_equal(dist, exp)
        for q in range(48):
            assert oracle.check_path(g.n, g.row_ptr, g.col, g.w, vtx[off[q]:off[q + 1]], int(pairs[q, 0]),
                                     int(pairs[q, 1]), int(exp[q])) == (0, 0), q
    refuse(1 << 62)
""")
