"""The integer square root under every heuristic, as the device computes it
(from a single-precision estimate): r^2 <= q < (r + 1)^2 for small values,
around squares of every size, and all over the range that graph creation
admits (below 2^63). Whole numbers: equality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _squares(lo, hi, count, rng):
    """r^2 - 2 .. r^2 + 2r + 1 at both ends for roots r spread over their logarithm."""
    r = np.exp(rng.uniform(np.log(lo), np.log(hi), count)).astype(np.uint64)
    one = np.uint64(1)
    s = r * r
    return np.concatenate([s - np.uint64(2), s - one, s, s + one, s + r, s + r + r - one, s + r + r, s + r + r + one])


def test_device_root_is_exact():
    from paper_2506_16488_amd import probe
    rng = np.random.default_rng(1)
    top = 3037000499                                  # floor(sqrt(2^63 - 1))
    q = np.concatenate([
        np.arange(1 << 22, dtype=np.uint64),
        _squares(2, top, 1 << 20, rng),
        _squares(1 << 20, top, 1 << 20, rng),
        _squares(1 << 31, top, 1 << 20, rng),
        np.exp2(rng.uniform(0, 63, 1 << 22)).astype(np.uint64),
        rng.integers(0, 1 << 63, 1 << 22, dtype=np.uint64),
        (np.uint64(1) << np.arange(63, dtype=np.uint64)), (np.uint64(1) << np.arange(1, 64, dtype=np.uint64)) - np.uint64(1),
    ])
    q = q[q < np.uint64(1 << 63)]
    r = probe.isqrt32(q).astype(np.uint64)
    low, high = r * r <= q, q < (r + np.uint64(1)) * (r + np.uint64(1))
    bad = np.nonzero(~(low & high))[0]
    assert bad.size == 0, [(int(q[i]), int(r[i])) for i in bad[:5]]
