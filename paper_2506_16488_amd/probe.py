"""The benchmark's scattered-access probe and the integer root's
(libppsp_probe.so).

Measurement and test tooling, outside the search library and its C interface:
the round kernel is bound by scattered 8-16 byte accesses to the search state,
and randbench measures the device's rate for exactly those accesses, so the
benchmark can price a launch against it; isqrt32 runs the device branch of the
heuristic's square root. The search path never loads it.
"""
from __future__ import annotations

import ctypes
import os

HERE = os.path.dirname(os.path.abspath(__file__))
SO_PATH = os.path.join(HERE, "libppsp_probe.so")
_lib = None


def _load():
    global _lib
    if _lib is None:
        if not os.path.exists(SO_PATH):
            raise ImportError("libppsp_probe.so is not built (run __graft_entry__.build())")
        import torch  # noqa: F401  (bind to torch's HIP runtime, as the search library does)
        _lib = ctypes.CDLL(SO_PATH)
        _lib.probe_randbench.argtypes = [ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int,
                                         ctypes.POINTER(ctypes.c_double)]
        _lib.probe_randbench.restype = ctypes.c_int
        _lib.probe_isqrt32.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_uint64, ctypes.c_void_p]
        _lib.probe_isqrt32.restype = ctypes.c_int
    return _lib


def randbench(words, accesses, kind, device=0) -> float:
    """Kernel milliseconds (second of two runs) for `accesses` scattered
    16-byte loads (kind 0) or 64-bit atomicMin (kind 1) over a fresh table of
    `words` 64-bit words. Raises ValueError on bad arguments, RuntimeError on
    a device failure."""
    ms = ctypes.c_double(0)
    rc = _load().probe_randbench(device, int(words), int(accesses), int(kind), ctypes.byref(ms))
    if rc == -1:
        raise ValueError("probe_randbench: bad arguments")
    if rc != 0:
        raise RuntimeError("probe_randbench failed (%d)" % rc)
    return ms.value


def isqrt32(q, device=0):
    """The device's integer square roots of q (uint64 array, below 2^63) as a uint32 array."""
    import numpy as np
    q = np.ascontiguousarray(q, np.uint64)
    out = np.empty(q.size, np.uint32)
    rc = _load().probe_isqrt32(device, q.ctypes.data, q.size, out.ctypes.data)
    if rc == -1:
        raise ValueError("probe_isqrt32: bad arguments")
    if rc != 0:
        raise RuntimeError("probe_isqrt32 failed (%d)" % rc)
    return out
