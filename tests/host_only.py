"""The host library built with other limits, in place of the product's for a test's plans."""

import contextlib
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2211_05322_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2211_05322_amd", "csrc")
SOURCES = [os.path.join(CSRC, f) for f in ("planner.cpp", "capi.cpp", "schedule.cpp", "pipeline.cpp")]
SOURCES.append(os.path.join(ROOT, "tests", "c", "host_only.cpp"))


def build(out, **limits):
    """limits: planner macros, e.g. RS_MAX_DESCS=1024."""
    cmd = ["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
           *[f"-D{k}=uint64_t({v})" for k, v in limits.items()], *SOURCES, "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    lib = B.load(str(out))
    lib.test_blocked_chunks.argtypes = lib.test_sets_in_turn.argtypes = [ctypes.c_void_p]
    lib.test_cached_limit.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    lib.test_slots_of_parts.argtypes = [ctypes.c_void_p]
    lib.test_transpose_plain.argtypes = [ctypes.c_void_p]
    lib.test_transpose_launch_lds.argtypes = [ctypes.c_void_p, ctypes.c_uint32]
    lib.test_blocked_chunks.restype = lib.test_cached_limit.restype = ctypes.c_int64
    return lib


@functools.lru_cache(maxsize=None)
def plain():
    """The product's host code and limits."""
    with tempfile.TemporaryDirectory(prefix="reshard_host_") as d:
        return build(os.path.join(d, "host.so"))  # stays mapped


@contextlib.contextmanager
def using(lib):
    """Plans made (and dropped) inside use `lib`."""
    product = B.load()
    B._lib = lib
    try:
        yield lib
    finally:
        B._lib = product
