"""Builds tests/host_rules.cpp (the library's host-side rules, which are plain C++ headers) and loads it."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_19442_amd", "csrc")


@functools.lru_cache(maxsize=None)
def lib() -> C.CDLL:
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "host_rules.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                        os.path.join(HERE, "host_rules.cpp"), "-o", out], check=True)
        L = C.CDLL(out)
    L.static_table_entries.restype = C.c_longlong
    L.m_tiles.restype = L.m_tiles_plain.restype = C.c_double
    L.m_tiles.argtypes = L.m_tiles_plain.argtypes = [C.c_double, C.c_int]
    i, q = C.c_int, C.c_longlong
    L.tile_grouped.argtypes = [i, q, i, i, i, i, i, q, q, i]
    return L
