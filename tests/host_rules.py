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


def tile_name(tile: int) -> str:
    """"16x32" for a K-split tile, "numbered" for those of agg_set_tile_config."""
    if tile < 8:
        return "numbered"
    rc = lib().tile_rows_and_columns(tile)
    return f"{rc >> 16}x{rc & 0xffff}"


def gemm_tile(num_cus: int, M: int, N: int, K: int, slices: bool = False):
    """The automatic choice for ag_gemm, or for gemm_rs and gemm_rs_scatter (slices), and how many of those tiles the problem has."""
    tile = lib().tile_plain(num_cus, M, N, K, int(slices))
    rc = lib().tile_rows_and_columns(tile)
    return tile_name(tile), -(-M // (rc >> 16)) * -(-N // (rc & 0xffff))


def kn_tile(num_cus: int, M: int, N: int, K: int, slices: bool = False):
    """The tile that reads a [K][N] operand in place, or None where it is transposed."""
    tile = lib().tile_of_kn(num_cus, M, N, K, int(slices))
    return None if tile < 0 else tile_name(tile)


def moe_tile(num_cus: int, tokens: int, topk: int, E: int, N: int, K: int, gathered: bool, f32: bool) -> str:
    """The automatic choice for ag_moe_gemm (gathered) and moe_rs on a context reserved for the problem."""
    return tile_name(lib().tile_grouped(num_cus, tokens * topk, E, N, K, int(gathered), int(f32), tokens * topk, 1 << 28, 0))


def _ks_tiles(grouped: int):
    out = (C.c_int * 16)()
    return list(out[:lib().ks_tiles(grouped, out)])


def dense_ks_tiles():
    return _ks_tiles(0)


def moe_ks_tiles():
    return _ks_tiles(1)
