"""No GPU: the rules by which the host sizes workspaces and picks tiles and grids."""
import ctypes as C
import itertools
import random
import time

import pytest

from host_rules import gemm_tile, kn_tile, lib, tile_name


def _play(entries, fails):
    n = len(entries)
    rc, has, leaked = (C.c_int * n)(), (C.c_int * n)(), C.c_int()
    room, base = (C.c_longlong * n)(), (C.c_longlong * n)()
    lib().moe_reserve_play(n, (C.c_longlong * n)(*entries), len(fails), (C.c_int * len(fails))(*fails), rc, has, room, base, C.byref(leaked))
    return list(rc), list(has), list(room), list(base), leaked.value


@pytest.mark.parametrize("entries", [(1040,), (70000, 1040), (40000, 90000, 1040, 50000), (1040, 70000, 32760, 32761)])
def test_a_table_holds_what_its_users_assume_whichever_allocation_fails(entries):
    """A MoE call checks the reserved size, and lists up to the fixed number of small tiles whatever was reserved: both have to
    fit into the table that is there, also behind a reservation that failed, which changes nothing."""
    fixed = lib().static_table_entries()
    for fails in itertools.product((0, 1), repeat=len(entries) + 1):
        rc, has, room, base, leaked = _play(entries, fails)
        asked = 0
        had = 0
        for i, e in enumerate(entries):
            if rc[i] == 0:
                asked = max(asked, e)
            assert base[i] == asked, (entries, fails, i)
            assert has[i] or not had                       # a table that was there is still there
            had = has[i]
            if has[i]:
                assert room[i] >= max(base[i], fixed), (entries, fails, i)
            else:
                assert base[i] == 0
        assert leaked == 0
        if not any(fails):
            assert all(r == 0 for r in rc)


@pytest.mark.parametrize("KC,rows,tile_rows,ld", [(1, 1, 64, 128), (1, 64, 64, 128), (5, 63, 64, 640), (7, 3, 64, 1024), (12, 128, 128, 1536), (31, 7, 128, 4000)])
def test_stages_past_the_end_of_k_load_nothing(KC, rows, tile_rows, ld):
    """The rings ask for up to eight stages past the last one (gemm_ks.h): none of those loads may reach memory, however the bounds
    check treats the scalar offset, and those of the real stages read the rows that are there."""
    assert lib().ks_stage_bad_accesses(KC, 64, rows, tile_rows, C.c_uint(ld)) == 0


@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 64])
def test_a_waiting_reducer_leaves_room_for_a_gemm_that_comes_later(W):
    """Registers of a SIMD lane: 512.  A reducer workgroup takes 64 at most, a large GEMM tile's 448, a K-split tile's up to 384 (two waves of 192;
    all but the 128x128 tile of a [K][N] operand up to 288).  However many blocks there are, half of the CUs have to keep room for a large
    tile and all for a K-split one.  Three reducers at once (three ranks of four on one GPU) have to leave every CU room for a K-split tile of 288, beside
    what an even spread puts on it; in worlds without an unrolled kernel for one of 192."""
    cus = 256
    for n_vec4 in (1, 1000, 256 * 256, 256 * 512, 1 << 18, 1 << 21, 1 << 25, 1 << 27):
        grid = lib().reduce_grid(W, cus, C.c_longlong(n_vec4), 0)
        assert 1 <= grid <= -(-n_vec4 // lib().reduce_threads(W, cus, C.c_longlong(n_vec4), 0))
        per_cu = [grid // cus + (i < grid % cus) for i in range(cus)]
        assert sum(512 - 64 * k >= 448 for k in per_cu) >= cus // 2, (W, n_vec4, grid)
        assert all(512 - 64 * k >= 384 for k in per_cu), (W, n_vec4, grid)
        spread = [3 * grid // cus + (i < 3 * grid % cus) for i in range(cus)]
        assert all(512 - 64 * k >= (288 if W in (2, 3, 4, 8) and n_vec4 < 1 << 27 else 192) for k in spread), (W, n_vec4, grid)
        assert lib().reduce_grid(W, cus, C.c_longlong(n_vec4), 1) <= cus


@pytest.mark.parametrize("W", [2, 3, 4, 5, 8, 64])
def test_a_reducer_beside_a_gemm_takes_the_same_share_of_every_cu(W):
    # a persistent GEMM ends with its slowest CU
    for n_vec4 in (256 * 1024, 1 << 21, 1 << 27):
        assert lib().reduce_grid(W, 256, C.c_longlong(n_vec4), 1) == 256


# (call, shards, epoch, stream, the stream keeps order) in turn; of every GEMM, what it is told and how often the runtime is asked
@pytest.mark.parametrize("W,calls,want", [
    (4, [("copy", 0b1111, 5, 1, 1), ("gemm", 0, 5, 1, 1)], [(1, 1)]),
    (4, [("copy", 0b0101, 5, 0, 1), ("copy", 0b1010, 5, 0, 1), ("gemm", 0, 5, 0, 1), ("gemm", 0, 5, 0, 1)], [(1, 1), (1, 1)]),
    (64, [("copy", (1 << 64) - 1, 5, 1, 1), ("gemm", 0, 5, 1, 1)], [(1, 1)]),
    (4, [("copy", 0b1111, 5, 1, 1), ("gemm", 0, 5, 2, 1)], [(0, 0)]),                                                  # copy and GEMM beside each other
    (4, [("copy", 0b0111, 5, 1, 1), ("gemm", 0, 5, 1, 1)], [(0, 0)]),                                                  # a shard is missing
    (4, [("copy", 0b0011, 5, 2, 1), ("copy", 0b1100, 5, 1, 1), ("gemm", 0, 5, 1, 1), ("gemm", 0, 5, 2, 1)], [(0, 0), (0, 0)]),
    (4, [("copy", 0b1111, 5, 1, 1), ("gemm", 0, 6, 1, 1)], [(0, 0)]),                                                  # of the epoch before
    (4, [("copy", 0b0011, 5, 1, 1), ("copy", 0b1100, 6, 1, 1), ("gemm", 0, 6, 1, 1)], [(0, 0)]),
    (4, [("copy", 0b1111, 5, 1, 0), ("gemm", 0, 5, 1, 1)], [(0, 0)]),                                                  # the copy was captured, ...
    (4, [("copy", 0b0011, 5, 1, 1), ("copy", 0b1100, 5, 1, 0), ("gemm", 0, 5, 1, 1)], [(0, 0)]),                       # ... a part of it, ...
    (4, [("copy", 0b1111, 5, 1, 1), ("gemm", 0, 5, 1, 0)], [(0, 1)]),                                                  # ... the GEMM is
])
def test_a_gemm_is_behind_the_copies_of_its_own_epoch_and_stream_only(W, calls, want):
    n = len(calls)
    ints = lambda k: (C.c_int * n)(*[c[k] for c in calls])
    answer, asked = (C.c_int * n)(), (C.c_int * n)()
    lib().delivered_play(W, n, (C.c_int * n)(*[int(c[0] == "gemm") for c in calls]), (C.c_ulonglong * n)(*[c[1] for c in calls]), ints(2),
                         (C.c_longlong * n)(*[c[3] for c in calls]), ints(4), answer, asked)
    assert [(answer[i], asked[i]) for i in range(n) if calls[i][0] == "gemm"] == want


def test_expected_number_of_tiles_is_the_sum_and_costs_no_more_for_long_segments():
    rng = random.Random(31)
    for bm in (16, 32, 64, 128, 256):
        for mean in [0.01, 0.5, 1.0, 15.9, 16.0, 256.0, 1e5, 1e6] + [10.0 ** rng.uniform(-2, 6) for _ in range(200)]:
            assert lib().m_tiles(mean, bm) == lib().m_tiles_plain(mean, bm), (mean, bm)
    # a MoE call makes this choice on the host: 16 Mi rows of one expert, 1000 calls (1.4 s if every tile is a term of the sum)
    t0 = time.monotonic()
    for _ in range(1000):
        assert 0 <= lib().tile_grouped(256, 1 << 24, 1, 128, 64, 0, 1, 1 << 24, 1 << 28, 0) < 8
    assert time.monotonic() - t0 < 0.8


@pytest.mark.parametrize("gathered,f32", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_the_order_of_the_sums_does_not_depend_on_what_was_reserved(gathered, f32):
    """All numbered tiles give the same bits and so does each K-split tile: whichever of them a call takes may depend on the problem
    only, not on whether its context was reserved for a larger one."""
    rng = random.Random(32)
    for _ in range(4000):
        P, E = int(10.0 ** rng.uniform(0, 5)), rng.randint(1, 128)
        N, K = rng.randint(1, 4096), 64 * rng.randint(1, 64)
        taken = set()
        for room in (0, 1, 500, 5000, 32760, 1 << 28):
            tile = lib().tile_grouped(256, P, E, N, K, gathered, f32, P, room, 0)
            taken.add(tile if tile >= 8 else "numbered")
        assert len(taken) == 1, (P, E, N, K, taken)


# Measured, us per call with routing, weights in no cache where they exceed it: the tile that a sum of fixed costs had picked, and the
# one that was taken before there were K-split tiles (128x128 in all of these).
@pytest.mark.parametrize("gathered,f32,tokens,topk,E,N,K,slow", [
    (1, 0, 578, 4, 5, 824, 3392, "64x64"),          # 49.7 against 33.4
    (1, 1, 752, 2, 60, 805, 3328, "16x64"),         # 107.9 against 78.5 (64x128: 72.7)
    (1, 1, 40, 2, 33, 681, 640, "16x64"),           # 19.7 against 16.6
    (1, 1, 5168, 2, 6, 160, 1920, "64x64"),         # 33.7 against 29.1
    (1, 0, 5056, 4, 6, 182, 2944, "64x64"),         # 79.7 against 66.3 (256x224: 62.3)
    (1, 1, 848, 2, 16, 900, 256, "64x64"),          # 19.8 against 17.0
    (0, 1, 40, 2, 62, 1856, 832, "16x64"),          # 55.9 against 49.4
    (0, 1, 344, 1, 52, 1756, 896, "16x64"),         # 59.2 against 54.2
    (0, 1, 96, 2, 48, 508, 768, "16x64"),           # 28.3 against 25.9
])
def test_moe_calls_do_not_take_a_tile_that_was_measured_slower_than_the_old_choice(gathered, f32, tokens, topk, E, N, K, slow):
    P = tokens * topk
    assert tile_name(lib().tile_grouped(256, P, E, N, K, gathered, f32, P, 1 << 28, 0)) != slow


# The same for GEMM + ReduceScatter, us per call with the reducer, every row wanted.
@pytest.mark.parametrize("M,N,K,slow", [
    (8, 3300, 128, "16x16"),                        # 12.7 against 10.5
    (12, 3472, 128, "16x16"),                       # 13.1 against 10.4
    (16, 7948, 320, "16x32"),                       # 14.6 against 12.9
    (8, 6972, 320, "16x32"),                        # 13.2 against 11.8
    (8, 4620, 128, "16x32"),                        # 12.2 against 11.6
])
def test_gemm_rs_does_not_take_a_tile_that_was_measured_slower_than_the_old_choice(M, N, K, slow):
    assert gemm_tile(256, M, N, K, slices=True)[0] != slow


def test_gemm_rs_with_fp32_stores_between_rounds_keeps_the_smaller_tile():
    # 4232 x 4060 x 2368 on 256x224 173.8 us, on 128x128 148.0; 4288 x 3852 x 2816 185.5 and 162.8
    for M, N, K in ((4232, 4060, 2368), (4288, 3852, 2816)):
        assert lib().tile_plain(256, M, N, K, 1) == 5
    assert lib().tile_plain(256, 8192, 8192, 3584, 1) == 6


def test_an_operand_is_read_in_place_only_where_the_order_of_the_numbered_tiles_does_not_count():
    rng = random.Random(65)
    several = 0
    for _ in range(20000):
        M, N, K = rng.randint(1, 8192), 8 * rng.randint(1, 896), 64 * rng.randint(1, 128)
        for slices in (False, True):
            tile, tiles = gemm_tile(256, M, N, K, slices)
            if tile == "numbered" and tiles > 256:
                several += 1
                assert kn_tile(256, M, N, K, slices) is None
    assert several > 1000


# Rows in place, us per call with the top-k reduction and the reducer: the tile of gemm_pipe.h that the costs name, and the numbered one.
@pytest.mark.parametrize("tokens,topk,E,N,K,tile", [
    (1064, 2, 25, 1308, 192, "numbered"),           # one round: 32.6 and 29.2
    (1552, 2, 62, 776, 256, "numbered"),            # 35.0 and 31.9
    (548, 4, 18, 1588, 256, "numbered"),            # 36.2 and 33.1
    (714, 1, 33, 1560, 576, "numbered"),            # 35.2 and 32.5
    (7896, 4, 9, 576, 512, "192x192"),              # several: 71.4 and 84.5
    (4392, 4, 28, 868, 256, "320x128"),             # 64.0 and 71.4
])
def test_rows_in_place_take_a_streaming_tile_for_several_rounds_only(tokens, topk, E, N, K, tile):
    P = tokens * topk
    assert tile_name(lib().tile_grouped(256, P, E, N, K, 0, 1, P, 1 << 28, 0)) == tile
