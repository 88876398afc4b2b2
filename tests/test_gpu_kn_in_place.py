"""A B stored [K][N] that the GEMMs read in place: every tile that does, at the edges of tiles, rings and 16-byte chunks, rows longer than N
whose rest is NaN, nothing behind the last row's N, more tiles than workgroups, several signals; the same bits with and without the other
ranks' rows; and operands that do not qualify, which are transposed.  Integer inputs: sums of at most 4 x 6464 are exact in fp32 in any order."""
import numpy as np
import pytest
import torch

import host_rules
import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu


def _cus():
    return agg.agg_device_info()[0]


def _ints(g, *shape):
    return torch.randint(-2, 3, shape, device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)


def _kn(g, K, N, ldb, offset=0):
    """B [K, N] and the buffer that holds it: rows of ldb elements from `offset` on, NaN everywhere else, no element behind the last one."""
    B = _ints(g, K, N)
    flat = torch.full((offset + (K - 1) * ldb + N,), float("nan"), device="cuda", dtype=torch.bfloat16)
    flat[offset:].as_strided((K, N), (ldb, 1)).copy_(B)
    return B, flat


# tile (None: transposed), W, rows per rank, K, N, ldb, offset
CASES = [
    ("64x64", 2, 6, 64, 8, 8, 0),                # one chunk of a row, one stage
    ("64x64", 3, 21, 192, 72, 80, 0),            # one row less than a tile, a second column tile of one chunk, padded rows
    ("64x64", 2, 65, 704, 752, 752, 8),
    ("64x64", 2, 32, 2112, 1200, 1208, 0),
    ("64x128", 2, 469, 704, 1336, 1344, 0),
    ("64x128", 2, 669, 64, 1088, 1088, 16),
    ("64x128", 2, 422, 2112, 1160, 1160, 0),
    ("128x128", 2, 689, 704, 1496, 1496, 0),
    ("128x128", 2, 626, 64, 1568, 1576, 0),
    ("128x128", 2, 624, 2112, 1584, 1584, 0),
    ("128x128", 2, 1435, 192, 1832, 1840, 0),    # more tiles than workgroups
    (None, 2, 6, 64, 12, 16, 0),                 # columns that are no whole chunks
    (None, 2, 6, 64, 16, 20, 0),                 # rows that do not start on 16 bytes
    (None, 2, 6, 64, 16, 16, 1),                 # nor does the first one
    (None, 2, 9, 6464, 24, 24, 0),               # a long K on few tiles: transposing is faster
]


@pytest.mark.parametrize("tile,W,Ms,K,N,ldb,offset", CASES)
def test_ag_gemm_exact(tile, W, Ms, K, N, ldb, offset):
    M = W * Ms
    if tile or (N % 8 == 0 and ldb % 8 == 0 and offset % 8 == 0):
        assert host_rules.kn_tile(_cus(), M, N, K) == tile
    g = torch.Generator(device="cuda").manual_seed(51)
    cps = 3 if Ms % 3 == 0 else 1
    shards, (B, flat) = [_ints(g, Ms, K) for _ in range(W)], _kn(g, K, N, ldb, offset)
    want = torch.cat(shards).float() @ B.float()
    ctx = agg.symm_alloc(W, W - 1, Ms * K * 2, W * cps)
    try:
        ps, cs = ctx.streams()
        C = torch.empty((M, N), device="cuda")
        agg.signal_reset(ctx)
        with pytest.raises(agg.AggError) as e:   # the buffer of a transposed copy has to be there either way
            agg.ag_gemm(ctx, M, N, K, flat.data_ptr() + 2 * offset, ldb, agg.B_KN, C, N, agg.F32, cs)
        assert e.value.code == agg.ERR_NOT_RESERVED
        agg.agg_reserve_b_kn(ctx, N, K)
        for dtype, tdt in ((agg.F32, torch.float32), (agg.BF16, torch.bfloat16)):
            C = torch.full((M, N + 3), 7.0, device="cuda", dtype=tdt)
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
            agg.ag_gemm(ctx, M, N, K, flat.data_ptr() + 2 * offset, ldb, agg.B_KN, C, N + 3, dtype, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(C[:, :N], want.to(tdt)) and bool((C[:, N:] == 7.0).all())
    finally:
        ctx.free()


@pytest.mark.parametrize("tile,W,Ms,K,N", [("64x64", 4, 25, 576, 200), ("64x128", 2, 342, 192, 624), ("128x128", 2, 689, 704, 1496)])
def test_gemm_rs_same_bits_with_and_without_the_other_rows(tile, W, Ms, K, N):
    M, rank = W * Ms, 1
    assert host_rules.kn_tile(_cus(), M, N, K, slices=True) == tile
    g = torch.Generator(device="cuda").manual_seed(52)
    A = torch.empty((M, K), device="cuda", dtype=torch.bfloat16).uniform_(-1, 1, generator=g)
    B = torch.empty((K, N), device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=g)
    want = (A.double().cpu() @ B.double().cpu()).cuda()
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        agg.agg_reserve_b_kn(ctx, N, K)
        cs = ctx.streams()[1]
        own = {}
        for P in (torch.full((M, N), 7.0, device="cuda"), None):
            slots = [torch.zeros((Ms, N), device="cuda") for _ in range(W)]
            slots[rank].fill_(float("nan"))
            R = torch.full((Ms, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            for w in range(W):
                if w != rank:
                    agg.signal_set(ctx, w, cs)
            agg.gemm_rs(ctx, M, N, K, A, K, B, N, agg.B_KN, slots, P, R, N, agg.F32, cs, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(R, slots[rank])
            own[P is None] = R
            if P is not None:
                P[rank * Ms:(rank + 1) * Ms] = R
                assert float((P - want).norm() / want.norm()) < 1e-6          # fp32 sums of K <= 704 products
        assert torch.equal(own[True], own[False])
    finally:
        ctx.free()


def test_weights_beyond_the_memory_side_cache():
    W, Ms, K, N = 2, 50, 4096, 33280             # 273 MB: the streaming hint
    tile = host_rules.kn_tile(_cus(), W * Ms, N, K)
    assert tile in ("64x128", "128x128")
    g = torch.Generator(device="cuda").manual_seed(53)
    shards, B = [_ints(g, Ms, K) for _ in range(W)], _ints(g, K, N)
    ctx = agg.symm_alloc(W, 0, Ms * K * 2, W)
    try:
        agg.agg_reserve_b_kn(ctx, N, K)
        ps, cs = ctx.streams()
        C = torch.full((W * Ms, N), float("nan"), device="cuda")
        agg.signal_reset(ctx)
        torch.cuda.synchronize()
        agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
        agg.ag_gemm(ctx, W * Ms, N, K, B, N, agg.B_KN, C, N, agg.F32, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        assert torch.equal(C, torch.cat(shards).float() @ B.float())
    finally:
        ctx.free()


# tile, rows per rank (of two), K, N: stages fewer than, as many as and one and two laps more than the slots of the 128x128 tile's ring of four,
# and the instances with the streaming hint (256 MB of weights and more)
@pytest.mark.parametrize("tile,Ms,K,N", [("128x128", 626, k, 1568) for k in (128, 256, 320, 512, 576)]
                         + [("64x64", 8, 8192, 16384), ("64x128", 64, 8192, 16384), ("128x128", 100, 8192, 16384)])
def test_every_length_of_the_short_ring_and_the_streaming_instances(tile, Ms, K, N):
    assert host_rules.kn_tile(_cus(), 2 * Ms, N, K) == tile
    g = torch.Generator(device="cuda").manual_seed(K)
    shards, B = [_ints(g, Ms, K) for _ in range(2)], _ints(g, K, N)
    ctx = agg.symm_alloc(2, 0, Ms * K * 2, 2)
    try:
        agg.agg_reserve_b_kn(ctx, N, K)
        assert torch.equal(_call(ctx, shards, 2 * Ms, N, K, B, N, agg.B_KN), torch.cat(shards).float() @ B.float())
    finally:
        ctx.free()


def _call(ctx, shards, M, N, K, B, ldb, layout):
    ps, cs = ctx.streams()
    C = torch.full((M, N), float("nan"), device="cuda")
    agg.signal_reset(ctx)
    torch.cuda.synchronize()
    agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
    agg.ag_gemm(ctx, M, N, K, B, ldb, layout, C, N, agg.F32, cs)
    torch.cuda.synchronize()
    assert agg.agg_status(ctx) == agg.OK
    return C


class _Problem:
    """Random inputs: read in place K is added up in two halves, by the numbered tiles in one run, so that the bits tell which it was."""

    def __init__(self, seed, Ms, K, N, cps=1, in_place=True):
        self.W, self.Ms, self.K, self.N = 4, Ms, K, N
        self.M = self.W * Ms
        assert host_rules.kn_tile(_cus(), self.M, self.N, self.K) == ("128x128" if in_place else None)
        assert host_rules.gemm_tile(_cus(), self.M, self.N, self.K)[0] == "numbered"
        g = torch.Generator(device="cuda").manual_seed(seed)
        self.shards = [torch.empty((Ms, self.K), device="cuda", dtype=torch.bfloat16).uniform_(-1, 1, generator=g) for _ in range(self.W)]
        self.kn = torch.empty((self.K, self.N), device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=g)
        self.nk = self.kn.t().contiguous()
        self.cps, self.open = cps, []
        self.in_place = self.by_kn(self.context())
        numbered = self.context()
        numbered.set_tile_config(5)
        self.copied = self.by_kn(numbered)
        assert torch.equal(self.in_place, self.copied) != in_place and torch.equal(self.copied, self.by_nk(numbered))

    def context(self):
        ctx = agg.symm_alloc(self.W, 0, self.Ms * self.K * 2, self.W * self.cps)
        self.open.append(ctx)
        agg.agg_reserve_b_kn(ctx, self.N, self.K)
        return ctx

    def by_kn(self, ctx):
        return _call(ctx, self.shards, self.M, self.N, self.K, self.kn, self.N, agg.B_KN)

    def by_nk(self, ctx):
        return _call(ctx, self.shards, self.M, self.N, self.K, self.nk, self.K, agg.B_NK)

    def close(self):
        for ctx in self.open:
            ctx.free()
        agg.agg_tune_table_clear()


@pytest.mark.parametrize("Ms,K,N", [(128, 8192, 7168), (256, 4096, 3584)])
def test_tuning_times_the_tiles_that_read_in_place(Ms, K, N):
    # beside the copy the call takes 82 us, with the best of the numbered tiles and its transposed copy 105; and 55 and 57, where a candidate
    # would have to be faster by 1
    p = _Problem(61, Ms, K, N)
    try:
        agg.agg_tune_table_clear()
        tuned, other = p.context(), p.context()
        C = torch.empty((p.M, p.N), device="cuda")
        res = agg.agg_autotune_ag_gemm(tuned, p.M, p.N, p.K, p.kn, p.N, agg.B_KN, C, p.N, agg.F32, p.shards, agg.PRODUCER_KERNEL, 3)
        assert res.configs_tried == 24 and (res.tile_config, res.tile_order) == (-1, agg.ORDER_ROTATED)
        assert agg.agg_tune_table_get(p.W, p.M, p.N, p.K).tile_config == -1
        assert agg.agg_tune_table_apply(other, p.M, p.N, p.K)
        for ctx in (tuned, other):
            assert torch.equal(p.by_kn(ctx), p.in_place)
    finally:
        p.close()


def _entry(tile, order):
    r = agg.TuneResult()
    r.tile_config, r.tile_order, r.producer_workgroups, r.configs_tried, r.best_ms = tile, order, 0, 24, 0.05
    return r


def test_what_is_tuned_for_one_layout_leaves_the_other_alone(tmp_path):
    p = _Problem(62, 128, 8192, 7168)
    try:
        agg.agg_tune_table_clear()
        for order in (agg.ORDER_ROTATED, agg.ORDER_SUBCHUNK):
            agg.agg_tune_table_put(p.W, p.M, p.N, p.K, _entry(5, order))
            ctx = p.context()
            assert agg.agg_tune_table_apply(ctx, p.M, p.N, p.K)
            assert torch.equal(p.by_nk(ctx), p.copied) and torch.equal(p.by_kn(ctx), p.in_place)
            ctx.set_tile_config(5)                              # by number: the transposed copy, and its bits
            assert torch.equal(p.by_kn(ctx), p.copied)
        # tuning the [K][N] operand keeps the entry of the other one, in memory and in a file
        tuned = p.context()
        C = torch.empty((p.M, p.N), device="cuda")
        res = agg.agg_autotune_ag_gemm(tuned, p.M, p.N, p.K, p.kn, p.N, agg.B_KN, C, p.N, agg.F32, p.shards, agg.PRODUCER_KERNEL, 3)
        assert res.tile_config == -1
        for _ in range(2):
            assert agg.agg_tune_table_size() == 2
            assert agg.agg_tune_table_get(p.W, p.M, p.N, p.K).tile_config == 5
            ctx = p.context()
            assert agg.agg_tune_table_apply(ctx, p.M, p.N, p.K)
            assert torch.equal(p.by_nk(ctx), p.copied) and torch.equal(p.by_kn(ctx), p.in_place)
            agg.agg_tune_table_save(str(tmp_path / "t.txt"))
            agg.agg_tune_table_clear()
            assert agg.agg_tune_table_load(str(tmp_path / "t.txt")) == 2
    finally:
        p.close()


def test_the_order_of_the_tiles_is_kept_where_it_counts_and_changes_no_bits():
    # one round of the numbered tile: all start at once, B may be read in place; two rounds: they follow the order that is asked for
    for Ms, K, N, cps, in_place in ((256, 4096, 3584, 2, True), (768, 2048, 2592, 6, False)):
        p = _Problem(63, Ms, K, N, cps, in_place)
        try:
            for order in (agg.ORDER_SUBCHUNK, agg.ORDER_ROTATED):
                ctx = p.context()
                ctx.set_tile_order(order)
                assert torch.equal(p.by_kn(ctx), p.in_place if in_place else p.copied), (Ms, order)
        finally:
            p.close()
