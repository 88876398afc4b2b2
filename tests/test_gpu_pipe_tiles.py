"""The grouped GEMM's tiles that walk all of a workgroup's tiles as one stream of K stages (csrc/gemm_pipe.h): segments at the edges of a
tile, K of one stage and more than a ring holds, several tiles per workgroup, rows of Y that start on 16 bytes and ones that do not, weights
beyond the memory-side cache, and signals that come while a workgroup is between two tiles.  The tile that is taken is asserted.
Integer inputs: sums of at most 4 x 6208 are exact in fp32 in any order."""
import numpy as np
import pytest
import torch

import host_rules
import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu


def _ints(g, *shape):
    return torch.randint(-2, 3, shape, device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)


def _routing(g, T, topk, E, bm):
    """Expert ids: with one expert per token, segments of 0, 1, bm - 1, bm and bm + 1 rows among the random ones."""
    if topk > 1:
        return torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    edges = [n for n in (0, 1, bm - 1, bm, bm + 1)][: E - 1]
    assert sum(edges) <= T
    rest = torch.randint(len(edges), E, (T - sum(edges),), device="cuda", generator=g)
    ids = torch.cat([torch.full((n,), e, device="cuda", dtype=torch.int64) for e, n in enumerate(edges)] + [rest])
    return ids[torch.randperm(T, device="cuda", generator=g)].to(torch.int32).view(T, 1).contiguous()


def _expected(X, B, ids):
    flat = ids.reshape(-1).long()
    order, lengths = torch.argsort(flat, stable=True), torch.bincount(flat, minlength=B.shape[0]).tolist()
    X, out, at = X(order).float(), [], 0
    for e, n in enumerate(lengths):
        out.append(X[at:at + n] @ B[e].float().t())
        at += n
    return order, torch.cat(out)


# tile, output type, tokens, top-k, experts, N, K, columns of Y behind the last one
GATHERED = [
    ("128x192", agg.F32, 6390, 1, 12, 701, 128, 0),
    ("128x192", agg.BF16, 4908, 3, 30, 1152, 320, 0),
    ("128x192", agg.BF16, 6028, 3, 37, 808, 832, 8),
    ("128x224", agg.F32, 1086, 1, 37, 1157, 64, 3),
    ("128x224", agg.F32, 6360, 2, 30, 1188, 192, 0),
    ("128x224", agg.BF16, 5256, 3, 36, 1016, 320, 0),
    ("192x192", agg.BF16, 5554, 3, 21, 1163, 64, 1),
    ("192x192", agg.BF16, 6480, 3, 36, 1008, 192, 0),
    ("192x192", agg.F32, 6502, 3, 36, 1064, 832, 4),
    ("320x128", agg.F32, 3634, 3, 24, 616, 64, 0),
    ("320x128", agg.BF16, 5362, 3, 27, 1094, 128, 2),
    ("320x128", agg.BF16, 5272, 3, 28, 1104, 320, 0),
    ("320x128", agg.BF16, 5270, 1, 23, 1168, 832, 0),
    ("128x192", agg.BF16, 3000, 1, 20, 1100, 6208, 0),         # 273 MB of weights: the streaming hint
    ("320x128", agg.BF16, 6600, 1, 22, 1024, 6208, 0),
]


@pytest.mark.parametrize("tile,dtype,T,topk,E,N,K,pad", GATHERED)
def test_gathered_rows_exact(tile, dtype, T, topk, E, N, K, pad):
    cus = agg.agg_device_info()[0]
    assert host_rules.moe_tile(cus, T, topk, E, N, K, True, dtype == agg.F32) == tile
    g = torch.Generator(device="cuda").manual_seed(41)
    W, cps = 2, 1
    while T // W % (2 * cps) == 0 and cps < 4:
        cps *= 2
    shards, B = [_ints(g, T // W, K) for _ in range(W)], _ints(g, E, N, K)
    ids = _routing(g, T, topk, E, int(tile.split("x")[0]))
    order, want = _expected(lambda o: torch.cat(shards)[o // topk], B, ids)
    tdt = torch.float32 if dtype == agg.F32 else torch.bfloat16
    tok, seg = torch.empty(T * topk, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 1, T // W * K * 2, W * cps)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        for gemm_first in (False, True):
            Y = torch.full((T * topk, N + pad), 7.0, device="cuda", dtype=tdt)
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            if not gemm_first:
                agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
            agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N + pad, dtype, cs)
            if gemm_first:                                      # chunk by chunk, by a few workgroups
                agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 2, ps)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(tok.long(), order // topk)
            assert torch.equal(Y[:, :N], want.to(tdt)) and bool((Y[:, N:] == 7.0).all())
    finally:
        ctx.free()


# tile, tokens, top-k, experts, N, K
IN_PLACE = [
    ("128x192", 5428, 3, 38, 920, 192),
    ("128x224", 5946, 3, 22, 1088, 192),
    ("192x192", 6548, 3, 24, 1140, 64),
    ("192x192", 5962, 3, 26, 1076, 320),
    ("320x128", 6106, 3, 30, 1004, 64),
    ("320x128", 6036, 3, 32, 960, 192),
]


@pytest.mark.parametrize("tile,T,topk,E,N,K", IN_PLACE)
def test_rows_in_place_exact(tile, T, topk, E, N, K):
    cus = agg.agg_device_info()[0]
    assert host_rules.moe_tile(cus, T, topk, E, N, K, False, True) == tile
    g = torch.Generator(device="cuda").manual_seed(42)
    W, rank = 2, 0
    H, B = _ints(g, T * topk, K), _ints(g, E, N, K)
    ids = _routing(g, T, topk, E, int(tile.split("x")[0]))
    order, want = _expected(lambda o: H, B, ids)
    gate = torch.ones((T, topk), device="cuda")
    pos_want = torch.empty_like(order)
    pos_want[order] = torch.arange(T * topk, device="cuda")
    tok, pos = (torch.empty(T * topk, device="cuda", dtype=torch.int32) for _ in range(2))
    seg = torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        cs = ctx.streams()[1]
        slots = [torch.zeros((T // W, N), device="cuda") for _ in range(W)]
        R = {}
        for Z in (torch.full((T, N), float("nan"), device="cuda"), None):     # all tokens' rows, and this rank's alone: the same bits
            Y = torch.full((T * topk, N), float("nan"), device="cuda")
            R[Z is None] = torch.full((T // W, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            agg.signal_set(ctx, 1, cs)
            agg.moe_rs(ctx, T, topk, E, N, K, H, B, ids, gate, Y, tok, seg, pos, slots, Z, R[Z is None], N, agg.F32, cs, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(pos.long(), pos_want)
            if Z is not None:
                assert torch.equal(Y, want)
                sums = want[pos.long()].reshape(T, topk, N).sum(dim=1)
                assert torch.equal(Z[T // W:], sums[T // W:])
            assert torch.equal(R[Z is None], sums[:T // W])
    finally:
        ctx.free()


def test_a_signal_that_never_comes_ends_the_launch():
    # 2 experts of some 2900 rows: a workgroup's later tiles wait for signals that its first one did not look at
    T, topk, E, N, K, W, cps = 5904, 1, 2, 3000, 192, 2, 4
    tile = host_rules.moe_tile(agg.agg_device_info()[0], T, topk, E, N, K, True, True)
    assert tile in ("128x192", "128x224", "192x192", "320x128")
    g = torch.Generator(device="cuda").manual_seed(43)
    shards, B = [_ints(g, T // W, K) for _ in range(W)], _ints(g, E, N, K)
    ids = torch.randint(0, E, (T, 1), device="cuda", generator=g).to(torch.int32)
    tok, seg = torch.empty(T, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    Y = torch.empty((T, N), device="cuda")
    ctx = agg.symm_alloc(W, 0, T // W * K * 2, W * cps)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        ctx.set_wait_limit_us(2000)
        agg.signal_reset(ctx)
        agg.ag_producer_emulate(ctx, shards, [], agg.PRODUCER_KERNEL, 0, ps)          # this rank's shard alone
        torch.cuda.synchronize()
        agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N, agg.F32, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.ERR_TIMEOUT
        # and the context works as before
        ctx.set_wait_limit_us(2000000)
        agg.signal_reset(ctx)
        agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
        agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N, agg.F32, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        assert torch.equal(Y, _expected(lambda o: torch.cat(shards)[o], B, ids)[1])
    finally:
        ctx.free()


@pytest.mark.parametrize("T,E", [(5904, 3), (6400, 4)])
def test_a_tile_that_is_done_is_stored_before_the_next_ones_signals_are_waited_for(T, E):
    # experts of some 1600 to 2000 rows, the other rank's shard never arrives: what a workgroup has computed before it comes to a tile with
    # rows of that shard is in Y, and nothing else is
    topk, N, K, W, cps = 1, 3000, 192, 2, 4
    cus = agg.agg_device_info()[0]
    tile = host_rules.moe_tile(cus, T, topk, E, N, K, True, True)
    assert tile in ("128x192", "128x224", "192x192", "320x128")
    bm, bn = map(int, tile.split("x"))
    g = torch.Generator(device="cuda").manual_seed(44)
    shards, B = [_ints(g, T // W, K) for _ in range(W)], _ints(g, E, N, K)
    ids = torch.randint(0, E, (T, 1), device="cuda", generator=g).to(torch.int32)
    order, want = _expected(lambda o: torch.cat(shards)[o], B, ids)
    own = (order < T // W).cpu().numpy()
    ends = np.cumsum(torch.bincount(ids.reshape(-1).long(), minlength=E).cpu().numpy())
    tiles = []                                                  # the list: an expert's columns one after the other, rows fastest
    for e, hi in enumerate(ends):
        lo = hi - (ends[e] - (ends[e - 1] if e else 0))
        tiles += [(m, min(m + bm, hi), n) for n in range(0, N, bn) for m in range(lo, hi, bm)]
    done = []
    for t, (lo, hi, n) in enumerate(tiles):                     # tile t is walked by the workgroup that has had tile t - cus
        done.append(bool(own[lo:hi].all()) and (t < cus or done[t - cus]))
    assert any(d and not done[t + cus] for t, d in enumerate(done[:-cus]))
    Y_want = torch.full((T, N), 7.0, device="cuda")
    for d, (lo, hi, n) in zip(done, tiles):
        if d:
            Y_want[lo:hi, n:n + bn] = want[lo:hi, n:n + bn]
    tok, seg = torch.empty(T, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 0, T // W * K * 2, W * cps)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        ctx.set_wait_limit_us(2000)
        for config in (5, -1):                                  # a numbered tile (128x128: another list) and the automatic choice
            Y = torch.full((T, N), 7.0, device="cuda")
            ctx.set_tile_config(config)
            agg.signal_reset(ctx)
            agg.ag_producer_emulate(ctx, shards, [], agg.PRODUCER_KERNEL, 0, ps)
            torch.cuda.synchronize()
            agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N, agg.F32, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.ERR_TIMEOUT
            assert bool(((Y == want) | (Y == 7.0)).all())
        assert torch.equal(Y, Y_want)
    finally:
        ctx.free()


# tile, output type, tokens, top-k, experts, N, K
SAME_BITS = [
    ("128x192", agg.BF16, 4908, 3, 30, 1152, 320),
    ("128x224", agg.F32, 6360, 2, 30, 1188, 192),
    ("192x192", agg.F32, 6502, 3, 36, 1064, 832),
    ("320x128", agg.BF16, 5270, 1, 23, 1168, 832),
    ("320x128", agg.F32, 3634, 3, 24, 616, 64),
]


@pytest.mark.parametrize("tile,dtype,T,topk,E,N,K", SAME_BITS)
def test_the_same_bits_as_the_numbered_tiles(tile, dtype, T, topk, E, N, K):
    # random inputs: a sum over K in another order would show
    assert host_rules.moe_tile(agg.agg_device_info()[0], T, topk, E, N, K, True, dtype == agg.F32) == tile
    g = torch.Generator(device="cuda").manual_seed(45)
    W = 2
    shards = [torch.empty((T // W, K), device="cuda", dtype=torch.bfloat16).uniform_(-1, 1, generator=g) for _ in range(W)]
    B = torch.empty((E, N, K), device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=g)
    ids = _routing(g, T, topk, E, int(tile.split("x")[0]))
    tdt = torch.float32 if dtype == agg.F32 else torch.bfloat16
    tok, seg = torch.empty(T * topk, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 1, T // W * K * 2, W)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        Y = {}
        for config in (-1, 4, 5, 6):                            # 16x16x32 MFMAs: 256x224, 128x128, 256x256
            Y[config] = torch.full((T * topk, N), float("nan"), device="cuda", dtype=tdt)
            ctx.set_tile_config(config)
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
            agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y[config], N, dtype, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
        for config in (4, 5, 6):
            assert torch.equal(Y[-1].view(torch.uint8), Y[config].view(torch.uint8)), config
    finally:
        ctx.free()
