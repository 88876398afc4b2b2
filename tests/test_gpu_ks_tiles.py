"""Every K-split tile in every form that the automatic choice reaches: whole matrices, GEMM + ReduceScatter's slices, MoE segments
(rows gathered by token, rows in place); each with K longer than its ring, pieces of K that do not fill the last pass, ragged
edges, and, where a choice with more tiles than workgroups exists, that as well.  What the choice takes is asserted.  Integer inputs:
sums of at most 4 x 6464 are exact in fp32 in any order."""
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


# tile, whether its workgroups take a second tile, W, rows per rank, K, N
TILES = [
    ("16x16", False, 2, 24, 2240, 1000),
    ("16x16", False, 3, 5, 2304, 513),
    ("16x32", False, 2, 24, 1728, 2531),
    ("16x32", True, 2, 8, 3392, 8501),
    ("32x32", False, 2, 40, 1152, 2500),
    ("32x32", True, 3, 6, 4544, 34911),         # 317 MB of weights: the streaming hint
    ("64x32", False, 3, 15, 1664, 4301),
    ("64x32", False, 4, 16, 1728, 5001),
    ("64x64", False, 2, 100, 576, 2501),
    ("64x64", True, 3, 6, 6464, 41569),
    ("64x128", False, 2, 300, 448, 2001),
    ("64x128", True, 2, 20, 320, 66307),
]


# The same for GEMM + ReduceScatter, whose choice counts the tiles that have to publish themselves.
SLICED_TILES = [
    ("16x16", False, 3, 5, 2304, 513),
    ("16x32", False, 2, 24, 1728, 2531),
    ("32x32", False, 2, 40, 1152, 2500),
    ("64x32", False, 8, 8, 3584, 8192),
    ("64x64", False, 2, 100, 576, 2501),
    ("64x64", False, 2, 8, 3392, 8501),
    ("64x128", False, 2, 300, 448, 2001),
    ("64x128", True, 2, 20, 320, 66307),
    ("64x128", True, 3, 6, 4544, 34911),
]


@pytest.mark.parametrize("tile,loops,W,Ms,K,N", TILES)
def test_ag_gemm_exact(tile, loops, W, Ms, K, N):
    name, tiles = host_rules.gemm_tile(_cus(), W * Ms, N, K)
    assert name == tile and (tiles > _cus()) == loops
    g = torch.Generator(device="cuda").manual_seed(31)
    shards, B = [_ints(g, Ms, K) for _ in range(W)], _ints(g, N, K)
    want = torch.cat(shards).float() @ B.float().t()
    ctx = agg.symm_alloc(W, W - 1, Ms * K * 2, W)
    try:
        ps, cs = ctx.streams()
        for dtype, tdt in ((agg.F32, torch.float32), (agg.BF16, torch.bfloat16)):
            C = torch.full((W * Ms, N + 3), 7.0, device="cuda", dtype=tdt)           # padded rows: the padding stays
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
            agg.ag_gemm(ctx, W * Ms, N, K, B, K, agg.B_NK, C, N + 3, dtype, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(C[:, :N], want.to(tdt)) and bool((C[:, N:] == 7.0).all())
    finally:
        ctx.free()


@pytest.mark.parametrize("tile,loops,W,Ms,K,N", SLICED_TILES)
def test_slices_exact(tile, loops, W, Ms, K, N):
    name, tiles = host_rules.gemm_tile(_cus(), W * Ms, N, K, slices=True)
    assert name == tile and (tiles > _cus()) == loops
    g = torch.Generator(device="cuda").manual_seed(31)
    A, B = _ints(g, W * Ms, K), _ints(g, N, K)
    want = A.float() @ B.float().t()
    rank = W - 1
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        # W slices, each with its signal, all but the last one at a destination of its own
        dst = [torch.full((Ms, N), float("nan"), device="cuda") if w != rank else None for w in range(W)]
        P = torch.full((W * Ms, N), 7.0, device="cuda")
        words = torch.zeros((W, agg.SIGNAL_STRIDE), device="cuda", dtype=torch.int32)
        agg.signal_reset(ctx)
        torch.cuda.synchronize()
        agg.gemm_rs_scatter(ctx, W * Ms, N, K, A, K, B, K, agg.B_NK, dst, P, [words[w] for w in range(W)], 1 % W, ctx.streams()[1])
        torch.cuda.synchronize()
        for w in range(W):
            part = dst[w] if w != rank else P[w * Ms:(w + 1) * Ms]
            assert torch.equal(part, want[w * Ms:(w + 1) * Ms]), w
        assert bool((P[:rank * Ms] == 7.0).all())
        assert words[:, 0].tolist() == [ctx.epoch] * W and int(words[:, 1:].abs().sum()) == 0
    finally:
        ctx.free()


def test_the_choices_above_reach_every_tile_of_the_dense_table():
    for table in (TILES, SLICED_TILES):
        assert {t[0] for t in table} == {host_rules.tile_name(t) for t in host_rules.dense_ks_tiles()}


# tile, output type, whether its workgroups take a second tile, tokens, top-k, experts, N, K
MOE_TILES = [
    ("16x32", agg.BF16, False, 60, 1, 20, 100, 1792),
    ("16x32", agg.F32, True, 120, 3, 38, 404, 1856),
    ("16x64", agg.F32, True, 462, 2, 93, 268, 832),
    ("16x64", agg.BF16, True, 1068, 1, 88, 305, 192),
    ("32x32", agg.F32, True, 4844, 3, 78, 28, 320),
    ("32x32", agg.BF16, False, 1398, 3, 6, 20, 1088),
    ("64x64", agg.F32, True, 1820, 3, 3, 268, 3392),
    ("64x64", agg.BF16, True, 1708, 2, 89, 277, 192),
    ("64x128", agg.F32, True, 1296, 2, 2, 1492, 1600),
    ("64x128", agg.BF16, True, 2096, 3, 4, 555, 576),
]


def _routing(g, T, topk, E):
    ids = torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    order = torch.argsort(ids.reshape(-1).long(), stable=True)
    return ids, order, torch.bincount(ids.reshape(-1).long(), minlength=E).tolist()


def _grouped(X, B, lengths):
    out, at = [], 0
    for e, n in enumerate(lengths):
        out.append(X[at:at + n] @ B[e].float().t())
        at += n
    return torch.cat(out)


def _loops(tile, N, lengths):
    bm, bn = (int(x) for x in tile.split("x"))
    return sum(-(-n // bm) for n in lengths) * -(-N // bn) > _cus()


@pytest.mark.parametrize("tile,dtype,loops,T,topk,E,N,K", MOE_TILES)
def test_moe_gathered_rows_exact(tile, dtype, loops, T, topk, E, N, K):
    assert host_rules.moe_tile(_cus(), T, topk, E, N, K, True, dtype == agg.F32) == tile
    g = torch.Generator(device="cuda").manual_seed(32)
    W = 2
    shards, B = [_ints(g, T // W, K) for _ in range(W)], _ints(g, E, N, K)
    ids, order, lengths = _routing(g, T, topk, E)
    assert _loops(tile, N, lengths) == loops
    want = _grouped(torch.cat(shards)[order // topk].float(), B, lengths)
    tdt = torch.float32 if dtype == agg.F32 else torch.bfloat16
    tok, seg = torch.empty(T * topk, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 0, T // W * K * 2, W)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        for call in (agg.ag_moe_gemm, agg.ag_moe_gemm_static):
            Y = torch.full((T * topk, N), float("nan"), device="cuda", dtype=tdt)
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
            call(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N, dtype, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(tok.long(), order // topk)
            assert torch.equal(Y, want.to(tdt))
    finally:
        ctx.free()


@pytest.mark.parametrize("tile,dtype,loops,T,topk,E,N,K", [m for m in MOE_TILES if m[1] == agg.F32])
def test_moe_rows_in_place_exact(tile, dtype, loops, T, topk, E, N, K):
    N = -(-N // 4) * 4
    assert host_rules.moe_tile(_cus(), T, topk, E, N, K, False, True) == tile
    g = torch.Generator(device="cuda").manual_seed(33)
    W, rank = 2, 1
    H, B = _ints(g, T * topk, K), _ints(g, E, N, K)
    ids, order, lengths = _routing(g, T, topk, E)
    assert _loops(tile, N, lengths) == loops
    want = _grouped(H.float(), B, lengths)
    gate = torch.ones((T, topk), device="cuda")
    pos_want = torch.empty_like(order)
    pos_want[order] = torch.arange(T * topk, device="cuda")
    tok, pos = (torch.empty(T * topk, device="cuda", dtype=torch.int32) for _ in range(2))
    seg = torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        slots = [torch.zeros((T // W, N), device="cuda") for _ in range(W)]
        Y, Z = torch.full((T * topk, N), float("nan"), device="cuda"), torch.full((T, N), float("nan"), device="cuda")
        R = torch.full((T // W, N), float("nan"), device="cuda")
        agg.signal_reset(ctx)
        torch.cuda.synchronize()
        agg.signal_set(ctx, 0, cs)
        agg.moe_rs(ctx, T, topk, E, N, K, H, B, ids, gate, Y, tok, seg, pos, slots, Z, R, N, agg.F32, cs, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        assert torch.equal(pos.long(), pos_want)
        assert torch.equal(Y, want)
        sums = Y[pos.long()].reshape(T, topk, N).sum(dim=1)
        assert torch.equal(R, sums[T // W:]) and torch.equal(Z[:T // W], sums[:T // W])
    finally:
        ctx.free()


def test_the_choices_above_reach_every_tile_of_the_moe_table():
    tiles = {host_rules.tile_name(t) for t in host_rules.moe_ks_tiles()}
    assert {m[0] for m in MOE_TILES} == tiles == {m[0] for m in MOE_TILES if m[1] == agg.F32} == {m[0] for m in MOE_TILES if m[1] == agg.BF16}
