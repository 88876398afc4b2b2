"""Worlds on both sides of what the launches' short arguments hold (eight ranks): the copy, the GEMM behind it, GEMM + ReduceScatter."""
import pytest
import torch

import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu


def _ints(g, *shape):
    return torch.randint(-2, 3, shape, device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)


@pytest.mark.parametrize("W", [1, 7, 8, 9, 64])
def test_ag_gemm(W):
    rows, N, K, rank = 6, 72, 128, W // 2
    g = torch.Generator(device="cuda").manual_seed(W)
    shards, B = [_ints(g, rows, K) for _ in range(W)], _ints(g, N, K)
    want = torch.cat(shards).float() @ B.float().t()
    ctx = agg.symm_alloc(W, rank, rows * K * 2, W)
    try:
        for mode in (agg.PRODUCER_KERNEL, agg.PRODUCER_KERNEL | agg.PRODUCER_NARROW | agg.PRODUCER_LOCAL_LAST):
            C = torch.full((W * rows, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            agg.ag_producer_emulate(ctx, shards, None, mode, 0, None)
            agg.ag_gemm(ctx, W * rows, N, K, B, K, agg.B_NK, C, N, agg.F32, None)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK and torch.equal(C, want)
    finally:
        ctx.free()


@pytest.mark.parametrize("W", [7, 8, 9, 64])
@pytest.mark.parametrize("two_streams", [False, True])
def test_gemm_rs(W, two_streams):
    Ms, N, K, rank = 6, 72, 128, W - 1
    g = torch.Generator(device="cuda").manual_seed(W)
    A, B = _ints(g, W * Ms, K), _ints(g, N, K)
    prod = A.float() @ B.float().t()
    slots = [torch.randint(-8, 9, (Ms, N), device="cuda", generator=g).float() for _ in range(W)]
    want = sum(slots[:rank]) + prod[rank * Ms:]
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        ps, cs = ctx.streams()
        P, R = torch.full((W * Ms, N), float("nan"), device="cuda"), torch.full((Ms, N), float("nan"), device="cuda")
        agg.signal_reset(ctx)
        torch.cuda.synchronize()
        for w in range(W - 1):
            agg.signal_set(ctx, w, cs)
        agg.gemm_rs(ctx, W * Ms, N, K, A, K, B, K, agg.B_NK, slots, P, R, N, agg.F32, ps if two_streams else cs, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        assert torch.equal(R, want) and torch.equal(P[:rank * Ms], prod[:rank * Ms])
    finally:
        ctx.free()
