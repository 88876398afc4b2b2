"""GEMM + ReduceScatter and MoE + ReduceScatter on one stream, where the reducer raises the own slot's signals, and on two, where the GEMM or
the top-k reduction does: the same bits, and every one of the signals raised."""
import numpy as np
import pytest
import torch

import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu


class _Words:
    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 3}


def _signals(ctx, n):
    return torch.as_tensor(_Words(ctx.signals, n * agg.SIGNAL_STRIDE), device="cuda").view(n, agg.SIGNAL_STRIDE)[:, 0]


def _both(W, rank, chunks, Ms, N, call, reserve=lambda ctx: None):
    """call(ctx, slots, R, gemm stream, reduce stream) on two streams and on one: R and the own slot of both."""
    n_signals = W * 4
    ctx = agg.symm_alloc(W, rank, 16, n_signals)
    g = torch.Generator(device="cuda").manual_seed(7)
    peers = [torch.randn((Ms, N), device="cuda", generator=g) for _ in range(W)]
    got = []
    try:
        ctx.set_rs_chunks(chunks)
        reserve(ctx)
        ps, cs = ctx.streams()
        for a, b in ((ps, cs), (ps, cs), (cs, cs), (cs, cs)):
            slots = [torch.full((Ms, N), float("nan"), device="cuda") if w == rank else peers[w] for w in range(W)]
            R = torch.full((Ms, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            for w in range(W):
                for c in range(chunks if w != rank else 0):
                    agg.signal_set(ctx, w * 4 + c, cs)
            call(ctx, slots, R, a, b)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            words = _signals(ctx, n_signals).cpu().numpy().reshape(W, 4)
            assert (words[:, :chunks] == ctx.epoch).all()
            assert not (words[rank, chunks:] == ctx.epoch).any()
            got.append((R.cpu().numpy().view(np.uint32), slots[rank].cpu().numpy().view(np.uint32)))
    finally:
        ctx.free()
    for R, own in got[1:]:
        assert np.array_equal(R, got[0][0]) and np.array_equal(own, got[0][1])
    want = sum(np.float64(1) * (peers[w].cpu().numpy() if w != rank else got[0][1].view(np.float32)) for w in range(W))
    # W fp32 additions: at most W half-ulps of the largest partial sum
    assert np.abs(got[0][0].view(np.float32) - want).max() <= W * 2.0 ** -23 * np.abs(want).max() * W


# worlds with and without an unrolled reducer; the own slot first, in the middle and last; one signal, and chunks; a K-split tile (few rows),
# a numbered one (256 x 4096 rows of whole tiles)
@pytest.mark.parametrize("W,rank,chunks,Ms,N,K", [(2, 0, 1, 8, 100, 128), (3, 2, 2, 6, 260, 320), (5, 1, 4, 16, 96, 64), (8, 7, 1, 64, 512, 256),
                                                  (4, 2, 4, 1024, 2048, 64)])
@pytest.mark.parametrize("other", [False, True])
def test_gemm_rs(W, rank, chunks, Ms, N, K, other):
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.empty((W * Ms, K), device="cuda", dtype=torch.bfloat16).uniform_(-1, 1, generator=g)
    B = torch.empty((N, K), device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=g)
    P = torch.empty((W * Ms, N), device="cuda") if other else None
    _both(W, rank, chunks, Ms, N, lambda ctx, slots, R, a, b: agg.gemm_rs(ctx, W * Ms, N, K, A, K, B, K, agg.B_NK, slots, P, R, N, agg.F32, a, b))


@pytest.mark.parametrize("W,rank,chunks,Ms,N,K,E,topk", [(2, 1, 1, 3, 100, 64, 4, 2), (4, 0, 2, 16, 128, 192, 8, 1), (8, 3, 1, 300, 512, 64, 16, 3),
                                                       (2, 0, 4, 5000, 1024, 64, 4, 1)])       # the last: several own blocks per workgroup of the reduction
@pytest.mark.parametrize("other", [False, True])
def test_moe_rs(W, rank, chunks, Ms, N, K, E, topk, other):
    g = torch.Generator(device="cuda").manual_seed(4)
    T = W * Ms
    H = torch.empty((T * topk, K), device="cuda", dtype=torch.bfloat16).uniform_(-1, 1, generator=g)
    B = torch.empty((E, N, K), device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=g)
    ids = torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    gate = torch.rand((T, topk), device="cuda", generator=g)
    Y, Z = torch.empty((T * topk, N), device="cuda"), torch.empty((T, N), device="cuda") if other else None
    tok, pos = (torch.empty(T * topk, device="cuda", dtype=torch.int32) for _ in range(2))
    seg = torch.empty(E + 1, device="cuda", dtype=torch.int32)
    _both(W, rank, chunks, Ms, N, lambda ctx, slots, R, a, b: agg.moe_rs(ctx, T, topk, E, N, K, H, B, ids, gate, Y, tok, seg, pos, slots, Z, R, N,
                                                                         agg.F32, a, b), lambda ctx: agg.agg_reserve_moe(ctx, T, topk, E, N))


def test_gemm_rs_scatter_beside_moe_rs():
    """Both count what has been stored before they raise a signal: on one context at the same time, each counts its own."""
    W, Ms, N, K, E, topk = 2, 512, 1024, 64, 4, 2
    T = W * Ms
    g = torch.Generator(device="cuda").manual_seed(5)

    def ints(*shape):
        return torch.randint(-2, 3, shape, device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)

    A, B, H, B2 = ints(T, K), ints(N, K), ints(T * topk, K), ints(E, N, K)
    ids = torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    gate = torch.ones((T, topk), device="cuda")
    flat = ids.reshape(-1).long()
    order = torch.argsort(flat, stable=True)
    rows = torch.empty((T * topk, N), device="cuda")
    for e in range(E):
        at = flat[order] == e
        rows[at] = H[at].float() @ B2[e].float().t()
    where = torch.empty_like(order)
    where[order] = torch.arange(T * topk, device="cuda")
    peer = torch.randint(-8, 9, (Ms, N), device="cuda", generator=g).float()
    want_own, want_P = rows[where].view(T, topk, N).sum(dim=1)[:Ms], A.float() @ B.float().t()
    ctx = agg.symm_alloc(W, 0, 16, W * 4)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        third = torch.cuda.Stream()
        Y, Z, R = (torch.empty((n, N), device="cuda") for n in (T * topk, T, Ms))
        tok, pos = (torch.empty(T * topk, device="cuda", dtype=torch.int32) for _ in range(2))
        seg = torch.empty(E + 1, device="cuda", dtype=torch.int32)
        own = torch.empty((Ms, N), device="cuda")
        for chunks in (1, 4) * 4:
            ctx.set_rs_chunks(chunks)
            P = [torch.full((Ms, N), float("nan"), device="cuda") for _ in range(W)]
            raised = torch.zeros((W, chunks, agg.SIGNAL_STRIDE), device="cuda", dtype=torch.int32)
            own.fill_(float("nan"))
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            for c in range(chunks):
                agg.signal_set(ctx, 4 + c, cs)
            agg.gemm_rs_scatter(ctx, T, N, K, A, K, B, K, agg.B_NK, P, None, [raised[w].data_ptr() for w in range(W)], 0, third)
            agg.moe_rs(ctx, T, topk, E, N, K, H, B2, ids, gate, Y, tok, seg, pos, [own, peer], Z, R, N, agg.F32, ps, cs)
            agg.gemm_rs_scatter(ctx, T, N, K, A, K, B, K, agg.B_NK, P, None, [raised[w].data_ptr() for w in range(W)], 0, third)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(own, want_own) and torch.equal(R, want_own + peer) and torch.equal(torch.cat(P), want_P)
            assert bool((raised[:, :, 0] == ctx.epoch).all())
    finally:
        ctx.free()
