"""AllGather-GEMM and MoE behind the copy of all shards on one stream, where no signal is looked at: right in every form, and only there."""
import pytest
import torch

import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu
W, K = 4, 192


def _ints(g, *shape):
    return torch.randint(-2, 3, shape, device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)


class Problem:
    """W shards of `rows` rows, whole numbers: every product is exact."""

    def __init__(self, rows, N, layout, out=agg.F32):
        g = torch.Generator(device="cuda").manual_seed(rows)
        self.rows, self.N, self.layout, self.out = rows, N, layout, out
        self.shards = [_ints(g, rows, K) for _ in range(W)]
        self.B = _ints(g, N, K) if layout == agg.B_NK else _ints(g, K, N)
        wide = self.B.float().t() if layout == agg.B_NK else self.B.float()
        self.want = torch.cat(self.shards).float() @ wide
        self.C = torch.empty((W * rows, N), device="cuda", dtype=torch.float32 if out == agg.F32 else torch.bfloat16)
        self.ctx = agg.symm_alloc(W, 1, rows * K * 2, W)
        if layout == agg.B_KN:
            agg.agg_reserve_b_kn(self.ctx, N, K)
        torch.cuda.synchronize()

    def deliver(self, stream, order=None, mode=agg.PRODUCER_KERNEL):
        agg.ag_producer_emulate(self.ctx, self.shards, order, mode, 0, stream)

    def gemm(self, stream):
        ld = K if self.layout == agg.B_NK else self.N
        agg.ag_gemm(self.ctx, W * self.rows, self.N, K, self.B, ld, self.layout, self.C, self.N, self.out, stream)

    def right(self):
        torch.cuda.synchronize()
        return agg.agg_status(self.ctx) == agg.OK and torch.equal(self.C.float(), self.want.to(self.C.dtype).float())


# a K-split tile with rings per wave, with a shared one, numbered tiles in several rounds; [K][N] in place and transposed
@pytest.mark.parametrize("rows,N,layout", [(3, 200, agg.B_NK), (250, 1500, agg.B_NK), (1024, 4096, agg.B_NK), (100, 1024, agg.B_KN), (3, 203, agg.B_KN)])
@pytest.mark.parametrize("where", ["default", "producer", "consumer", "other"])
def test_copy_and_gemm_on_one_stream(rows, N, layout, where):
    p = Problem(rows, N, layout)
    try:
        ps, cs = p.ctx.streams()
        other = torch.cuda.Stream()
        st = {"default": None, "producer": ps, "consumer": cs, "other": other.cuda_stream}[where]
        for epoch in range(3):
            for x in p.shards:
                x.neg_()                                   # other rows in every epoch: nothing of the one before may be seen
            p.want.neg_()
            p.C.fill_(float("nan"))
            torch.cuda.synchronize()
            agg.signal_reset(p.ctx)
            if epoch == 1:                                 # over several calls, the own shard first and not again
                p.deliver(st, [2])
                p.deliver(st, [3, 0], agg.PRODUCER_KERNEL | agg.PRODUCER_SKIP_LOCAL)
            else:
                p.deliver(st)
            p.gemm(st)
            assert p.right(), epoch
    finally:
        p.ctx.free()


def test_one_shard_from_another_stream():
    p = Problem(250, 1500, agg.B_NK)
    try:
        ps, cs = p.ctx.streams()
        for first, last in ((cs, ps), (ps, cs), (cs, ps)):
            for x in p.shards:
                x.neg_()                                   # other rows each time: a GEMM that does not wait finds those of the time before
            p.want.neg_()
            p.C.fill_(float("nan"))
            torch.cuda.synchronize()
            agg.signal_reset(p.ctx)
            p.deliver(first, [2, 0])
            p.deliver(last, [3], agg.PRODUCER_KERNEL | agg.PRODUCER_SKIP_LOCAL)
            p.gemm(cs)
            assert p.right()
    finally:
        p.ctx.free()


@pytest.mark.parametrize("what", ["a shard is missing", "only the epoch before", "nothing"])
def test_what_was_not_delivered_is_waited_for(what):
    p = Problem(3, 200, agg.B_NK)
    try:
        p.ctx.set_wait_limit_us(2000)
        agg.signal_reset(p.ctx)
        if what == "a shard is missing":
            p.deliver(None, [2, 3])
        elif what == "only the epoch before":
            p.deliver(None)
            agg.signal_reset(p.ctx)
        p.gemm(None)
        torch.cuda.synchronize()
        assert agg.agg_status(p.ctx) == agg.ERR_TIMEOUT
    finally:
        p.ctx.free()


def _captured(stream, what):
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=torch.cuda.ExternalStream(stream), capture_error_mode="thread_local"):
        what()
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("rows,N", [(3, 200), (250, 1500)])
def test_epoch_on_the_device(rows, N):
    p = Problem(rows, N, agg.B_NK)
    try:
        ps, cs = p.ctx.streams()
        p.ctx.set_wait_limit_us(2000)
        p.ctx.set_device_epoch(True)
        p.C.fill_(float("nan"))
        agg.signal_reset(p.ctx, cs)
        p.deliver(cs)
        p.gemm(cs)
        assert p.right()
        # a replay moves the epoch on behind the host's back: the copies are of the epoch before
        reset = _captured(cs, lambda: agg.signal_reset(p.ctx, cs))
        agg.signal_reset(p.ctx, cs)
        p.deliver(cs)
        reset.replay()
        torch.cuda.synchronize()
        p.gemm(cs)
        torch.cuda.synchronize()
        assert agg.agg_status(p.ctx) == agg.ERR_TIMEOUT
        # a replay brings the GEMM without the copy
        agg.signal_reset(p.ctx, cs)
        p.deliver(cs)
        gemm = _captured(cs, lambda: p.gemm(cs))
        p.C.fill_(float("nan"))
        gemm.replay()
        assert p.right()
        agg.signal_reset(p.ctx, cs)
        gemm.replay()
        torch.cuda.synchronize()
        assert agg.agg_status(p.ctx) == agg.ERR_TIMEOUT
    finally:
        p.ctx.free()


def test_copies_that_were_only_recorded_are_waited_for():
    p = Problem(250, 1500, agg.B_NK)
    try:
        ps, cs = p.ctx.streams()
        p.deliver(cs)                                      # (what is set up on first use)
        p.gemm(cs)
        assert p.right()
        p.ctx.set_wait_limit_us(2000)
        agg.signal_reset(p.ctx)
        copy = _captured(cs, lambda: p.deliver(cs))
        p.gemm(cs)
        torch.cuda.synchronize()
        assert agg.agg_status(p.ctx) == agg.ERR_TIMEOUT
        copy.replay()
        torch.cuda.synchronize()
        p.C.fill_(float("nan"))
        torch.cuda.synchronize()
        p.gemm(cs)
        assert p.right()
    finally:
        p.ctx.free()


@pytest.mark.parametrize("rows,E,topk,N", [(4, 8, 2, 96), (200, 4, 1, 520), (1500, 8, 2, 1024)])
def test_moe(rows, E, topk, N):
    g = torch.Generator(device="cuda").manual_seed(E)
    T = W * rows
    shards, B = [_ints(g, rows, K) for _ in range(W)], _ints(g, E, N, K)
    ids = torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    flat = ids.reshape(-1).long()
    order = torch.argsort(flat, stable=True)
    X = torch.cat(shards).float()[order // topk]
    want = torch.empty((T * topk, N), device="cuda")
    for e in range(E):
        sel = flat[order] == e
        want[sel] = X[sel] @ B[e].float().t()
    Y = torch.full((T * topk, N), float("nan"), device="cuda")
    tok, seg = torch.empty(T * topk, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 0, rows * K * 2, W)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        agg.signal_reset(ctx)
        torch.cuda.synchronize()
        agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, None)
        agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N, agg.F32, None)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK and torch.equal(Y, want)
    finally:
        ctx.free()
