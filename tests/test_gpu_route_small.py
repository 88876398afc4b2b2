"""The routing of few pairs, which no workgroup shares with another: at the edges of a lane's eight pairs, of a wave and of the largest number
that it takes (and one more, which goes to the other kernel), with one and with the most experts, with ids outside them, for all tokens and for
this rank's alone; and calls of both kinds in turn on one context.  Integer inputs: everything is exact."""
import pytest
import torch

import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu

# tokens, top-k, experts
CASES = [(2, 1, 1), (4, 2, 3), (14, 1, 4096), (170, 3, 64), (254, 4, 8), (2046, 1, 5), (2048, 1, 300), (1024, 2, 64), (682, 3, 7), (684, 3, 7), (2050, 1, 64),
         (512, 4, 2000), (1364, 3, 33), (2048, 2, 1000), (1366, 3, 12)]


@pytest.mark.parametrize("outside", [False, True])
def test_routing_exact(outside):
    W, rank, N, K = 2, 1, 68, 64
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        for T, topk, E in CASES:
            agg.agg_reserve_moe(ctx, T, topk, E, N)
        cs = ctx.streams()[1]
        for T, topk, E in CASES:
            g = torch.Generator(device="cuda").manual_seed(T + E)
            P = T * topk
            ids = torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
            if outside:
                drop = torch.rand((T, topk), device="cuda", generator=g) < 0.2
                ids[drop] = torch.tensor([-1, E, 1 << 30], device="cuda", dtype=torch.int32)[torch.randint(0, 3, (int(drop.sum()),), device="cuda", generator=g)]
            flat = ids.reshape(-1).long()
            inside = (flat >= 0) & (flat < E)
            order = torch.nonzero(inside).reshape(-1)
            order = order[torch.argsort(flat[order], stable=True)]
            n = order.numel()
            lengths = torch.bincount(flat[inside], minlength=E)
            seg_want = torch.cat([lengths.new_zeros(1), lengths.cumsum(0)])
            pos_want = torch.full((P,), -1, device="cuda", dtype=torch.int64)
            pos_want[order] = torch.arange(n, device="cuda")
            H = torch.randint(-2, 3, (P, K), device="cuda", generator=g).to(torch.bfloat16)
            B = torch.randint(-2, 3, (E, N, K), device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)
            gate = torch.randint(1, 3, (T, topk), device="cuda", generator=g).float()
            prod = torch.bmm(B[flat[order]].float(), H[:n].float().unsqueeze(2).contiguous()).squeeze(2)
            rows = torch.zeros((P + 1, N), device="cuda")
            rows[:n] = prod
            Z_want = (rows[pos_want].view(T, topk, N) * gate.unsqueeze(2)).sum(dim=1)
            for Z in (torch.full((T, N), float("nan"), device="cuda"), None):
                Y = torch.full((P, N), float("nan"), device="cuda")
                tok, pos = (torch.full((P,), -7, device="cuda", dtype=torch.int32) for _ in range(2))
                seg = torch.full((E + 1,), -7, device="cuda", dtype=torch.int32)
                slots = [torch.zeros((T // W, N), device="cuda") for _ in range(W)]
                R = torch.full((T // W, N), float("nan"), device="cuda")
                agg.signal_reset(ctx)
                torch.cuda.synchronize()
                agg.signal_set(ctx, 0, cs)
                agg.moe_rs(ctx, T, topk, E, N, K, H, B, ids, gate, Y, tok, seg, pos, slots, Z, R, N, agg.F32, cs, cs)
                torch.cuda.synchronize()
                assert agg.agg_status(ctx) == agg.OK
                assert torch.equal(seg.long(), seg_want), (T, topk, E)
                assert torch.equal(tok[:n].long(), order // topk) and bool((tok[n:] == -7).all()), (T, topk, E)
                assert torch.equal(pos.long(), pos_want), (T, topk, E)
                assert torch.equal(R, Z_want[T // W:]), (T, topk, E)
                if Z is not None:
                    assert torch.equal(Y[:n], prod) and torch.equal(Z[:T // W], Z_want[:T // W]), (T, topk, E)
    finally:
        ctx.free()
