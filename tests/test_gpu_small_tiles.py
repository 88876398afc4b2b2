"""The K-split GEMM kernels that the automatic tile choice takes for small problems, at the sizes where they can go wrong:
one row, one short of and one past a tile, a single piece of K, fewer pieces than waves, a ragged last column block with
aligned and unaligned rows, slices smaller and larger than a tile.  Integer inputs: exact.  (Every tile in every form, with K longer
than its ring and more tiles than workgroups: test_gpu_ks_tiles.py.)"""
import numpy as np
import pytest
import torch

import oracle
import paper_2504_19442_amd as agg
import workloads as wl
from harness import AgGemmRun, dev_bf16, host_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,Ms,K,N,chunks", [
    (1, 1, 64, 16, 1),          # one row, one piece of K (seven of eight waves have none)
    (3, 1, 576, 40, 1),         # 16-row tiles, nine pieces over eight waves
    (2, 17, 192, 99, 1),        # three tiles of 16 rows, odd columns
    (4, 16, 4096, 200, 2),      # 16 x 16 tiles, deep K
    (2, 35, 448, 1500, 1),      # 16 x 32
    (5, 26, 640, 1302, 2),      # 32 x 32, columns not a multiple of four
    (3, 11, 128, 4100, 1),      # 64 x 64, half a tile of rows, two pieces of K
    (2, 260, 448, 1200, 4),     # 64 x 64 over several signals
    (3, 333, 512, 1999, 1),     # 64 x 128, odd columns
    (3, 333, 64, 2001, 3),      # one piece of K
    (2, 33, 64, 6148, 1),       # 64 x 64, the second tile of rows almost empty, a single piece of K
])
def test_ag_gemm_small_shapes_exact(W, Ms, K, N, chunks):
    sh = wl.AgGemmShape(f"ag_small_{W}_{Ms}_{K}_{N}", 21, W, Ms, K, N)
    inp = wl.make_ag_gemm(sh, a_dist=("int", 2), b_dist=("int", 2))
    rank = W - 1
    want = oracle.ag_gemm(inp.shards, inp.B_kn, rank)
    run = AgGemmRun(inp, rank, chunks_per_shard=chunks)
    try:
        for local in (False, True):                       # own shard from T, and in place
            run.ctx.set_local_shard(run.remote[rank] if local else None)
            for consumer_first in (True, False):
                C = run.run(consumer_first=consumer_first).cpu().numpy()
                assert np.array_equal(C.astype(np.float64), want), (local, consumer_first)
        C16 = host_bits(run.run(out_dtype=agg.BF16))
        assert np.array_equal(C16, wl.f32_to_bf16_bits(want.astype(np.float32)))
    finally:
        run.close()


@pytest.mark.parametrize("W,Ms,K,N,chunks", [
    (4, 1, 64, 16, 1), (8, 8, 576, 260, 4), (2, 40, 192, 1500, 2), (3, 100, 320, 2000, 5), (2, 300, 128, 900, 3),
])
def test_gemm_rs_small_shapes_exact(W, Ms, K, N, chunks):
    sh = wl.GemmRsShape(f"rs_small_{W}_{Ms}_{K}_{N}", 22, W, W * Ms, K, N)
    rank = 1
    inp = wl.make_gemm_rs(sh, rank=rank, a_dist=("int", 2), b_dist=("int", 2), slot_dist=("int", 5))
    A = wl.bf16_bits_to_f32(inp.A_loc).astype(np.float64)
    prod = A @ wl.bf16_bits_to_f32(inp.B_kn).astype(np.float64)
    want = prod[rank * Ms:(rank + 1) * Ms] + sum(s.astype(np.float64) for s in inp.peer_slots.values())
    A_d, B_d = dev_bf16(inp.A_loc), dev_bf16(np.ascontiguousarray(inp.B_kn.T))
    ctx = agg.symm_alloc(W, rank, 16, W * chunks)
    try:
        ctx.set_rs_chunks(chunks)
        ps, cs = ctx.streams()
        slots = [torch.from_numpy(inp.peer_slots[w]).cuda() if w != rank else torch.empty((Ms, N), device="cuda") for w in range(W)]
        for other, two_streams in ((True, True), (True, False), (False, True)):
            slots[rank].fill_(float("nan"))
            P = torch.full((W * Ms, N), float("nan"), device="cuda") if other else None
            R = torch.full((Ms, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            for w in range(W):
                for c in range(chunks):
                    if w != rank:
                        agg.signal_set(ctx, w * chunks + c, cs)
            agg.gemm_rs(ctx, W * Ms, N, K, A_d, K, B_d, K, agg.B_NK, slots, P, R, N, agg.F32, ps if two_streams else cs, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert np.array_equal(R.cpu().numpy().astype(np.float64), want)
            if other:
                got = P.cpu().numpy()
                assert np.isnan(got[rank * Ms:(rank + 1) * Ms]).all()            # the own rows went to the slot
                keep = [r for r in range(W * Ms) if not rank * Ms <= r < (rank + 1) * Ms]
                assert np.array_equal(got[keep].astype(np.float64), prod[keep])
    finally:
        ctx.free()


@pytest.mark.parametrize("K,N,ldb,offset", [
    (64, 8, 8, 0),              # one 16-byte piece per row
    (128, 63, 64, 0),           # a ragged last piece, a wave's tile not full
    (192, 130, 136, 0),         # second column tile almost empty, padded rows
    (320, 257, 264, 8),         # base moved by 16 bytes
    (128, 100, 104, 1),         # base not 16-byte aligned
    (64, 65, 65, 0),            # odd leading dimension: every row at another alignment
])
def test_b_given_as_k_by_n_any_alignment_exact(K, N, ldb, offset):
    sh = wl.AgGemmShape(f"ag_kn_{K}_{N}", 23, 2, 24, K, N)
    inp = wl.make_ag_gemm(sh, a_dist=("int", 2), b_dist=("int", 2))
    want = oracle.ag_gemm(inp.shards, inp.B_kn, 0)
    # rows of ldb elements from `offset` on, and not one element more behind the last row's N
    flat = np.full(offset + (K - 1) * ldb + N, 0x7FC0, dtype=np.uint16)           # NaN wherever no element of B is
    for k in range(K):
        flat[offset + k * ldb: offset + k * ldb + N] = inp.B_kn[k]
    B = dev_bf16(flat)
    run = AgGemmRun(inp, 0)
    try:
        agg.agg_reserve_b_kn(run.ctx, N, K)
        C = torch.full((sh.M, N), float("nan"), device="cuda")
        agg.signal_reset(run.ctx)
        agg.ag_producer_emulate(run.ctx, run.remote, None, agg.PRODUCER_KERNEL, 0, run.prod)
        agg.ag_gemm(run.ctx, sh.M, N, K, B.data_ptr() + 2 * offset, ldb, agg.B_KN, C, N, agg.F32, run.prod)
        torch.cuda.synchronize()
        assert agg.agg_status(run.ctx) == agg.OK
        assert np.array_equal(C.cpu().numpy().astype(np.float64), want)
    finally:
        run.close()


@pytest.mark.parametrize("W,tpr,K,N,E,topk", [
    (4, 1, 64, 32, 4, 1),           # one piece of K, a token or none per expert
    (2, 3, 192, 100, 7, 2),         # rows of a tile beyond the segment, ragged columns
    (8, 8, 1024, 130, 16, 2),       # eight rows per expert
    (2, 96, 320, 66, 6, 2),         # segments of 64 rows: some end inside a third tile of 32
    (3, 111, 128, 1999, 5, 3),      # odd columns, the smallest numbered tile
    (8, 128, 64, 260, 8, 2),        # 256 rows per expert, 64 x 64 tiles
])
def test_moe_small_shapes_exact(W, tpr, K, N, E, topk):
    sh = wl.MoeShape(f"moe_small_{tpr}_{K}_{N}", 24, W, tpr, K, N, E, topk)
    inp = wl.make_moe(sh, x_dist=("int", 2), w_dist=("int", 2))
    tok_ref, _, seg_ref = oracle.moe_route(inp.topk_ids, E)
    X = wl.bf16_bits_to_f32(np.concatenate(inp.shards)).astype(np.float64)
    want = np.empty((sh.T * topk, N))
    for e in range(E):
        rows = slice(int(seg_ref[e]), int(seg_ref[e + 1]))
        want[rows] = X[tok_ref[rows]] @ wl.bf16_bits_to_f32(inp.W_ekn[e]).astype(np.float64)
    shards = [dev_bf16(s) for s in inp.shards]
    B = dev_bf16(np.ascontiguousarray(np.transpose(inp.W_ekn, (0, 2, 1))))
    ids = torch.from_numpy(inp.topk_ids).cuda()
    tok = torch.empty(sh.T * topk, device="cuda", dtype=torch.int32)
    seg = torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 0, tpr * K * 2, W)
    try:
        agg.agg_reserve_moe(ctx, sh.T, topk, E, N)
        ps, cs = ctx.streams()
        for call in (agg.ag_moe_gemm, agg.ag_moe_gemm_static):
            for dtype, tdt in ((agg.F32, torch.float32), (agg.BF16, torch.bfloat16)):
                Y = torch.full((sh.T * topk, N), float("nan"), device="cuda", dtype=tdt)
                agg.signal_reset(ctx)
                torch.cuda.synchronize()
                agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
                call(ctx, sh.T, topk, E, N, K, ids, B, tok, seg, Y, N, dtype, cs)
                torch.cuda.synchronize()
                assert agg.agg_status(ctx) == agg.OK
                assert np.array_equal(tok.cpu().numpy(), tok_ref) and np.array_equal(seg.cpu().numpy().astype(np.int64), seg_ref)
                if dtype == agg.F32:
                    assert np.array_equal(Y.cpu().numpy().astype(np.float64), want)
                else:
                    assert np.array_equal(host_bits(Y), wl.f32_to_bf16_bits(want.astype(np.float32)))
    finally:
        ctx.free()


@pytest.mark.parametrize("W,tpr,K,N,E,topk", [(4, 4, 192, 64, 8, 2), (8, 16, 640, 260, 16, 2), (2, 300, 64, 512, 4, 1)])
def test_moe_rs_own_tokens_alone_are_the_same_bits_as_with_all(W, tpr, K, N, E, topk):
    sh = wl.MoeRsShape(f"moers_small_{tpr}_{K}", 25, W, tpr, K, N, E, topk)
    rank = W - 1
    inp = wl.make_moe_rs(sh, rank=rank)
    want = oracle.moe_rs(inp.H, inp.W2_ekn, inp.topk_ids, inp.gate, inp.peer_slots, W, rank)
    P = sh.T * topk
    H, B = dev_bf16(inp.H), dev_bf16(np.ascontiguousarray(np.transpose(inp.W2_ekn, (0, 2, 1))))
    ids, gate = torch.from_numpy(inp.topk_ids).cuda(), torch.from_numpy(inp.gate).cuda()
    tok, pos = (torch.empty(P, device="cuda", dtype=torch.int32) for _ in range(2))
    seg = torch.empty(E + 1, device="cuda", dtype=torch.int32)
    slots = [torch.from_numpy(inp.peer_slots[w]).cuda() if w != rank else torch.empty((tpr, N), device="cuda") for w in range(W)]
    ctx = agg.symm_alloc(W, rank, 16, W)
    try:
        agg.agg_reserve_moe(ctx, sh.T, topk, E, N)
        ps, cs = ctx.streams()
        got = []
        for other, two_streams in ((True, True), (False, True), (True, False)):
            slots[rank].fill_(float("nan"))
            Y = torch.full((P, N), float("nan"), device="cuda")
            Z = torch.full((sh.T, N), float("nan"), device="cuda") if other else None
            R = torch.full((tpr, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            for w in range(W):
                if w != rank:
                    agg.signal_set(ctx, w, cs)
            agg.moe_rs(ctx, sh.T, topk, E, N, K, H, B, ids, gate, Y, tok, seg, pos, slots, Z, R, N, agg.F32, ps if two_streams else cs, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            got.append(R.cpu().numpy())
        rel = np.linalg.norm(got[0] - want) / np.linalg.norm(want)
        assert rel <= 1e-6, rel           # fp32 sums of K = 64 .. 640 products
        for g in got[1:]:
            assert np.array_equal(g.view(np.uint32), got[0].view(np.uint32))
    finally:
        ctx.free()


def test_gemm_rs_own_slice_alone_is_the_same_bits_as_with_all():
    for W, Ms, K, N in ((8, 8, 640, 512), (4, 40, 448, 1500), (2, 300, 320, 900)):
        sh = wl.GemmRsShape(f"rs_bits_{Ms}", 26, W, W * Ms, K, N)
        inp = wl.make_gemm_rs(sh, rank=0)
        A, B = dev_bf16(inp.A_loc), dev_bf16(np.ascontiguousarray(inp.B_kn.T))
        ctx = agg.symm_alloc(W, 0, 16, W)
        try:
            _, cs = ctx.streams()
            slots = [torch.zeros((Ms, N), device="cuda") for _ in range(W)]
            got = []
            for other in (True, False):
                P = torch.zeros((W * Ms, N), device="cuda") if other else None
                R = torch.zeros((Ms, N), device="cuda")
                agg.signal_reset(ctx)
                for w in range(1, W):
                    agg.signal_set(ctx, w, cs)
                agg.gemm_rs(ctx, W * Ms, N, K, A, K, B, K, agg.B_NK, slots, P, R, N, agg.F32, cs, cs)
                torch.cuda.synchronize()
                assert agg.agg_status(ctx) == agg.OK
                got.append(R.cpu().numpy().view(np.uint32))
            assert np.array_equal(got[0], got[1]), (W, Ms)
        finally:
            ctx.free()


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3, 4, 5, 6, 7])
def test_odd_row_widths_every_tile(tile):
    """Rows of C that start at any element: widths that leave 1, 3 and 6 columns behind the last 16 bytes, padded rows whose padding
    stays untouched, and slices whose borders lie inside a block of 32 rows."""
    for W, Ms, K, N, pad in ((2, 150, 128, 331, 0), (1, 270, 64, 517, 1), (3, 45, 192, 262, 3)):
        sh = wl.AgGemmShape(f"ag_odd_{N}", 27, W, Ms, K, N)
        inp = wl.make_ag_gemm(sh, a_dist=("int", 2), b_dist=("int", 2))
        want = oracle.ag_gemm(inp.shards, inp.B_kn, 0)
        run = AgGemmRun(inp, 0)
        try:
            run.ctx.set_tile_config(tile)
            agg.signal_reset(run.ctx)
            agg.ag_producer_emulate(run.ctx, run.remote, None, agg.PRODUCER_KERNEL, 0, run.cons)
            for dtype, tdt in ((agg.F32, torch.float32), (agg.BF16, torch.bfloat16)):
                C = torch.full((sh.M, N + pad), 7.0, device="cuda", dtype=tdt)
                torch.cuda.synchronize()
                agg.ag_gemm(run.ctx, sh.M, N, K, run.B_nk, K, agg.B_NK, C, N + pad, dtype, run.cons)
                torch.cuda.synchronize()
                got = C.float().cpu().numpy()
                ref = want if dtype == agg.F32 else wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(want.astype(np.float32)))
                assert np.array_equal(got[:, :N], ref.astype(np.float32)), (W, Ms, N, dtype)
                assert (got[:, N:] == 7.0).all()
        finally:
            run.close()
    # the product cut into slices of 44 rows, odd width, every slice at a destination of its own
    W, Ms, K, N = 4, 44, 128, 331
    inp = wl.make_gemm_rs(wl.GemmRsShape("rs_odd", 28, W, W * Ms, K, N), a_dist=("int", 2), b_dist=("int", 2))
    prod = wl.bf16_bits_to_f32(inp.A_loc).astype(np.float64) @ wl.bf16_bits_to_f32(inp.B_kn).astype(np.float64)
    A, B = dev_bf16(inp.A_loc), dev_bf16(np.ascontiguousarray(inp.B_kn.T))
    ctx = agg.symm_alloc(W, 0, 16, W)
    try:
        ctx.set_tile_config(tile)
        _, cs = ctx.streams()
        dst = [torch.full((Ms, N), float("nan"), device="cuda") for _ in range(W)]
        torch.cuda.synchronize()
        agg.gemm_rs_scatter(ctx, W * Ms, N, K, A, K, B, K, agg.B_NK, dst, None, None, 1, cs)
        torch.cuda.synchronize()
        got = torch.cat(dst).cpu().numpy().astype(np.float64)
        assert np.array_equal(got, prod)
    finally:
        ctx.free()


@pytest.mark.parametrize("W,tpr,K,N,E,topk", [(2, 8, 2048, 1024, 64, 2), (8, 256, 4096, 1028, 32, 1)])
def test_moe_weights_beyond_the_memory_side_cache_exact(W, tpr, K, N, E, topk):
    # 268 MB of weights, a row or two and 64 rows per expert; small integers, so that fp32 sums are exact in any order
    T = W * tpr
    g = torch.Generator(device="cuda").manual_seed(29)
    shards = [torch.randint(-2, 3, (tpr, K), device="cuda", generator=g).to(torch.bfloat16) for _ in range(W)]
    B = torch.randint(-2, 3, (E, N, K), device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16)
    ids = torch.rand((T, E), device="cuda", generator=g).argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    flat = ids.reshape(-1).long()
    order = torch.argsort(flat, stable=True)
    X = torch.cat(shards)[order // topk].float()
    want = torch.empty((T * topk, N), device="cuda")
    for e in range(E):
        rows = (flat[order] == e).nonzero().reshape(-1)
        if rows.numel():
            want[rows] = X[rows] @ B[e].float().t()
    tok, seg = torch.empty(T * topk, device="cuda", dtype=torch.int32), torch.empty(E + 1, device="cuda", dtype=torch.int32)
    ctx = agg.symm_alloc(W, 0, tpr * K * 2, W)
    try:
        agg.agg_reserve_moe(ctx, T, topk, E, N)
        ps, cs = ctx.streams()
        Y = torch.full((T * topk, N), float("nan"), device="cuda")
        agg.signal_reset(ctx)
        torch.cuda.synchronize()
        agg.ag_producer_emulate(ctx, shards, None, agg.PRODUCER_KERNEL, 0, ps)
        agg.ag_moe_gemm(ctx, T, topk, E, N, K, ids, B, tok, seg, Y, N, agg.F32, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        assert torch.equal(tok.long(), order // topk)
        assert torch.equal(Y, want)
    finally:
        ctx.free()


def test_tuning_a_small_problem_does_not_end_on_a_slower_tile():
    # 16 rows: with the best of the numbered tiles the function takes twice as long as untuned
    W, Ms, K, N = 8, 2, 8192, 3584
    g = torch.Generator(device="cuda").manual_seed(30)
    shards = [torch.randint(-2, 3, (Ms, K), device="cuda", generator=g).to(torch.bfloat16) for _ in range(W)]
    B = torch.randint(-2, 3, (N, K), device="cuda", generator=g).to(torch.bfloat16)
    want = torch.cat(shards).float() @ B.float().t()
    C = torch.full((W * Ms, N), float("nan"), device="cuda")
    ctx, other = agg.symm_alloc(W, 0, Ms * K * 2, W), agg.symm_alloc(W, 0, Ms * K * 2, W)
    try:
        torch.cuda.synchronize()
        res = agg.agg_autotune_ag_gemm(ctx, W * Ms, N, K, B, K, agg.B_NK, C, N, agg.F32, shards, agg.PRODUCER_KERNEL, 3)
        assert res.configs_tried == 24 and (res.tile_config, res.tile_order) == (-1, agg.ORDER_ROTATED)
        assert res.producer_workgroups > 0 and 0.0 < res.best_ms < 1000.0
        assert agg.agg_tune_table_get(W, W * Ms, N, K).tile_config == -1
        assert agg.agg_tune_table_apply(other, W * Ms, N, K)
        for c in (ctx, other):
            ps, cs = c.streams()
            C.fill_(float("nan"))
            agg.signal_reset(c)
            torch.cuda.synchronize()
            agg.ag_producer_emulate(c, shards, None, agg.PRODUCER_KERNEL, 0, ps)
            agg.ag_gemm(c, W * Ms, N, K, B, K, agg.B_NK, C, N, agg.F32, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(c) == agg.OK
            assert torch.equal(C, want)
    finally:
        ctx.free()
        other.free()
        agg.agg_tune_table_clear()
