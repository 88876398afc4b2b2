"""The reducer for world sizes with and without an unrolled kernel of their own: all slots there before it starts, and slots
that come while it waits, in ascending and descending order; bit-exact against the ordered fp32 sum."""
import numpy as np
import pytest
import torch

import oracle
import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,Ms,N", [(3, 40, 52), (4, 1, 4), (6, 24, 100), (7, 65, 36), (9, 16, 64), (16, 33, 1024), (64, 5, 12)])
def test_reducer_world_sizes_bit_exact(W, Ms, N):
    rng = np.random.default_rng(7300 + W)
    data = [(rng.standard_normal((Ms, N)) * 10.0 ** rng.integers(-3, 5, size=(Ms, N))).astype(np.float32) for _ in range(W)]
    want = oracle.rs_reduce_f32(data)
    dev = [torch.from_numpy(d).cuda() for d in data]
    ctx = agg.symm_alloc(W, 0, 16, W)
    try:
        ps, cs = ctx.streams()
        prod = torch.cuda.ExternalStream(ps)
        for order in (None, list(range(W)), list(reversed(range(W)))):
            slots = [torch.full((Ms, N), float("nan"), device="cuda") for _ in range(W)]
            R = torch.full((Ms, N), float("nan"), device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()

            def deliver(w):
                with torch.cuda.stream(prod):
                    slots[w].copy_(dev[w])
                agg.signal_set(ctx, w, prod)

            if order is None:
                for w in range(W):
                    deliver(w)
                prod.synchronize()
            agg.rs_reduce(ctx, Ms, N, slots, R, N, agg.F32, 0, cs)
            for w in order or []:
                deliver(w)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert np.array_equal(R.cpu().numpy().view(np.uint32), want.view(np.uint32)), order
    finally:
        ctx.free()


# blocks of 256 float4 per workgroup: fewer than the unrolled loop holds, as many, one more, several laps; whole and partial last blocks
@pytest.mark.parametrize("W", [2, 3, 4, 8])
@pytest.mark.parametrize("n_vec4,workgroups", [(1, 0), (255, 1), (256, 3), (257, 1), (513, 2), (256 * 4, 1), (256 * 5 - 3, 1), (256 * 23 + 1, 5), (256 * 1100 + 77, 0)])
def test_reducer_loop_lengths_bit_exact(W, n_vec4, workgroups):
    g = torch.Generator(device="cuda").manual_seed(7500 + W)
    slots = [torch.randn((n_vec4, 4), device="cuda", generator=g) * 10.0 ** w for w in range(W)]
    want = torch.zeros((n_vec4, 4), device="cuda")
    for s in slots:
        want = want + s
    ctx = agg.symm_alloc(W, 0, 16, W)
    try:
        _, cs = ctx.streams()
        agg.signal_reset(ctx)
        for w in range(W):
            agg.signal_set(ctx, w, cs)
        for ldr, dtype in ((4, torch.float32), (8, torch.float32), (12, torch.bfloat16)):
            R = torch.full((n_vec4 + 1, ldr), 3.0, device="cuda", dtype=dtype)
            torch.cuda.synchronize()
            agg.rs_reduce(ctx, n_vec4, 4, slots, R, ldr, agg.F32 if dtype == torch.float32 else agg.BF16, workgroups, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(R[:-1, :4], want.to(dtype))
            assert bool((R[:, 4:] == 3.0).all()) and bool((R[-1] == 3.0).all())
    finally:
        ctx.free()


@pytest.mark.parametrize("W,Ms,N,ldr", [(8, 1024, 8192, 8192), (16, 1024, 4100, 4104), (3, 2048, 11000, 11000), (2, 4096, 8188, 8188)])
def test_reducer_slots_beyond_the_memory_side_cache_bit_exact(W, Ms, N, ldr):
    # 256 MB of slots and more (the last: just below); the reference adds the slots in order, one fp32 rounding each
    g = torch.Generator(device="cuda").manual_seed(7400 + W)
    slots = [torch.randn((Ms, N), device="cuda", generator=g) for _ in range(W)]
    want = torch.zeros((Ms, N), device="cuda")
    for s in slots:
        want = want + s
    ctx = agg.symm_alloc(W, 0, 16, W)
    try:
        _, cs = ctx.streams()
        agg.signal_reset(ctx)
        for w in range(W):
            agg.signal_set(ctx, w, cs)
        R = torch.full((Ms, ldr), 3.0, device="cuda")
        torch.cuda.synchronize()
        agg.rs_reduce(ctx, Ms, N, slots, R, ldr, agg.F32, 0, cs)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        assert torch.equal(R[:, :N].contiguous().view(torch.int32), want.view(torch.int32))
        assert bool((R[:, N:] == 3.0).all())
    finally:
        ctx.free()


@pytest.mark.parametrize("tile,W", [(6, 2), (6, 3), (6, 4), (4, 6)])
def test_a_gemm_launched_behind_a_waiting_reducer_feeds_it(tile, W):
    """The reducer is launched first, with the library's own grid, and waits for all slots; the GEMM that produces them comes
    afterwards on another stream, on large tiles, and has to find room."""
    Ms, N, K = 64 * (12 // W), 8192, 64              # 3072 to 1024 blocks of the reducer: more than two for every CU
    g = torch.Generator(device="cuda").manual_seed(7500 + W)
    A = torch.randint(-2, 3, (W * Ms, K), device="cuda", generator=g).to(torch.bfloat16)
    B = torch.randint(-2, 3, (N, K), device="cuda", generator=g).to(torch.bfloat16)
    P = A.float() @ B.float().t()
    want = P.reshape(W, Ms, N).sum(dim=0)             # small integers: exact in any order
    ctx = agg.symm_alloc(W, 0, 16, W)
    try:
        ctx.set_tile_config(tile)
        ps, cs = ctx.streams()
        slots = [torch.full((Ms, N), float("nan"), device="cuda") for _ in range(W)]
        R = torch.full((Ms, N), float("nan"), device="cuda")
        signals = [ctx.signals + w * agg.SIGNAL_STRIDE * 4 for w in range(W)]
        for reducer_first in (False, True):            # (the first run also gets the kernels loaded)
            agg.signal_reset(ctx)
            torch.cuda.synchronize()
            if reducer_first:
                agg.rs_reduce(ctx, Ms, N, slots, R, N, agg.F32, 0, cs)
            agg.gemm_rs_scatter(ctx, W * Ms, N, K, A, K, B, K, agg.B_NK, slots, None, signals, 0, ps)
            if not reducer_first:
                agg.rs_reduce(ctx, Ms, N, slots, R, N, agg.F32, 0, cs)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(R, want)
    finally:
        ctx.free()
