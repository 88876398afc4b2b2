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


# blocks of 256 or 192 float4 per workgroup: fewer than the unrolled loop holds, as many, one more, several laps; whole and partial last blocks
@pytest.mark.parametrize("W", [2, 3, 4, 8])
@pytest.mark.parametrize("n_vec4,workgroups", [(1, 0), (255, 1), (256, 3), (257, 1), (513, 2), (256 * 4, 1), (256 * 5 - 3, 1), (256 * 23 + 1, 5), (256 * 1100 + 77, 0),
                                                (191, 0), (193, 1), (192 * 2, 3), (192 * 7 + 5, 2), (192 * 256 * 3 + 11, 0)])
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


# Row chunks: shorter than a block, not whole blocks, several laps long; the last chunks' signals raised while the reducer waits for them
@pytest.mark.parametrize("W", [2, 3, 4, 8])
@pytest.mark.parametrize("rows,chunks,workgroups", [(16, 16, 1), (300, 3, 1), (256 * 9, 4, 2), (256 * 41 - 5, 7, 3), (256 * 300, 16, 0)])
def test_reducer_chunk_lengths_bit_exact(W, rows, chunks, workgroups):
    rows = rows // chunks * chunks
    g = torch.Generator(device="cuda").manual_seed(7600 + W)
    data = [torch.randn((rows, 4), device="cuda", generator=g) * 10.0 ** w for w in range(W)]
    want = torch.zeros((rows, 4), device="cuda")
    for x in data:
        want = want + x
    ctx = agg.symm_alloc(W, 0, 16, W * 16)
    try:
        ctx.set_rs_chunks(chunks)
        ps, cs = ctx.streams()
        prod = torch.cuda.ExternalStream(ps)
        for late in range(min(chunks, 3)):               # chunks that arrive behind the launch
            slots = [torch.full((rows, 4), float("nan"), device="cuda") for _ in range(W)]
            R = torch.full((rows, 8), 3.0, device="cuda")
            agg.signal_reset(ctx)
            torch.cuda.synchronize()

            def deliver(c):
                part = slice(c * (rows // chunks), (c + 1) * (rows // chunks))
                for w in range(W):
                    with torch.cuda.stream(prod):
                        slots[w][part].copy_(data[w][part])
                    agg.signal_set(ctx, w * 16 + c, prod)

            for c in range(chunks - late):
                deliver(c)
            prod.synchronize()
            agg.rs_reduce(ctx, rows, 4, slots, R, 8, agg.F32, workgroups, cs)
            for c in range(chunks - late, chunks):
                deliver(c)
            torch.cuda.synchronize()
            assert agg.agg_status(ctx) == agg.OK
            assert torch.equal(R[:, :4].contiguous().view(torch.int32), want.view(torch.int32)) and bool((R[:, 4:] == 3.0).all())
    finally:
        ctx.free()


@pytest.mark.parametrize("W", [2, 8])
def test_reducer_of_chunked_slots_takes_the_time_of_whole_ones(W):
    # 1024 x 8192, us with one signal per slot and with four: 21.5 and 21.5, 51.7 and 52.5 (with a loop that drains at every block 41.5, 84.4)
    Ms, N = 1024, 8192
    slots = [[torch.zeros((Ms, N), device="cuda") for _ in range(W)] for _ in range(8 // W + 1)]
    R = torch.empty((Ms, N), device="cuda")
    ctx = agg.symm_alloc(W, 0, 16, W * 4)
    try:
        agg.signal_reset(ctx)
        for k in range(W * 4):
            agg.signal_set(ctx, k, None)

        def median_us(chunks):
            ctx.set_rs_chunks(chunks)
            times = []
            for _ in range(9):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                for k in range(20):
                    agg.rs_reduce(ctx, Ms, N, slots[k % len(slots)], R, N, agg.F32, 0, None)
                b.record()
                b.synchronize()
                times.append(a.elapsed_time(b) * 50.0)
            return sorted(times)[4]

        median_us(1)
        whole, four = median_us(1), median_us(4)
        assert agg.agg_status(ctx) == agg.OK
        assert four <= 1.3 * whole, (whole, four)
    finally:
        ctx.free()


@pytest.mark.parametrize("W,n_vec4", [(2, (1 << 27) - 1), (2, 1 << 27), (3, (1 << 27) + 300)])
def test_reducer_on_both_sides_of_slots_of_2_gib_bit_exact(W, n_vec4):
    slots = [torch.empty((n_vec4, 4), device="cuda") for _ in range(W)]
    for w, x in enumerate(slots):
        x.view(-1).copy_(torch.arange(n_vec4 * 4, device="cuda", dtype=torch.int32).mul_(w + 1).bitwise_and_(0xffff))       # whole numbers: exact
    R = torch.full((n_vec4, 4), float("nan"), device="cuda")
    ctx = agg.symm_alloc(W, 0, 16, W)
    try:
        agg.signal_reset(ctx)
        for w in range(W):
            agg.signal_set(ctx, w, None)
        agg.rs_reduce(ctx, n_vec4, 4, slots, R, 4, agg.F32, 0, None)
        torch.cuda.synchronize()
        assert agg.agg_status(ctx) == agg.OK
        for x in slots:
            R -= x
        assert bool((R == 0.0).all())
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


@pytest.mark.parametrize("tile,W", [(6, 2), (6, 3), (6, 4), (4, 6), (6, 8)])
def test_a_gemm_launched_behind_a_waiting_reducer_feeds_it(tile, W):
    """The reducer is launched first, with the library's own grid, and waits for all slots; the GEMM that produces them comes
    afterwards on another stream, on large tiles, and has to find room."""
    Ms, N, K = 64 * (12 // W), 8192, 64              # 3072 to 512 blocks of the reducer: two and more for every CU
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
