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
