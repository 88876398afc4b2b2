"""The copy kernel at the edges of its slices: chunks that one, four and eight loads per lane cover, that do so but for 16 bytes, and that
are a multiple of the slice and 16 bytes more, by workgroups of four waves and of one, with fewer workgroups than chunks and more.  T holds
the shards, nothing else in it is touched, and every signal is raised."""
import pytest
import torch

import paper_2504_19442_amd as agg

pytestmark = pytest.mark.gpu


class _Ints:
    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 3}


def _words(ptr, n):
    return torch.as_tensor(_Ints(ptr, n), device="cuda")


# bytes of a chunk, chunks per shard
CHUNKS = [(16, 1), (4096, 1), (4096 + 16, 2), (16384 - 16, 1), (16384, 4), (16384 + 16, 1), (32768 - 16, 2), (32768, 3), (32768 + 16, 1), (65536, 1),
          (65536 + 16, 2), (333 * 1984 * 2, 1), (1 << 20, 1), ((1 << 20) + 48, 4)]


@pytest.mark.parametrize("mode,workgroups", [(agg.PRODUCER_KERNEL, 0), (agg.PRODUCER_KERNEL, 3), (agg.PRODUCER_KERNEL | agg.PRODUCER_NARROW, 0),
                                             (agg.PRODUCER_KERNEL | agg.PRODUCER_NARROW, 5)])
def test_every_byte_of_every_chunk(mode, workgroups):
    W, rank = 3, 1
    for chunk, per_shard in CHUNKS:
        shard = chunk * per_shard
        g = torch.Generator(device="cuda").manual_seed(chunk)
        shards = [torch.randint(-(1 << 31), (1 << 31) - 1, (shard // 4,), device="cuda", generator=g, dtype=torch.int32) for _ in range(W)]
        ctx = agg.symm_alloc(W, rank, shard, W * per_shard)
        try:
            T = _words(ctx.staging, W * shard // 4)
            for _ in range(2):
                T.fill_(7)
                agg.signal_reset(ctx)
                agg.ag_producer_emulate(ctx, shards, None, mode, workgroups, torch.cuda.current_stream())
                torch.cuda.synchronize()
                assert torch.equal(T, torch.cat(shards)), (chunk, per_shard)
                signals = _words(ctx.signals, W * per_shard * agg.SIGNAL_STRIDE).view(-1, agg.SIGNAL_STRIDE)[:, 0]
                assert bool((signals == ctx.epoch).all()), (chunk, per_shard)
        finally:
            ctx.free()
