"""The calls that a tensor-parallel program makes to this library, as cases that can be timed and compared.

Five operations through the public entry points of the package: AllGather-GEMM (`ag_gemm`, with the emulated arrival
that feeds it), GEMM + ReduceScatter (`gemm_rs`), the ReduceScatter reducer alone (`rs_reduce`), the MoE AllGather
grouped GEMM (`ag_moe`) and MoE + ReduceScatter (`moe_rs`).  Sizes are those of the workloads of this repository (the
8B- and 70B-MLP-shaped layers, Table 4, Table 5), from a decode step of a few tokens to a whole prefill, and ragged ones.

Small calls go on the caller's current stream, one kernel after the other; large ones put arrival and computation on
the context's two streams and join them, which is what overlapping is for.
"""
import math

import torch

import paper_2504_19442_amd as agg

TORCH_TYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
AGG_TYPE = {"bf16": agg.BF16, "f32": agg.F32}


def listed():
    return [
        # A decode step of the 8B-MLP layer: 16 tokens on 8 ranks, the smallest call, latency and the weights' bytes.
        {"name": "ag_gemm_decode_16", "op": "ag_gemm", "W": 8, "rank": 0, "rows": 2, "K": 4096, "N": 3584, "out": "bf16",
         "layout": "nk", "signals": 1, "overlap": False},
        # The same step of the 70B-MLP layer with a full serving batch of 128 sequences.
        {"name": "ag_gemm_batch_128", "op": "ag_gemm", "W": 8, "rank": 0, "rows": 16, "K": 8192, "N": 7168, "out": "bf16",
         "layout": "nk", "signals": 1, "overlap": False},
        # Nothing a multiple of a tile: three ranks, odd rows, odd columns, fp32 output (a head or a router's logits).
        {"name": "ag_gemm_ragged", "op": "ag_gemm", "W": 3, "rank": 1, "rows": 333, "K": 1984, "N": 1999, "out": "f32",
         "layout": "nk", "signals": 1, "overlap": False},
        # A prefill chunk of 1024 tokens on 4 ranks with the weights stored [K][N], as a checkpoint may hold them.
        {"name": "ag_gemm_chunk_kn", "op": "ag_gemm", "W": 4, "rank": 0, "rows": 256, "K": 4096, "N": 3584, "out": "bf16",
         "layout": "kn", "signals": 1, "overlap": False},
        # The 8B-MLP workload: prefill of 4096 tokens, arrival beside the GEMM, a single round of tiles.
        {"name": "ag_gemm_8b_mlp", "op": "ag_gemm", "W": 8, "rank": 0, "rows": 512, "K": 4096, "N": 3584, "out": "bf16",
         "layout": "nk", "signals": 4, "overlap": True},
        # The 70B-MLP workload, the benchmark's headline and the largest call.
        {"name": "ag_gemm_70b_mlp", "op": "ag_gemm", "W": 8, "rank": 0, "rows": 1024, "K": 8192, "N": 7168, "out": "bf16",
         "layout": "nk", "signals": 4, "overlap": True},
        # The second half of the MLP in a decode step of 64 tokens: partial product, scatter, bf16 result.
        {"name": "gemm_rs_decode_64", "op": "gemm_rs", "W": 8, "rows": 8, "K": 3584, "N": 8192, "out": "bf16",
         "other": True, "overlap": False},
        # The second half of the MLP at its full size, the reducer on a stream of its own.
        {"name": "gemm_rs_full", "op": "gemm_rs", "W": 8, "rows": 1024, "K": 3584, "N": 8192, "out": "f32",
         "other": True, "overlap": True},
        # The reducer alone at the same size: what the rank does when the partial products come from elsewhere.
        {"name": "rs_reduce_full", "op": "rs_reduce", "W": 8, "rows": 1024, "N": 8192, "out": "f32"},
        # MoE layer of Table 4: 8192 tokens, 64 experts, top 2.
        {"name": "ag_moe_full", "op": "ag_moe", "W": 8, "rows": 1024, "K": 4096, "N": 2048, "E": 64, "topk": 2, "out": "bf16",
         "signals": 4, "overlap": True},
        # The same layer in a decode step of 64 tokens: nearly every expert is asked for, by a row or two.
        {"name": "ag_moe_decode_64", "op": "ag_moe", "W": 8, "rows": 8, "K": 4096, "N": 2048, "E": 64, "topk": 2, "out": "bf16",
         "signals": 1, "overlap": False},
        # Second MoE layer of Table 5: 8192 tokens, a rank's K slice, every token's partial sums.
        {"name": "moe_rs_full", "op": "moe_rs", "W": 8, "rows": 1024, "K": 192, "N": 2048, "E": 64, "topk": 2, "out": "f32",
         "other": True, "overlap": True},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["ag_gemm", "ag_gemm", "ag_gemm", "gemm_rs", "gemm_rs", "rs_reduce", "ag_moe", "ag_moe", "moe_rs"])
    W = rng.choice([2, 3, 4, 8, 8])
    out = rng.choice(["bf16", "bf16", "f32"])
    rows = _log(rng, 2, 1024)                          # per rank
    large = W * rows >= 1024
    if op == "ag_gemm":
        return {"op": op, "W": W, "rank": rng.randrange(W), "rows": rows, "K": 64 * _log(rng, 4, 128), "N": _log(rng, 96, 7168),
                "out": out, "layout": rng.choice(["nk", "nk", "nk", "kn"]), "signals": 4 if rows % 4 == 0 and large else 1,
                "overlap": large}
    if op == "gemm_rs":
        return {"op": op, "W": W, "rows": rows, "K": 64 * _log(rng, 2, 56), "N": 4 * _log(rng, 24, 2048), "out": out,
                "other": rng.random() < 0.8, "overlap": large}
    if op == "rs_reduce":
        return {"op": op, "W": W, "rows": rows, "N": 4 * _log(rng, 24, 2048), "out": out}
    E = _log(rng, 4, 64)
    topk = rng.choice([1, 2, 2, 4])
    if op == "ag_moe":
        return {"op": op, "W": W, "rows": rows, "K": 64 * _log(rng, 4, 64), "N": _log(rng, 96, 2048), "E": E, "topk": topk,
                "out": out, "signals": 4 if rows % 4 == 0 and large else 1, "overlap": large}
    return {"op": op, "W": W, "rows": rows, "K": 64 * _log(rng, 1, 16), "N": 4 * _log(rng, 24, 512), "E": E, "topk": topk,
            "out": out, "other": rng.random() < 0.8, "overlap": large}


class State(dict):
    """What a program keeps between calls; the context goes back to the library when the program drops it."""

    def __del__(self):
        if self.get("ctx") is not None:
            self["ctx"].free()
            self["ctx"] = None


def _inputs(c, seed):
    """The case's inputs, from the seed alone: activations in [-1, 1), weights N(0, 0.02), partial sums N(0, 1)."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def uniform(*shape):
        return torch.empty(shape, device="cuda", dtype=torch.bfloat16).uniform_(-1.0, 1.0, generator=g)

    def weights(*shape):
        return torch.empty(shape, device="cuda", dtype=torch.bfloat16).normal_(0.0, 0.02, generator=g)

    W, rows, N, op = c["W"], c["rows"], c["N"], c["op"]
    T, d = W * rows, {}
    if op == "ag_gemm":
        d["shards"] = [uniform(rows, c["K"]) for _ in range(W)]
        d["B"] = weights(N, c["K"]) if c["layout"] == "nk" else weights(c["K"], N)
    elif op == "gemm_rs":
        d["A"], d["B"] = uniform(T, c["K"]), weights(N, c["K"])
    elif op == "ag_moe":
        d["shards"] = [uniform(rows, c["K"]) for _ in range(W)]
        d["B"] = weights(c["E"], N, c["K"])
    elif op == "moe_rs":
        d["H"], d["B"] = uniform(T * c["topk"], c["K"]), weights(c["E"], N, c["K"])
        gate = torch.rand((T, c["topk"]), device="cuda", generator=g) + 0.1
        d["gate"] = (gate / gate.sum(dim=1, keepdim=True)).contiguous()
    if op in ("ag_moe", "moe_rs"):
        keys = torch.rand((T, c["E"]), device="cuda", generator=g)
        d["ids"] = keys.argsort(dim=1)[:, : c["topk"]].to(torch.int32).contiguous()      # distinct experts per token
    if op in ("gemm_rs", "rs_reduce", "moe_rs"):
        d["slots"] = [torch.randn((rows, N), device="cuda", generator=g) for _ in range(W)]
    return d


class _Words:
    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 3}


def prepare(case, seed):
    s = State(_inputs(case, seed))
    c = s["case"] = dict(case)
    W, rows, N, op = c["W"], c["rows"], c["N"], c["op"]
    T = W * rows
    gathers = op in ("ag_gemm", "ag_moe")
    per_rank = c["signals"] if gathers else 1
    ctx = s["ctx"] = agg.symm_alloc(W, c.get("rank", 0), rows * c["K"] * 2 if gathers else 16, W * per_rank)
    s["prod"], s["cons"] = (torch.cuda.ExternalStream(x) for x in ctx.streams())
    s["go"], s["done_a"], s["done_b"] = torch.cuda.Event(), torch.cuda.Event(), torch.cuda.Event()
    if op == "ag_gemm":
        s["C"] = torch.empty((T, N), device="cuda", dtype=TORCH_TYPE[c["out"]])
        if c["layout"] == "kn":
            agg.agg_reserve_b_kn(ctx, N, c["K"])
        s["mode"] = agg.PRODUCER_KERNEL
        if c["overlap"]:
            # as the benchmark runs it: the own shard read in place and copied last, and the narrow copy kernel where
            # the GEMM runs for more than one round of tiles
            ctx.set_local_shard(s["shards"][c["rank"]])
            s["mode"] |= agg.PRODUCER_LOCAL_LAST
            if (T + 255) // 256 * ((N + 223) // 224) >= 512:
                s["mode"] |= agg.PRODUCER_NARROW
    else:
        s["mode"] = agg.PRODUCER_KERNEL
    if op in ("ag_moe", "moe_rs"):
        P = T * c["topk"]
        agg.agg_reserve_moe(ctx, T, c["topk"], c["E"], N)
        s["tok"] = torch.empty((P,), device="cuda", dtype=torch.int32)
        s["seg"] = torch.empty((c["E"] + 1,), device="cuda", dtype=torch.int32)
        s["pos"] = torch.empty((P,), device="cuda", dtype=torch.int32)
        s["Y"] = torch.empty((P, N), device="cuda", dtype=TORCH_TYPE[c["out"]] if op == "ag_moe" else torch.float32)
    if not gathers:
        s["R"] = torch.empty((rows, N), device="cuda", dtype=TORCH_TYPE[c["out"]])
        s["other"] = torch.zeros((T, N), device="cuda") if c.get("other") else None
        # the signal words of the slots that come from elsewhere: for the reducer alone all, else those of ranks 1, 2, ..
        words = torch.as_tensor(_Words(ctx.signals, W * agg.SIGNAL_STRIDE), device="cuda").view(W, agg.SIGNAL_STRIDE)
        s["peer_signals"] = words[0 if op == "rs_reduce" else 1:, 0]
    return s


def _on_streams(s, first, second):
    """first(stream) beside second(stream), both behind and in front of the current stream's work; where the case does
    not overlap them, one after the other on the current stream."""
    cur = torch.cuda.current_stream()
    if not s["case"]["overlap"]:
        first(cur)
        second(cur)
        return
    a, b = s["prod"], s["cons"]
    s["go"].record(cur)
    a.wait_event(s["go"])
    b.wait_event(s["go"])
    first(a)
    second(b)
    s["done_a"].record(a)
    s["done_b"].record(b)
    cur.wait_event(s["done_a"])
    cur.wait_event(s["done_b"])


def _reduce_streams(s):
    """Streams of the product and of the reducer, started behind the current stream; and the join."""
    cur = torch.cuda.current_stream()
    if not s["case"]["overlap"]:
        return cur, cur, lambda: None
    a, b = s["prod"], s["cons"]
    s["go"].record(cur)
    a.wait_event(s["go"])
    b.wait_event(s["go"])

    def join():
        s["done_a"].record(a)
        s["done_b"].record(b)
        cur.wait_event(s["done_a"])
        cur.wait_event(s["done_b"])

    return a, b, join


def run(s):
    c, ctx = s["case"], s["ctx"]
    W, rows, N, op = c["W"], c["rows"], c["N"], c["op"]
    T, out = W * rows, AGG_TYPE[c["out"]]
    agg.signal_reset(ctx)
    if op == "ag_gemm":
        K = c["K"]
        ldb, layout = (K, agg.B_NK) if c["layout"] == "nk" else (N, agg.B_KN)
        _on_streams(s, lambda st: agg.ag_producer_emulate(ctx, s["shards"], None, s["mode"], 0, st),
                    lambda st: agg.ag_gemm(ctx, T, N, K, s["B"], ldb, layout, s["C"], N, out, st))
        return {"C": s["C"]}
    if op == "ag_moe":
        _on_streams(s, lambda st: agg.ag_producer_emulate(ctx, s["shards"], None, s["mode"], 0, st),
                    lambda st: agg.ag_moe_gemm(ctx, T, c["topk"], c["E"], N, c["K"], s["ids"], s["B"], s["tok"], s["seg"], s["Y"],
                                               N, out, st))
        return {"Y": s["Y"], "sorted_token": s["tok"], "offsets": s["seg"]}
    s["peer_signals"].fill_(ctx.epoch)                 # the peers' slots have arrived: one kernel raises their signals
    if op == "rs_reduce":
        agg.rs_reduce(ctx, rows, N, s["slots"], s["R"], N, out, 0, torch.cuda.current_stream())
        return {"R": s["R"]}
    a, b, join = _reduce_streams(s)
    if op == "gemm_rs":
        agg.gemm_rs(ctx, T, N, c["K"], s["A"], c["K"], s["B"], c["K"], agg.B_NK, s["slots"], s["other"], s["R"], N, out, a, b)
        got = {"R": s["R"], "own": s["slots"][0]}
    else:
        agg.moe_rs(ctx, T, c["topk"], c["E"], N, c["K"], s["H"], s["B"], s["ids"], s["gate"], s["Y"], s["tok"], s["seg"], s["pos"],
                   s["slots"], s["other"], s["R"], N, out, a, b)
        got = {"R": s["R"], "own": s["slots"][0], "sorted_token": s["tok"], "offsets": s["seg"], "positions": s["pos"]}
    join()
    if s["other"] is not None:
        got["other"] = s["other"]
    return got


def work(c):
    W, rows, N, op = c["W"], c["rows"], c["N"], c["op"]
    T, esz = W * rows, 2 if c["out"] == "bf16" else 4
    if op == "rs_reduce":
        return {"bytes": (W * 4 + esz) * rows * N, "flops": W * rows * N}
    K = c["K"]
    if op == "ag_gemm":
        return {"bytes": 2 * K * (T + N) + T * N * esz, "flops": 2 * T * N * K}
    # the slots of the other ranks are read, the own one is written; the result is written
    reduced = W * rows * N * 4 + rows * N * esz
    other = (T - rows) * N * 4 if c.get("other") else 0
    wanted = T if c.get("other") or op == "ag_moe" else rows        # rows of the product that are asked for
    if op == "gemm_rs":
        return {"bytes": 2 * K * (wanted + N) + other + reduced, "flops": 2 * wanted * N * K + W * rows * N}
    P = wanted * c["topk"]
    experts = c["E"] * (1.0 - (1.0 - c["topk"] / c["E"]) ** wanted)    # expected number with at least one token
    if op == "ag_moe":
        return {"bytes": 2 * K * (T + experts * N) + P * N * esz + 8 * P, "flops": 2 * P * N * K}
    return {"bytes": 2 * K * (P + experts * N) + other + reduced + 16 * T * c["topk"], "flops": 2 * P * N * (K + 1) + W * rows * N}


def tolerance(c):
    if c["op"] == "rs_reduce":
        # 2-norm against 64 bits 5.6e-8 for the fp32 sum of eight slots
        return {"rel": 7e-3, "max": 1.6e-2} if c["out"] == "bf16" else {"rel": 3e-7, "max": 2e-6}
    # bf16 results: one rounding to 8 bits, 2-norm 1.7e-3 against 64 bits, at most 2^-8 of a value: times four
    # fp32 results: up to 8192 products summed in fp32, 2-norm 2.6e-7 to 5e-7 against 64 bits: times four
    return {"rel": 7e-3, "max": 1.6e-2} if c["out"] == "bf16" else {"rel": 2e-6, "max": 2e-5}


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    W, rows, N, op = c["W"], c["rows"], c["N"], c["op"]
    T = W * rows
    if op == "ag_gemm":
        A = torch.cat(d["shards"]).double()
        return {"C": A @ (d["B"].double().t().contiguous() if c["layout"] == "nk" else d["B"].double())}
    slots = [x.double() for x in d.get("slots", [])]
    if op == "rs_reduce":
        return {"R": sum(slots)}
    if op == "gemm_rs":
        prod = d["A"].double() @ d["B"].double().t().contiguous()
        own = prod[:rows].contiguous()
        got = {"R": own + sum(slots[1:]), "own": own}
        if c["other"]:
            prod[:rows] = 0.0                          # the own slice's rows are not written there
            got["other"] = prod
        return got
    # MoE: the (token, slot) pairs by (expert, token, slot)
    topk, E = c["topk"], c["E"]
    flat = d["ids"].reshape(-1).long()
    order = torch.argsort(flat, stable=True)
    ends = torch.cumsum(torch.bincount(flat, minlength=E), 0)
    offsets = torch.cat([ends.new_zeros(1), ends])
    at = offsets.tolist()
    X = torch.cat(d["shards"])[order // topk] if op == "ag_moe" else d["H"]
    Y = torch.empty((T * topk, N), device="cuda", dtype=torch.float64)
    for e in range(E):
        if at[e + 1] > at[e]:
            Y[at[e]:at[e + 1]] = X[at[e]:at[e + 1]].double() @ d["B"][e].double().t().contiguous()
    tokens = (order // topk).to(torch.int32)
    if op == "ag_moe":
        return {"Y": Y, "sorted_token": tokens, "offsets": offsets.to(torch.int32)}
    pos = torch.empty_like(order)
    pos[order] = torch.arange(T * topk, device="cuda")
    Z = (Y[pos].view(T, topk, N) * d["gate"].double().unsqueeze(2)).sum(dim=1)
    own = Z[:rows].contiguous()
    got = {"R": own + sum(slots[1:]), "own": own, "sorted_token": tokens, "offsets": offsets.to(torch.int32),
           "positions": pos.to(torch.int32)}
    if c["other"]:
        Z[:rows] = 0.0
        got["other"] = Z
    return got
