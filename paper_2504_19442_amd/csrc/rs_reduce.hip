// ReduceScatter reduction (Algorithm 3, stream 2): R = sum over w = 0..W-1 of slot_w, fp32, added in
// that order starting from +0 whatever order the slots arrive in, so the result is bit-identical
// across arrival orders.  Each workgroup waits (acquire) for slot w's signal before its first read of
// slot w.  The kernel is bandwidth bound: W reads and one write per element, 16 bytes per lane per
// access; streaming stores.
// What is left beside the bytes is the start: the signals are looked at by the lanes of one wave side by side (one after
// the other by one thread, each a trip to memory, cost 4 us per workgroup), and where all slots are there the first
// block is loaded like every other.
// Once all slots are there, loads never stop: the register of a slot's value is loaded again, for the next block, as soon as the value
// has been added, so that W x RU loads per lane are in flight throughout, where a block that is loaded whole, added and stored drains them in
// between.  Few workgroups then do better than many (reduce_workgroups), and 64 registers are enough for every world size: a
// workgroup fits beside any GEMM of this library.  Blocks loaded whole, and this, us per call with the kernel that raises the signals, slots not
// touched lately: eight slots of 1024 x 8192 55.0 and 50.8, of 1000 x 8000 57.5 and 52.7, four 39.7 and 32.2, three 37.3 and 26.8, two 27.6 and 21.7;
// behind the GEMM of gemm_rs, 8192 x 8192 x 3584, 430 and 417.  In row chunks, with 4 / 16 chunks of 1024 x 8192: eight slots
// 56.1 / 60.4 and 52.5 / 52.7, four 42.8 / 50.6 and 32.1 / 32.3, two 32.2 / 34.4 and 21.5 / 21.6.
// ReduceArgs::own: behind the GEMM on its own stream there is nothing to wait for in the own slot, and its signals are raised here, by one
// workgroup, instead of by every tile or by a kernel of its own (api.hip: gemm_rs, moe_rs).
#include "agg_internal.h"

namespace agg {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;


// Wave 0 of a workgroup waits for the n signals f(0) .. f(n - 1), one lane each (64 at a time): they are looked at side by
// side, each look is a trip to memory.  f < 0: nothing to wait for.  False in the lanes that gave up.
template <class F>
__device__ inline bool wait_signals(const ReduceCommon& a, int n, int epoch, int lane, F&& f)
{
    bool ok = true;
    for (int k = lane; k < n; k += 64) {
        const long long at = f(k);
        if (at < 0) continue;
        const int* fp = a.flags + at * kSignalStride;
        const long long t0 = wall_clock64();
        while (__hip_atomic_load(fp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch) {
            if (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > a.wait_ticks) {
                __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = false;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return ok;
}

template <class I>      // I: an integer type that holds the number of float4
__device__ inline void store_out(const ReduceCommon& a, I i, f32x4 v)
{
    long long off;
    if (a.row_vec4) {
        const I row = i / (I)a.row_vec4;
        off = row * a.ldr + (long long)(i - row * (I)a.row_vec4) * 4;
    } else {
        off = (long long)i * 4;
    }
    if (a.r_is_f32) {
        __builtin_nontemporal_store(v, (f32x4*)((float*)a.R + off));
    } else {
        bf16x4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = (__bf16)v[k];
        *(bf16x4*)((__bf16*)a.R + off) = o;
    }
}

// The signals that stand for what was complete when this kernel started.
__device__ inline void raise_own(const ReduceCommon& a, int epoch, int tid)
{
    if (a.own >= 0 && blockIdx.x == 0 && tid < a.chunks)
        __hip_atomic_store(a.flags + ((long long)a.own * a.flag_step + tid) * kSignalStride, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool NT>      // NT: the slots are read past the caches (launch_reduce)
__device__ inline f32x4 load_in(const f32x4* p) { return NT ? __builtin_nontemporal_load(p) : *p; }

// WT slots below 2 GiB, loads never stop.  RU: float4 per lane in flight per slot.  THREADS: reduce_shape.
// A slot that arrives in row chunks: a workgroup walks the rows upwards and looks at the signals again before the first load of a chunk that
// had not arrived when it last looked, while its loads of the chunk before are still on their way; the reduction of the first
// chunks runs while the later ones are still being produced.
// (64 registers, asked for as such: asked for as eight waves per SIMD, the scalars would have to fit too, and spill.)
template <int WT, int RU, bool NT, int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_num_vgpr(64))) void reduce_flow_kernel(const ReduceSlots<8> a)
{
    const int tid = threadIdx.x;
    const int epoch = a.epoch_ptr ? __hip_atomic_load(a.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : a.epoch;
    const unsigned stride = gridDim.x * THREADS;     // (32-bit offsets: at most 2^16 workgroups)
    const unsigned count = (unsigned)a.n_vec4;
    const bool chunked = a.chunks > 1;
    raise_own(a, epoch, tid);
    __shared__ int s_seen;
    int seen = 0;               // units 0 .. seen - 1 have arrived: slots, or row chunks of every slot (uniform over the workgroup)
    // Wave 0 looks at as many signals at once as it has lanes, until units 0 .. want - 1 have arrived; one acquire (an L2 invalidate) covers
    // all that have.  False: the wait was given up.
    auto look = [&](int want) {
        bool ok = true;
        if (tid < 64) {
            const int units = chunked ? a.chunks : WT, per = chunked ? 64 / WT : 64;
            const int unit = chunked ? tid / WT : tid, slot = chunked ? tid % WT : tid;
            int upto = seen;
            const long long t0 = wall_clock64();
            for (;;) {
                const int u = upto + unit, w = chunked ? slot : u;
                const bool here = unit >= per || u >= units || w == a.own
                    || __hip_atomic_load(a.flags + ((long long)w * a.flag_step + (chunked ? u : 0)) * kSignalStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= epoch;
                const unsigned long long missing = ~__ballot(here);
                upto += missing ? (int)__builtin_ctzll(missing) / (chunked ? WT : 1) : per;
                if (upto >= units) { upto = units; break; }
                if (!missing) continue;
                if (upto >= want) break;
                if (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > a.wait_ticks) {
                    ok = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (!ok && tid == 0) __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 0) s_seen = upto;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        if (__syncthreads_or(!ok)) return false;
        seen = s_seen;
        __syncthreads();
        return true;
    };
    unsigned pos = blockIdx.x * THREADS;             // this workgroup's next block
    if (pos >= count) return;
    look(0);
    if (!chunked && seen < WT) {
        // slots still to arrive: the first blocks take them one by one in the order of Algorithm 3
        f32x4 acc[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < WT; ++w) {
            if (w >= seen && !look(w + 1)) return;
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                const unsigned i = pos + u * stride + tid;
                acc[u] = acc[u] + (i < count ? ((const f32x4*)a.slot[w])[i] : f32x4{0.f, 0.f, 0.f, 0.f});      // one fp32 rounding each
            }
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const unsigned i = pos + u * stride + tid;
            if (i < count) store_out(a, i, acc[u]);
        }
        pos += RU * stride;
        if (pos >= count) return;
    }
    unsigned ready;                               // float4 of every slot that have arrived
    auto arrived = [&] { ready = chunked && seen < a.chunks ? (unsigned)(seen * a.chunk_vec4) : count; };
    // The blocks p, p + stride, .. of one pass, as far as there are any, have arrived.
    auto wait_for = [&](unsigned p) {
        if (ready == count || p >= count) return true;
#pragma unroll
        for (int u = 1; u < RU; ++u)
            if (p + stride < count) p += stride;
        const unsigned end = p + THREADS < count ? p + THREADS : count;
        if (end <= ready) return true;
        if (!look((int)((end - 1) / (unsigned)a.chunk_vec4) + 1)) return false;
        arrived();
        return true;
    };
    arrived();
    if (!wait_for(pos)) return;
    f32x4 v[RU][WT];
    auto fetch = [&](int u, int w, unsigned p) {  // past the end: zero
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.slot[w]), 0, count * 16u, 0x00020000);
        v[u][w] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (p + tid) * 16u, 0, NT ? 2 : 0));
    };
#pragma unroll
    for (int u = 0; u < RU; ++u)
#pragma unroll
        for (int w = 0; w < WT; ++w) fetch(u, w, pos + u * stride);
    for (;;) {
        if (!wait_for(pos + RU * stride)) return;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < WT; ++w) {
                sum = sum + v[u][w];
                asm volatile("" : "+v"(sum));        // added before its register is loaded again
                fetch(u, w, pos + RU * stride);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (pos + tid < count) store_out(a, pos + tid, sum);
            pos += stride;
            if (pos >= count) return;
        }
    }
}

// Any world size: every block is loaded whole, four slots at a time.
template <int RU, bool NT>   // RU = float4 per lane per slot and block
__global__ __launch_bounds__(256) void reduce_kernel(const ReduceArgs a)
{
    const int tid = threadIdx.x;
    const int W = a.W;
    const int epoch = a.epoch_ptr ? __hip_atomic_load(a.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : a.epoch;
    const long long stride = (long long)gridDim.x * 256;
    raise_own(a, epoch, tid);
    __shared__ int s_upto;
    int seen = 0;                      // slots 0..seen-1 are known to have arrived (uniform over the workgroup)
    // Wave 0 looks at all slots' signals at once (lane w at slot w's) until slots 0 .. want - 1 have arrived; one acquire (an
    // L2 invalidate) covers all that have.  False: the wait was given up.
    auto look = [&](int want) {
        bool ok = true;
        if (tid < 64) {
            const int* fp = a.flags + (long long)(tid < W ? tid : 0) * a.flag_step * kSignalStride;
            const long long t0 = wall_clock64();
            int upto;
            for (;;) {
                const bool here = tid >= W || tid == a.own || __hip_atomic_load(fp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= epoch;
                const unsigned long long missing = ~__ballot(here);
                upto = missing ? (int)__builtin_ctzll(missing) : W;
                if (upto >= want) break;
                if (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > a.wait_ticks) {
                    ok = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (!ok && tid == 0) __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 0) s_upto = upto;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        if (__syncthreads_or(!ok)) return false;
        seen = s_upto;
        __syncthreads();
        return true;
    };
    int chunks_seen = 0;               // chunked slots: row chunks 0..chunks_seen-1 of EVERY slot have arrived
    for (long long base = (long long)blockIdx.x * 256 + tid; base - tid < a.n_vec4; base += stride * RU) {
        f32x4 acc[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (a.chunks > 1) {
            // Slots that arrive in row chunks, each chunk with a signal of its own: a workgroup walks the rows
            // upwards, so before it enters a chunk it waits for that chunk (and any it skipped) of all W slots,
            // and the reduction of the first chunks runs while the later ones are still being produced.
            long long last = (base - tid) + (long long)(RU - 1) * stride + 255;
            if (last >= a.n_vec4) last = a.n_vec4 - 1;
            const int need = (int)(last / a.chunk_vec4);
            if (need >= chunks_seen) {
                bool ok = true;
                if (tid < 64) {
                    const int c0 = chunks_seen;
                    ok = wait_signals(a, (need - c0 + 1) * W, epoch, tid, [&](int k) {
                        return k % W == a.own ? -1ll : (long long)(k % W) * a.flag_step + c0 + k / W;
                    });
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                }
                if (__syncthreads_or(!ok)) return;
                chunks_seen = need + 1;
            }
        } else if (seen < W) {
            look(0);                   // when all have arrived, the block is loaded whole below
        }
        if (a.chunks <= 1 && seen < W) {
            // slots still to arrive: take them one by one in the order of Algorithm 3
            for (int w = 0; w < W; ++w) {
                if (w >= seen && !look(w + 1)) return;
                const f32x4* s = (const f32x4*)a.slot[w];
#pragma unroll
                for (int u = 0; u < RU; ++u) {
                    const long long i = base + u * stride;
                    const f32x4 v = (i < a.n_vec4) ? s[i] : f32x4{0.f, 0.f, 0.f, 0.f};
                    acc[u] = acc[u] + v;                              // R = R + T[w], one fp32 rounding each
                }
            }
        } else {
            // every slot has arrived: all loads of the block first, then the additions in slot order
            for (int w0 = 0; w0 < W; w0 += 4) {          // four slots at a time
                f32x4 v[4][RU];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (w0 + k >= W) break;
                    const f32x4* s = (const f32x4*)a.slot[w0 + k];
#pragma unroll
                    for (int u = 0; u < RU; ++u) {
                        const long long i = base + u * stride;
                        v[k][u] = (i < a.n_vec4) ? load_in<NT>(s + i) : f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (w0 + k >= W) break;
#pragma unroll
                    for (int u = 0; u < RU; ++u) acc[u] = acc[u] + v[k][u];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const long long i = base + u * stride;
            if (i < a.n_vec4) store_out(a, i, acc[u]);
        }
    }
}

// RU: about eight loads in flight per lane.  At most 64 registers each (the second launch bound; 59 in any world): the GEMM's waves leave 64
// per SIMD lane, so a reducer runs on the same compute units.
template <bool NT>
static void launch_reduce_nt(const ReduceArgs& a, ReduceShape shape, hipStream_t stream)
{
    const dim3 grid(shape.workgroups), wg(shape.threads);
    if (!reduce_flows(a.W, a.n_vec4)) {
        hipLaunchKernelGGL((reduce_kernel<2, NT>), grid, wg, 0, stream, a);
        return;
    }
    // (arguments for eight slots where there are no more: every launch carries them.  Always for 64, here and in gemm_ks.h, and this, us per
    // call that the host's launches bound: 17.3 and 16.5, 64 x 8192 x 3584 on one stream 20.6 and 20.5)
    ReduceSlots<8> e;
    static_cast<ReduceCommon&>(e) = a;
    for (int w = 0; w < 8; ++w) e.slot[w] = a.slot[w];
    auto flow = [&](auto threads_c) {
        constexpr int T = decltype(threads_c)::value;
        switch (a.W) {
            case 8: hipLaunchKernelGGL((reduce_flow_kernel<8, 1, NT, T>), grid, wg, 0, stream, e); break;
            case 4: hipLaunchKernelGGL((reduce_flow_kernel<4, 2, NT, T>), grid, wg, 0, stream, e); break;
            case 3: hipLaunchKernelGGL((reduce_flow_kernel<3, 3, NT, T>), grid, wg, 0, stream, e); break;
            default: hipLaunchKernelGGL((reduce_flow_kernel<2, 4, NT, T>), grid, wg, 0, stream, e); break;
        }
    };
    if (shape.threads == 192) flow(std::integral_constant<int, 192>{});
    else flow(std::integral_constant<int, 256>{});
}

// From 256 MB of slots on, the size of the memory-side cache, the loads carry the streaming hint.  Both sides, us, ordinary loads
// and hint, eight slots of 1024 x 8192 (268 MB): slots not touched lately 54.6 and 50.4, slots that have just been written
// 47.7 and 47.7; 336 MB: 68.3 and 62.1, just written 65.0 and 64.0.  Four slots of 2048 x 8192 59.3 and 55.6, just written 49.0 and
// 47.5; two 70.5 and 68.3, just written 60.0 and 57.6.  What loses is a loop that reads one and the same slots without anyone
// writing them in between (part of them then stays in that cache): 45.2 and 48.1, with four slots 46.9 and 53.3; from
// 336 MB on that, too, is faster with the hint (64.6 and 60.0).  Below the line the hint gains on slots not touched lately (134 MB
// 31.1 and 28.1, 201 MB 42.2 and 39.2) and loses up to 5 % on ones that the cache holds, which slots of that size usually
// are: ordinary loads.
hipError_t launch_reduce(const ReduceArgs& a, ReduceShape shape, hipStream_t stream)
{
    if (a.n_vec4 * 16 * a.W >= (256ll << 20)) launch_reduce_nt<true>(a, shape, stream);
    else launch_reduce_nt<false>(a, shape, stream);
    return hipGetLastError();
}

}  // namespace agg
