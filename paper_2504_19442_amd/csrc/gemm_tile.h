// What the GEMM kernels of this library share: the walk over the output tiles (Section 3.7), the wait for the signals of a
// tile's rows, and the count of finished tiles that raises the signals of GEMM + ReduceScatter.
#pragma once
#include "agg_internal.h"

#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "these kernels name gfx950 instructions and registers (MFMA forms, accumulator registers, global->LDS loads)"
#endif

#include <type_traits>
#include <utility>

namespace agg {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(3))) const bf16x8 lds_frag;

// Raw buffer descriptor over `bytes` bytes at p: loads whose per-lane offset is >= bytes return zero, which
// is how rows past the edge of A or B are masked.  0x00020000 = 32-bit data format, no swizzle (gfx9 family).
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// The vector type V at any even address.  Rows of C start wherever its leading dimension puts them; a store through this
// type is one instruction all the same (the hardware allows its address to be unaligned), and rows of any width are
// stored 16 bytes at a time (one element at a time, 4000 x 3267 x 1024 in bf16 took 51 us; 32 like this, 3264 columns 29).
template <class V> struct Unaligned { typedef V type __attribute__((aligned(2))); };
template <class V> using unaligned_t = typename Unaligned<V>::type;

// s_waitcnt immediate that waits only for vmcnt <= n (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]).
__host__ __device__ constexpr int vmcnt_imm(int n) { return (n & 0xF) | (0x7 << 4) | (0xF << 8) | ((n >> 4) << 14); }

// compile-time loop: f(std::integral_constant<int, I>) for I in [0, N)
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

constexpr int BK = 64;                 // bf16 per stage
constexpr int ROW_BYTES = BK * 2;      // 128-byte rows in LDS: one cache line per row and stage
constexpr int UNIT_ROWS = 8;           // one wave-wide 16-byte-per-lane load covers 8 rows

// One output tile: rows [m0, m0 + BM), columns [n0, n0 + BN); rows of A at or past m_lim read as zero, rows of the output
// outside [st_lo, st_hi) are not stored; signals f_lo..f_hi cover its rows of A.
struct TileWork {
    int m0, n0, m_lim, f_lo, f_hi, expert, st_lo, st_hi;
    bool from_local;                   // the tile lies inside this rank's own shard, which is read where the caller keeps it
};

// Tile t of the launch's list; false: nothing of it is wanted.
template <int BM, int BN, bool GROUPED>
__device__ __forceinline__ bool tile_work(const GemmParams& p, int t, TileWork& w)
{
    w.f_lo = 0; w.f_hi = -1; w.expert = 0; w.st_lo = 0; w.from_local = false;
    if constexpr (GROUPED) {
        const MoeTile mt = p.tile_tab[t];
        w.expert = __builtin_amdgcn_readfirstlane(mt.expert);
        w.m0 = __builtin_amdgcn_readfirstlane(mt.m0);
        w.m_lim = __builtin_amdgcn_readfirstlane(mt.m_end);
        w.st_lo = __builtin_amdgcn_readfirstlane(mt.st_lo);
        w.st_hi = __builtin_amdgcn_readfirstlane(mt.st_hi);
        if (w.st_hi <= w.st_lo) return false;     // no row of this tile is wanted (MoE + ReduceScatter without Z_other)
        w.n0 = __builtin_amdgcn_readfirstlane(mt.n_tile) * BN;
        w.f_lo = __builtin_amdgcn_readfirstlane(mt.f_lo);
        w.f_hi = __builtin_amdgcn_readfirstlane(mt.f_hi);
    } else {
        int m_tile, n_tile;
        const int per_panel = p.panel_m * p.tiles_n;
        const int panel = t / per_panel;
        const int pm = min(p.panel_m, p.tiles_m - panel * p.panel_m);
        const int q = t - panel * per_panel;
        const int blk = q / (pm * p.group_n);
        const int r = q - blk * pm * p.group_n;
        const int gn = min(p.group_n, p.tiles_n - blk * p.group_n);
        const int mi = r / gn;
        n_tile = blk * p.group_n + (r - mi * gn);
        const int v = panel * p.panel_m + mi;            // place in the order of m-tiles
        if (p.order == AGG_ORDER_SUBCHUNK) {
            // the local shard, then sub-chunk 0 of every peer (in pull order), sub-chunk 1 of every peer, ...
            if (v < p.tiles_per_shard) {
                m_tile = p.rank * p.tiles_per_shard + v;
            } else {
                const int v2 = v - p.tiles_per_shard;
                const int per_c = (p.world - 1) * p.tiles_per_chunk;
                const int c = v2 / per_c, rem = v2 - c * per_c;
                const int jj = rem / p.tiles_per_chunk, k = rem - jj * p.tiles_per_chunk;
                const int shard = (p.rank + 1 + jj) % p.world;
                m_tile = shard * p.tiles_per_shard + c * p.tiles_per_chunk + k;
            }
        } else {
            m_tile = (p.m_tile_start + v) % p.tiles_m;
        }
        w.m0 = m_tile * BM;
        w.n0 = n_tile * BN;
        w.m_lim = p.M;
        w.st_hi = p.M;
        // a tile that lies inside this rank's own shard reads it where the caller keeps it: nothing to wait for
        w.from_local = p.A_local && w.m0 >= p.local_lo && w.m0 + BM <= p.local_hi;
        if (p.flags && !w.from_local) {
            w.f_lo = w.m0 / p.rows_per_flag;
            w.f_hi = min((min(w.m0 + BM, p.M) - 1) / p.rows_per_flag, p.n_flags - 1);
        }
    }
    return true;
}

// The wait for the signals of a tile's rows (wait + consume_token, Section 2.2), by one wave of the workgroup; nonzero in the
// lanes that gave up.
// The wave polls (lane l takes signals f_lo + l, f_lo + l + 64, ...) and, once it has seen them all, executes
// the acquire: the wave that observed the signals is the wave that orders the loads of A after them.  The
// acquire invalidates this CU's L1 and this XCD's L2 lines of remotely written memory, so that no load of
// A behind it is served from a line cached before the data arrived; one wave does it for the workgroup
// (invalidates from all waves of all CUs queue up behind each other at the L2), and a barrier holds the
// other waves back until it is done.
template <class Params>
__device__ __forceinline__ int poll_signals(const Params& p, int f_lo, int f_hi, int epoch, int lane)
{
    int gave_up = 0;
    for (int f = f_lo + lane; f <= f_hi; f += 64) {
        const int* fp = p.flags + (long long)f * kSignalStride;
        const long long t0 = wall_clock64();
        while (__hip_atomic_load(fp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch) {
            if (__hip_atomic_load(p.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
                wall_clock64() - t0 > p.wait_ticks) {
                gave_up = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    if (gave_up) __hip_atomic_store(p.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return gave_up;
}

// One look at them, by one wave: whether any is still to come.  If none is, the acquire is done as well.
template <class Params>
__device__ __forceinline__ bool signals_missing(const Params& p, int f_lo, int f_hi, int epoch, int lane)
{
    bool missing = false;
    for (int f = f_lo + lane; f <= f_hi; f += 64)
        missing |= __hip_atomic_load(p.flags + (long long)f * kSignalStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch;
    const bool any = __ballot(missing) != 0;
    if (!any) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return any;
}

// The wait for a whole workgroup; true: a wait was given up, and the launch drains (agg_status reports the time-out).
__device__ __forceinline__ bool tile_wait_gave_up(const GemmParams& p, int f_lo, int f_hi, int epoch, int wave, int lane)
{
    int gave_up = 0;
    if (wave == 0) gave_up = poll_signals(p, f_lo, f_hi, epoch, lane);
    return __syncthreads_or(gave_up);
}

// Where row `row` of the output goes, from column n0 on: C, or (GEMM-RS) the destination of its slice; nullptr = not stored.
__device__ __forceinline__ char* out_row(const GemmParams& p, bool grouped, int row, int st_lo, int st_hi, int n0, int esz)
{
    if (row < st_lo || row >= st_hi) return nullptr;
    if (!grouped && p.n_slices) {
        const int w = row / p.slice_rows;
        if (p.slice_dst[w])
            return (char*)p.slice_dst[w] + ((long long)(row - w * p.slice_rows) * p.ldc_slice + n0) * esz;
    }
    return p.C ? (char*)p.C + ((long long)row * p.ldc + n0) * esz : nullptr;
}

// GEMM-RS: count the tile at row m0 for every chunk of every slice it touches; the last tile of a chunk raises the
// chunk's signal (the notify of Algorithm 3: those rows are complete where their reducer will read them).  Called by all
// waves of the workgroup.
template <int BM, class Params>
__device__ __forceinline__ void tile_publish(const Params& p, int m0, int epoch, int tid)
{
    const int w_lo = m0 / p.slice_rows, w_hi = (min(m0 + BM, p.M) - 1) / p.slice_rows;
    bool any = false;
    for (int w = w_lo; w <= w_hi; ++w) any = any || p.slice_flag[w] != nullptr;
    if (any) {
        __builtin_amdgcn_s_waitcnt(0);   // this wave's stores of the tile have reached L2 ...
        __syncthreads();                 // ... and so have every other wave's, before thread 0 publishes them
        if (tid == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const int m_end = min(m0 + BM, p.M);
            for (int w = w_lo; w <= w_hi; ++w) {
                if (!p.slice_flag[w]) continue;
                const int s0 = w * p.slice_rows;                       // first row of slice w
                const int c_lo = (max(m0, s0) - s0) / p.chunk_rows;
                const int c_hi = (min(m_end, s0 + p.slice_rows) - 1 - s0) / p.chunk_rows;
                for (int c = c_lo; c <= c_hi; ++c) {
                    // tiles that touch these rows: their m-tiles times all n-tiles
                    const int r0 = s0 + c * p.chunk_rows;
                    const int mt_lo = r0 / BM, mt_hi = (r0 + p.chunk_rows - 1) / BM;
                    const int target = (mt_hi - mt_lo + 1) * p.tiles_n;
                    int* ctr = p.slice_ctr + w * p.slice_chunks + c;
                    const int prev = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
                    if (prev == target - 1) {
                        __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_store(p.slice_flag[w] + c * kSignalStride, epoch, __ATOMIC_RELEASE,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }
    }
}

}  // namespace agg
