// The GEMM kernels for small and narrow problems, where the waves of a workgroup split K instead of the tile's rows.
//
// gemm_ks_kernel: wave w of S computes the whole BM x BN tile over its own 64-wide pieces of K (piece w, w + S, ...), streams
// them through an LDS ring of its own (NST stages; no barrier, only its own loads are waited for) and meets the others
// once, at the end, when the S partial tiles are added up through LDS in wave order.
// gemm_km_kernel: for tiles whose stage is too large for a ring per wave; all waves share the ring (one barrier per stage of
// 64), two groups of NW waves take half of the stage's K each, and the waves of a group take a part of the columns each.
//
// What bounds such a problem is how soon, how many and how often bytes are asked for, not the matrix pipes: a few rows of
// A against all of B.  So the tile is small enough that every compute unit has one, up to 144 KiB of loads are on their way
// per compute unit, every byte is read from LDS once (gemm_ks) or twice (gemm_km) and not by all waves, and B's first stages
// are asked for before the signals are looked at (looking takes 2 to 3 us: the poll, the L2 invalidate, a barrier).
// Operands go through LDS although no wave shares them: a load in the MFMA's fragment layout (consecutive lanes on
// different rows) runs at 16 B/clk per compute unit, whole 128-byte lines at 57.  What a workgroup does before its first
// load counts as much as the loads (10 % to 30 % of a launch here): the launch's arguments are one compact struct, and no
// integer is divided on the way (multipliers come from the host): 10.0 -> 8.5 us at 16 x 3584 x 4096.
// The time left is B from HBM (5.4 to 6.4 TB/s) plus A through the load path (118 KB/us per compute unit): the two add up, the
// path holds only about 24 KiB of misses and hits queue behind them.  What is not near any bound is the start: every instance
// spills 30 to 110 scalar registers (each slot's stage bound and descriptor are lifted out of the tile loop).
//
// Measured against the 128x128 tile of the large kernel (us per GEMM, B not in cache): 16 x 3584 x 4096 24.9 -> 8.5 (16x16
// tiles), 64 x 8192 x 3584 33.3 -> 18.5 (64x32), 128 x 7168 x 8192 74.6 -> 42 (64x64), 999 x 1999 x 1984 21 -> 15.6 (64x128).
// KN: a B stored [K][N], read in place by gemm_km_kernel (64x64, 64x128, 128x128): no transposed copy, which costs a kernel, its bytes twice and
// an event.  Transposing and GEMM, and in place, us: 1024 x 3584 x 4096 49.6 -> 38.6 (128x128), 376 x 5160 x 1984 29.7 -> 17.8 (64x128),
// 84 x 240 x 704 12.2 -> 7.6 (64x64).  Of these, us per call with the copy, the same weights again and again, without and with: an instance per cache
// policy of B's loads 1024 x 3584 x 4096 40.7 and 39.1, x 1024 18.9 and 18.2, 256 x 4096 x 4096 (64x64) 25.1 and 23.2, 512 x 3584 x 4096 (64x128)
// 30.1 and 29.5; in the 128x128 tile parts of 64x64 per wave instead of 128x32 (x 4096) 40.1 and 39.1, and four stages ahead instead
// of three 40.0 and 39.1.
#pragma once
#include "gemm_tile.h"
#include "ks_stage.h"

namespace agg {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_;

// what the rows of the output are
enum KsKind { KS_PLAIN, KS_SLICED, KS_GROUPED };      // one matrix; GEMM + ReduceScatter's slices; MoE segments

// Quotient by a divisor known to the host: exact for n * d < 2^32 (div_mul).
__host__ __device__ inline unsigned div_mul(unsigned d) { return d <= 1 ? 0u : (unsigned)(((1ull << 32) + d - 1) / d); }
__device__ __forceinline__ int div_by(int n, unsigned mul) { return mul ? (int)__umulhi((unsigned)n, mul) : n; }

struct KsParams {
    const uint16_t *A, *A_local, *B;
    void* C;
    int lda, ldb, ldc;                    // elements
    int M, N, KC;                         // KC = K / 64
    int tiles_m, total_tiles, grid, m_tile_start;
    unsigned tiles_m_mul, flag_mul;
    int local_lo, local_hi;
    const int* flags;
    const int* epoch_ptr;
    int* err;
    long long wait_ticks;
    int epoch, n_flags, c_is_f32;
    int b_streams;                        // B's loads carry the streaming hint (launch_ks)
    // KS_GROUPED
    const int* row_index;
    const MoeTile* tile_tab;
    const int* n_tiles_dev;
    long long b_group_stride;
    unsigned a_bytes;
};

// KS_SLICED: as in GemmParams, for up to WORLD slices (every launch carries them)
template <int WORLD>
struct KsSlices {
    int M, tiles_n, slice_rows, slice_chunks, chunk_rows, ldc_slice;
    unsigned slice_mul;
    int* slice_ctr;
    void* slice_dst[WORLD];
    int* slice_flag[WORLD];
};
struct KsNoSlices {};

template <int BM, int BN, int S, int NST>
struct KsCfg {
    static constexpr int A_UNITS = BM / UNIT_ROWS, B_UNITS = BN / UNIT_ROWS;
    static constexpr int L = A_UNITS + B_UNITS;              // loads of a stage (one wave)
    static constexpr int STAGE = (BM + BN) * ROW_BYTES;      // bytes of a stage
    static constexpr int RING = S * NST * STAGE;
    static constexpr int PITCH = BN + 4;                     // floats per row of a partial tile in LDS
    static constexpr int RED = S * BM * PITCH * 4;
    static constexpr int LDS_BYTES = RING > RED ? RING : RED;
    static constexpr int RB = BM / 16, CB = BN / 16;
    static_assert(BM % 16 == 0 && BN % 16 == 0 && (NST - 1) * L <= 63 && LDS_BYTES <= 159 * 1024, "tile");
};

// Tile t of the launch's list: where it is, and the signals that cover its rows of A; false: nothing of it is wanted.
template <int BM, int BN, KsKind KIND>
__device__ __forceinline__ bool ks_tile(const KsParams& p, int t, TileWork& w)
{
    w.m_lim = 0; w.f_lo = 0; w.f_hi = -1; w.expert = 0; w.st_lo = 0; w.from_local = false;
    if constexpr (KIND == KS_GROUPED) {
        const MoeTile mt = p.tile_tab[t];
        w.expert = __builtin_amdgcn_readfirstlane(mt.expert);
        w.m0 = __builtin_amdgcn_readfirstlane(mt.m0);
        w.m_lim = __builtin_amdgcn_readfirstlane(mt.m_end);
        w.st_lo = __builtin_amdgcn_readfirstlane(mt.st_lo);
        w.st_hi = __builtin_amdgcn_readfirstlane(mt.st_hi);
        w.n0 = __builtin_amdgcn_readfirstlane(mt.n_tile) * BN;
        w.f_lo = __builtin_amdgcn_readfirstlane(mt.f_lo);
        w.f_hi = __builtin_amdgcn_readfirstlane(mt.f_hi);
        return w.st_hi > w.st_lo;
    } else {
        // the m-tiles of one column block side by side, the one of the first row first
        const int n_tile = div_by(t, p.tiles_m_mul);
        int m_tile = t - n_tile * p.tiles_m + p.m_tile_start;
        if (m_tile >= p.tiles_m) m_tile -= p.tiles_m;
        w.m0 = m_tile * BM;
        w.n0 = n_tile * BN;
        w.st_hi = p.M;
        w.from_local = p.A_local && w.m0 >= p.local_lo && w.m0 + BM <= p.local_hi;
        if (p.flags && !w.from_local) {
            w.f_lo = div_by(w.m0, p.flag_mul);
            w.f_hi = min(div_by(min(w.m0 + BM, p.M) - 1, p.flag_mul), p.n_flags - 1);
        }
        return true;
    }
}

// The wait for a tile's signals by wave 0, and what the other waves see of it: true = a wait was given up.  `behind` is
// what wave 0 does between its wait and the barrier.
template <class F>
__device__ __forceinline__ bool ks_wait(const KsParams& p, const TileWork& w, int* s_gave_up, int wave, int lane, F&& behind)
{
    if (wave == 0) {
        const int epoch = p.epoch_ptr ? __hip_atomic_load(p.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : p.epoch;
        const bool any = __ballot(poll_signals(p, w.f_lo, w.f_hi, epoch, lane)) != 0;
        if (lane == 0) *s_gave_up = any;
        behind();
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);                            // lgkmcnt(0): the word is written
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    return *s_gave_up != 0;
}

// The sum of NP partial tiles in LDS (rows of PITCH floats), in that order, to memory.
template <int BM, int BN, int NP, int THREADS, KsKind KIND, class SL>
__device__ __forceinline__ void ks_store(const KsParams& p, const SL& sl, const TileWork& w, const float* red, int tid)
{
    constexpr int PITCH = BN + 4;
    const int n_valid = min(BN, p.N - w.n0);
    auto store = [&](auto tag) {
        using T = decltype(tag);
        typedef __attribute__((__vector_size__(4 * sizeof(T)))) T Tx4;
        // where row r of the tile goes; nullptr = not stored
        auto row_at = [&](int r) -> T* {
            const int row = w.m0 + r;
            if (row < w.st_lo || row >= w.st_hi) return nullptr;
            if constexpr (KIND == KS_SLICED) {
                const int sw = div_by(row, sl.slice_mul);
                if (T* d = (T*)sl.slice_dst[sw]) return d + (long long)(row - sw * sl.slice_rows) * sl.ldc_slice + w.n0;
                if (!p.C) return nullptr;
            }
            return (T*)p.C + (long long)row * p.ldc + w.n0;
        };
        for (int idx = tid; idx < BM * BN / 4; idx += THREADS) {
            const int r = idx / (BN / 4), c = idx % (BN / 4) * 4;
            T* dst = row_at(r);
            if (!dst || c >= n_valid) continue;
            f32x4_ v = *(const f32x4_*)(red + r * PITCH + c);
#pragma unroll
            for (int k = 1; k < NP; ++k) v = v + *(const f32x4_*)(red + (k * BM + r) * PITCH + c);
            if (c + 4 <= n_valid) {
                *(unaligned_t<Tx4>*)(dst + c) = Tx4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
            } else {                           // the ragged end of the row
                dst[c] = (T)v[0];
                if (c + 1 < n_valid) dst[c + 1] = (T)v[1];
                if (c + 2 < n_valid) dst[c + 2] = (T)v[2];
            }
        }
    };
    if (p.c_is_f32) store(float{}); else store(__bf16{});
}

// Asks for all of the launch's arguments at once: fetched where they are used they are two trips to memory in a row (0.2 us of
// 4.5 to 19 us kernels).
__device__ __forceinline__ void ks_fetch_params(const KsParams& p)
{
    asm volatile("" ::"s"(p.A), "s"(p.A_local), "s"(p.B), "s"(p.C), "s"(p.lda), "s"(p.KC), "s"(p.tiles_m), "s"(p.tiles_m_mul), "s"(p.flags),
                 "s"(p.err), "s"(p.n_flags), "s"(p.wait_ticks), "s"(p.local_lo));
}

// Private rings.
template <int BM, int BN, int S, int NST, KsKind KIND, class SL>
__global__ __launch_bounds__(S * 64)
void gemm_ks_kernel(const KsParams p, const SL sl)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using C_ = KsCfg<BM, BN, S, NST>;
    constexpr int L = C_::L, RB = C_::RB, CB = C_::CB, PITCH = C_::PITCH;
    constexpr bool GROUPED = KIND == KS_GROUPED;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    __shared__ int s_gave_up;
    ks_fetch_params(p);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the LDS layout of a stage is that of the large kernel: rows of 128 bytes, 16-byte chunk c of row r in slot c ^ ((r >> 1) & 7)
    const int ld_row = lane >> 3;
    const int ld_chunk_even = (lane & 7) ^ ((lane >> 4) & 7);
    const int ld_chunk_odd = (lane & 7) ^ ((4 + (lane >> 4)) & 7);
    int fr_off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) fr_off[h] = (lane & 15) * ROW_BYTES + (((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) << 4);
    const unsigned lds_wave = (unsigned)(unsigned long)(lds_byte*)LDS_PTR(lds) + wave * (NST * C_::STAGE);

    const int KC = p.KC;
    const int n_st = KC > wave ? (KC - wave + S - 1) / S : 0;      // this wave's stages
    const int total_tiles = GROUPED ? *p.n_tiles_dev : p.total_tiles;
    const int G = p.grid, g = blockIdx.x;
    const int g0 = (G & 7) == 0 ? (g & 7) * (G >> 3) + (g >> 3) : g;      // neighbouring tiles go to one XCD
    const unsigned lda2 = (unsigned)p.lda * 2u, ldb2 = (unsigned)p.ldb * 2u;

    for (int t = g0; t < total_tiles; t += G) {
        TileWork w;
        if (!ks_tile<BM, BN, KIND>(p, t, w)) continue;
        const int m0 = w.m0, n0 = w.n0;
        const bool gated = p.flags && w.f_hi >= w.f_lo;

        const uint16_t* a_base = GROUPED ? p.A
                               : w.from_local ? p.A_local + (long long)(m0 - p.local_lo) * p.lda : p.A + (long long)m0 * p.lda;
        const uint16_t* b_base = p.B + (GROUPED ? (long long)w.expert * p.b_group_stride : 0ll) + (long long)n0 * p.ldb;
        const unsigned a_bytes = GROUPED ? p.a_bytes : (unsigned)min(BM, p.M - m0) * lda2;
        const unsigned b_bytes = (unsigned)min(BN, p.N - n0) * ldb2;
        unsigned ld_off[L];
        if constexpr (GROUPED) {
            // the tokens' rows first: what they are is on its way before anything else is asked for
#pragma unroll
            for (int u = 0; u < C_::A_UNITS; ++u) {
                const int row = m0 + u * UNIT_ROWS + ld_row;
                ld_off[u] = row < w.m_lim ? (unsigned)(p.row_index ? p.row_index[row] : row) : 0xFFFFFFFFu;
            }
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int u = GROUPED ? C_::A_UNITS : 0; u < L; ++u) {
            const int chunk = (u & 1) ? ld_chunk_odd : ld_chunk_even;
            ld_off[u] = u < C_::A_UNITS ? (unsigned)(u * UNIT_ROWS + ld_row) * lda2 + (unsigned)(chunk * 16)
                                        : (unsigned)((u - C_::A_UNITS) * UNIT_ROWS + ld_row) * ldb2 + (unsigned)(chunk * 16);
        }
        // the loads of this wave's stage s into ring slot `slot`, B's rows or A's; a stage past the end takes an empty
        // descriptor: nothing is fetched, and the count of outstanding loads stays the same on every path
        auto issue = [&](int s, auto slot_c, auto is_a_c) {
            constexpr int slot = decltype(slot_c)::value;
            constexpr bool is_a = decltype(is_a_c)::value;
            constexpr int u0 = is_a ? 0 : C_::A_UNITS, n = is_a ? C_::A_UNITS : C_::B_UNITS;
            const int c = wave + s * S;
            const KsStage st = ks_stage(c, KC, ROW_BYTES, is_a ? a_bytes : b_bytes);
            const __amdgpu_buffer_rsrc_t rs = make_rsrc(is_a ? a_base : b_base, st.bytes);
            auto load = [&](auto aux_c) {
                static_for<n>([&](auto u_c) {
                    constexpr int u = u0 + decltype(u_c)::value;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_byte*)(unsigned long)(lds_wave + slot * C_::STAGE + u * 1024), 16,
                                                             ld_off[u], st.k_off, 0, decltype(aux_c)::value);
                });
            };
            if (!is_a && p.b_streams) load(std::integral_constant<int, 2>{});      // 2 = nt
            else load(std::integral_constant<int, 0>{});
        };
        using IsA = std::true_type;
        using IsB = std::false_type;
        // B does not wait for any signal: its first stages are on their way while wave 0 looks at the signals
        if (wave != 0 || !gated) static_for<NST>([&](auto j_c) { issue(decltype(j_c)::value, j_c, IsB{}); });
        if (gated && ks_wait(p, w, &s_gave_up, wave, lane, [&] { static_for<NST>([&](auto j_c) { issue(decltype(j_c)::value, j_c, IsB{}); }); })) {
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // the launch drains; agg_status reports the time-out
            return;
        }
        if constexpr (GROUPED) {
            // rows past the segment end get an offset outside the descriptor and load as zero
#pragma unroll
            for (int u = 0; u < C_::A_UNITS; ++u) {
                const unsigned tok = ld_off[u];
                ld_off[u] = tok != 0xFFFFFFFFu ? tok * lda2 + (unsigned)(((u & 1) ? ld_chunk_odd : ld_chunk_even) * 16) : 0xFFFFFF00u;
            }
        }
        static_for<NST>([&](auto j_c) { issue(decltype(j_c)::value, j_c, IsA{}); });

        f32x4_ acc[RB][CB];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) acc[i][j] = f32x4_{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < n_st; s0 += NST) {
            static_for<NST>([&](auto j_c) {
                constexpr int slot = decltype(j_c)::value;
                const int s = s0 + slot;
                if (s >= n_st) return;
                asm volatile("" ::: "memory");
                // stage s has landed (the first NST stages were asked for as all of B, then all of A)
                if (s0 == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1 - slot) * C_::A_UNITS + slot * L));
                else __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * L));
                __builtin_amdgcn_sched_barrier(0);
                bf16x8 fa[2][RB], fb[2][CB];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const unsigned at = lds_wave + slot * C_::STAGE + fr_off[h];
#pragma unroll
                    for (int j = 0; j < CB; ++j) fb[h][j] = *(lds_frag*)(unsigned long)(at + (RB + j) * 2048);
#pragma unroll
                    for (int i = 0; i < RB; ++i) fa[h][i] = *(lds_frag*)(unsigned long)(at + i * 2048);
                }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0xC07F);                        // the fragments are in registers: the slot is free
                __builtin_amdgcn_sched_barrier(0);
                issue(s + NST, j_c, IsB{});
                issue(s + NST, j_c, IsA{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int j = 0; j < CB; ++j)
#pragma unroll
                        for (int i = 0; i < RB; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j], fa[h][i], acc[i][j], 0, 0, 0);
            });
        }

        // ---- the S partial tiles into LDS, and their sum, in wave order, to memory
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));              // (the loads past the end write zeros into the ring)
        __syncthreads();
        float* const red = (float*)lds;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
                *(f32x4_*)(red + (wave * BM + i * 16 + (lane & 15)) * PITCH + j * 16 + 4 * (lane >> 4)) = acc[i][j];
        __syncthreads();
        ks_store<BM, BN, S, S * 64, KIND>(p, sl, w, red, tid);
        if constexpr (KIND == KS_SLICED) {
            const int epoch = p.epoch_ptr ? __hip_atomic_load(p.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : p.epoch;
            tile_publish<BM>(sl, m0, epoch, tid);
        }
        __syncthreads();                       // the ring is free again
    }
#else
    (void)p; (void)sl;
#endif
}

// One ring, shared: stages of 64 x (BM + BN), the waves split a stage's K in two and the columns in NW.
// WM: the NW parts are WM parts of the rows times NW / WM of the columns.
template <int BM, int BN, int NW, int NST, int WM = 1>
struct KmCfg {
    static constexpr int S = 2 * NW;                         // waves: two halves of a stage's K times NW parts of the tile
    static constexpr int WN = NW / WM;
    static constexpr int A_UNITS = BM / UNIT_ROWS, B_UNITS = BN / UNIT_ROWS;
    static constexpr int LA = A_UNITS / S, LB = B_UNITS / S, L = LA + LB;     // loads of a stage, per wave
    static constexpr int STAGE = (BM + BN) * ROW_BYTES;
    static constexpr int RING = NST * STAGE;
    static constexpr int PITCH = BN + 4;
    static constexpr int RED = 2 * BM * PITCH * 4;
    static constexpr int LDS_BYTES = RING > RED ? RING : RED;
    static constexpr int RB = BM / WM / 16, CB = BN / WN / 16;
    // Stages on their way ahead of the one whose fragments are multiplied.  With a short ring the slot of that stage is filled again at
    // once, for which its reads must be back at the barrier; with a longer one the slot of the stage before, and no read is waited for.
    // NST - 1 and NST, us per call: [K][N] 1024 x 3584 x 4096 (128x128, four slots) 40.0 and 39.1, 200 x 16384 x 8192 85.0 and 84.1;
    // 999 x 1999 x 1984 (64x128, six) 20.6 and 20.7.
    static constexpr int AHEAD = NST <= 4 ? NST : NST - 1;
    static_assert(NW % WM == 0 && A_UNITS % S == 0 && B_UNITS % S == 0 && NST % 2 == 0 && NST >= 4 && LDS_BYTES <= 159 * 1024, "tile");
};

// STREAM ([K][N] only): B's loads carry the streaming hint.
template <int BM, int BN, int NW, int NST, KsKind KIND, class SL, bool KN = false, int WM = 1, bool STREAM = false>
__global__ __launch_bounds__(128 * NW)
void gemm_km_kernel(const KsParams p, const SL sl)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using C_ = KmCfg<BM, BN, NW, NST, WM>;
    constexpr int AHEAD = C_::AHEAD;
    constexpr int S = C_::S, LA = C_::LA, LB = C_::LB, L = C_::L, RB = C_::RB, CB = C_::CB, PITCH = C_::PITCH;
    constexpr bool GROUPED = KIND == KS_GROUPED;
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    __shared__ int s_gave_up;
    ks_fetch_params(p);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave & 1, nw = WM > 1 ? (wave >> 1) % C_::WN : wave >> 1, mw = WM > 1 ? (wave >> 1) / C_::WN : 0;
    const int ld_row = lane >> 3;
    // unit u = wave + S * i: S is even, so a wave's units are all even or all odd
    const int ld_chunk = (lane & 7) ^ (((wave & 1) * 4 + (lane >> 4)) & 7);
    const unsigned lds_u = (unsigned)(unsigned long)(lds_byte*)LDS_PTR(lds);
    const unsigned lds_ld = lds_u + wave * 1024;
    const unsigned fr_0 = lds_u + (lane & 15) * ROW_BYTES + (((4 * kh + (lane >> 4)) ^ ((lane >> 1) & 7)) << 4);
    const unsigned fr = fr_0 + mw * RB * 2048, fr_b = fr_0 + (BM / 16 + nw * CB) * 2048;
    // KN: B is [K][N].  A stage of it is 64 rows of one k each, BN columns (whole lines), 16-byte chunk c of row k in slot c ^ kn_swizzle(k).
    // Lane l of a wave takes the CB columns from CB (l % 16) on of the wave's 16 CB, of the eight k that its fragments hold: eight
    // reads of 2 CB bytes, and a byte permute per column and pair of k puts them into CB fragments, number j that of the columns
    // CB n + j.  (The hardware's transposing LDS read would do without the permutes, but the compiler waits for all loads in flight in front of
    // it: five times slower.)  The swizzle puts the rows that a read's 16-lane groups take into different banks.
    static_assert(!KN || ((CB == 2 || (CB == 4 && BN == 128)) && KIND != KS_GROUPED && (BN == 64 || BN == 128)), "[K][N] operand");
    constexpr int KN_ROW = BN * 2;
    auto kn_swizzle = [](int k) { return CB == 4 ? ((k >> 3) & 1) << 3 | ((k >> 4) & 1) << 2 : ((k >> 3) & (BN / 32 - 1)) << 2; };
    const int kn_k = 32 * kh + 8 * (lane >> 4), kn_n = lane & 15;
    const unsigned fr_kn = lds_u + BM * ROW_BYTES + kn_k * KN_ROW
                         + (((nw * CB * 2 + kn_n * CB / 8) ^ kn_swizzle(kn_k)) << 4) + kn_n * CB * 2 % 16;

    const int KC = p.KC;
    const int total_tiles = GROUPED ? *p.n_tiles_dev : p.total_tiles;
    const int G = p.grid, g = blockIdx.x;
    const int g0 = (G & 7) == 0 ? (g & 7) * (G >> 3) + (g >> 3) : g;
    const unsigned lda2 = (unsigned)p.lda * 2u, ldb2 = (unsigned)p.ldb * 2u;

    for (int t = g0; t < total_tiles; t += G) {
        TileWork w;
        if (!ks_tile<BM, BN, KIND>(p, t, w)) continue;
        const int m0 = w.m0, n0 = w.n0;
        const bool gated = p.flags && w.f_hi >= w.f_lo;
        const uint16_t* a_base = GROUPED ? p.A
                               : w.from_local ? p.A_local + (long long)(m0 - p.local_lo) * p.lda : p.A + (long long)m0 * p.lda;
        const uint16_t* b_base = KN ? p.B + n0 : p.B + (GROUPED ? (long long)w.expert * p.b_group_stride : 0ll) + (long long)n0 * p.ldb;
        const unsigned a_bytes = GROUPED ? p.a_bytes : (unsigned)min(BM, p.M - m0) * lda2;
        const unsigned b_bytes = KN ? (unsigned)(KC * BK - 1) * ldb2 + (unsigned)(p.N - n0) * 2u : (unsigned)min(BN, p.N - n0) * ldb2;
        unsigned off_a[LA], off_b[LB];
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int r = (wave + S * i) * UNIT_ROWS + ld_row;
            if constexpr (GROUPED) off_a[i] = m0 + r < w.m_lim ? (unsigned)(p.row_index ? p.row_index[m0 + r] : m0 + r) : 0xFFFFFFFFu;
            else off_a[i] = (unsigned)r * lda2 + (unsigned)(ld_chunk * 16);
        }
        if constexpr (GROUPED) asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            if constexpr (KN) {
                const int q = (wave + S * i) * 64 + lane, k = q / (BN / 8), c = (q % (BN / 8)) ^ kn_swizzle(k);
                off_b[i] = n0 + c * 8 < p.N ? (unsigned)k * ldb2 + (unsigned)(c * 16) : 0x80000000u;      // columns past the edge load as zero
            } else {
                off_b[i] = (unsigned)((wave + S * i) * UNIT_ROWS + ld_row) * ldb2 + (unsigned)(ld_chunk * 16);
            }
        }
        auto issue_b = [&](int s, auto slot_c) {
            constexpr int slot = decltype(slot_c)::value;
            const KsStage st = ks_stage(s, KC, KN ? BK * (int)ldb2 : ROW_BYTES, b_bytes);
            const __amdgpu_buffer_rsrc_t rs = make_rsrc(b_base, st.bytes);
            auto load = [&](auto aux_c) {
                static_for<LB>([&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_byte*)(unsigned long)(lds_ld + slot * C_::STAGE + (C_::A_UNITS + S * i) * 1024),
                                                             16, off_b[i], st.k_off, 0, decltype(aux_c)::value);
                });
            };
            // 2 = nt; [K][N]: an instance each
            if constexpr (KN) load(std::integral_constant<int, STREAM ? 2 : 0>{});
            else if (p.b_streams) load(std::integral_constant<int, 2>{});
            else load(std::integral_constant<int, 0>{});
        };
        auto issue_a = [&](int s, auto slot_c) {
            constexpr int slot = decltype(slot_c)::value;
            const KsStage st = ks_stage(s, KC, ROW_BYTES, a_bytes);
            const __amdgpu_buffer_rsrc_t rs = make_rsrc(a_base, st.bytes);
            static_for<LA>([&](auto i_c) {
                constexpr int i = decltype(i_c)::value;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_byte*)(unsigned long)(lds_ld + slot * C_::STAGE + S * i * 1024), 16,
                                                         off_a[i], st.k_off, 0, 0);
            });
        };
        auto issue_all_b = [&] { static_for<AHEAD>([&](auto j_c) { issue_b(decltype(j_c)::value, j_c); }); };
        if (wave != 0 || !gated) issue_all_b();
        if (gated && ks_wait(p, w, &s_gave_up, wave, lane, issue_all_b)) {
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // the launch drains; agg_status reports the time-out
            return;
        }
        if constexpr (GROUPED) {
#pragma unroll
            for (int i = 0; i < LA; ++i)
                off_a[i] = off_a[i] != 0xFFFFFFFFu ? off_a[i] * lda2 + (unsigned)(ld_chunk * 16) : 0xFFFFFF00u;
        }
        static_for<AHEAD>([&](auto j_c) { issue_a(decltype(j_c)::value, j_c); });

        f32x4_ acc[RB][CB];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) acc[i][j] = f32x4_{0.f, 0.f, 0.f, 0.f};
        constexpr int NM1 = RB * CB / 2;
        bf16x8 fa[2][RB], fb[2][CB];
        typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
        typedef std::conditional_t<CB == 4, __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned, unsigned> kn_cols;
        kn_cols kn[2][KN ? 8 : 1];             // CB columns of each k of KN's next fragments
        auto read_frags = [&](auto slot_c, auto set_c) {
            constexpr int slot = decltype(slot_c)::value, set = decltype(set_c)::value;
            if constexpr (KN) {
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    kn[set][k] = *(__attribute__((address_space(3))) const kn_cols*)(unsigned long)(fr_kn + slot * C_::STAGE + k * KN_ROW);
            } else
#pragma unroll
            for (int j = 0; j < CB; ++j) fb[set][j] = *(lds_frag*)(unsigned long)(fr_b + slot * C_::STAGE + j * 2048);
#pragma unroll
            for (int i = 0; i < RB; ++i) fa[set][i] = *(lds_frag*)(unsigned long)(fr + slot * C_::STAGE + i * 2048);
        };
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((AHEAD - 1) * LA));   // stage 0 has landed
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_frags(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        for (int s0 = 0; s0 < KC; s0 += NST) {
            // the fragments of stage s are in one register set; those of stage s + 1 are read into the other while it is
            // multiplied
            static_for<NST>([&](auto j_c) {
                constexpr int slot = decltype(j_c)::value;
                const int s = s0 + slot;
                if (s >= KC) return;
                asm volatile("" ::: "memory");
                // stage s + 1 has landed; behind the barrier that holds for all waves, and nobody needs stage s - 1 any more
                // (AHEAD = NST: nor stage s, this wave's reads of it are back)
                constexpr int reads_back = AHEAD == NST ? ~(0xF << 8) : ~0;
                if (s0 == 0 && slot <= AHEAD - 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm((AHEAD - 2 - slot) * LA + slot * L) & reads_back);
                else __builtin_amdgcn_s_waitcnt(vmcnt_imm((AHEAD - 2) * L) & reads_back);
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                read_frags(std::integral_constant<int, (slot + 1) % NST>{}, std::integral_constant<int, (slot + 1) & 1>{});
                if constexpr (KN) {
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        u32x4 f;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const kn_cols lo = kn[slot & 1][2 * k], hi = kn[slot & 1][2 * k + 1];
                            const unsigned sel = j & 1 ? 0x07060302u : 0x05040100u;
                            if constexpr (CB == 4) f[k] = __builtin_amdgcn_perm(hi[j / 2], lo[j / 2], sel);
                            else f[k] = __builtin_amdgcn_perm(hi, lo, sel);
                        }
                        fb[slot & 1][j] = __builtin_bit_cast(bf16x8, f);
                    }
                }
                auto multiply = [&](auto from_c, auto to_c) {
                    static_for<decltype(to_c)::value - decltype(from_c)::value>([&](auto n_c) {
                        constexpr int n = decltype(from_c)::value + decltype(n_c)::value, j = n / RB, i = n % RB;
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[slot & 1][j], fa[slot & 1][i], acc[i][j], 0, 0, 0);
                    });
                };
                // One LDS read behind each MFMA, and the loads in the middle: all eight waves come from the barrier at once, and reads (or
                // loads) ahead of the first MFMA hold each of them at the same queue while the matrix cores have nothing to do.  Reads
                // and loads first, reads between MFMAs, and this, us: [K][N] 1024 x 3584 x 4096 (128x128) 40.2, 39.2, 38.6;
                // 512 x 3584 x 4096 (64x128) 29.4, 28.6, 25.5; [N][K] 256 x 4096 x 4096 (64x64) 23.5, 22.7, 22.5; 512 x 3584 x 4096
                // (64x128) 23.3, 22.6, 22.0.
                multiply(std::integral_constant<int, 0>{}, std::integral_constant<int, NM1>{});
                static_for<NM1>([&](auto) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // LDS read
                });
                __builtin_amdgcn_sched_barrier(0);
                issue_b(s + AHEAD, std::integral_constant<int, (slot + AHEAD) % NST>{});
                issue_a(s + AHEAD, std::integral_constant<int, (slot + AHEAD) % NST>{});
                __builtin_amdgcn_sched_barrier(0);
                multiply(std::integral_constant<int, NM1>{}, std::integral_constant<int, RB * CB>{});
                __builtin_amdgcn_sched_barrier(0);
            });
        }

        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        __syncthreads();
        float* const red = (float*)lds;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            float* const to = red + (kh * BM + (mw * RB + i) * 16 + (lane & 15)) * PITCH + nw * CB * 16;
            if constexpr (KN) {                // block j holds columns CB n + j: a lane's 4 CB columns are consecutive
                float c[4 * CB];
#pragma unroll
                for (int v = 0; v < 4 * CB; ++v) c[v] = acc[i][v % CB][v / CB];
#pragma unroll
                for (int q = 0; q < CB; ++q) *(f32x4_*)(to + 4 * CB * (lane >> 4) + 4 * q) = f32x4_{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
            } else {
#pragma unroll
                for (int j = 0; j < CB; ++j) *(f32x4_*)(to + j * 16 + 4 * (lane >> 4)) = acc[i][j];
            }
        }
        __syncthreads();
        ks_store<BM, BN, 2, S * 64, KIND>(p, sl, w, red, tid);
        if constexpr (KIND == KS_SLICED) {
            const int epoch = p.epoch_ptr ? __hip_atomic_load(p.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : p.epoch;
            tile_publish<BM>(sl, m0, epoch, tid);
        }
        __syncthreads();
    }
#else
    (void)p; (void)sl;
#endif
}

// SHARED: gemm_km_kernel with X = NW, else gemm_ks_kernel with X = S.
template <bool SHARED, int BM, int BN, int X, int NST, KsKind KIND, bool KN = false, int WM = 1, class SL>
static hipError_t launch_ks_kind(const KsParams& p, const SL& sl, hipStream_t stream)
{
    using C_ = std::conditional_t<SHARED, KmCfg<BM, BN, X, NST, WM>, KsCfg<BM, BN, X, NST>>;
    void (*kernel)(const KsParams, const SL);
    constexpr bool BY_HINT = SHARED && KN;             // an instance without the streaming hint and one with it
    if constexpr (BY_HINT) kernel = p.b_streams ? gemm_km_kernel<BM, BN, X, NST, KIND, SL, KN, WM, true> : gemm_km_kernel<BM, BN, X, NST, KIND, SL, KN, WM, false>;
    else if constexpr (SHARED) kernel = gemm_km_kernel<BM, BN, X, NST, KIND, SL, KN, WM>;
    else kernel = gemm_ks_kernel<BM, BN, X, NST, KIND, SL>;
    constexpr int threads = SHARED ? 128 * X : 64 * X;
    static bool attr_set[2] = {false, false};
    bool& set = attr_set[BY_HINT && p.b_streams];
    if (!set) {
        hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, C_::LDS_BYTES);
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL(kernel, dim3(p.grid), dim3(threads), C_::LDS_BYTES, stream, p, sl);
    return hipGetLastError();
}

// The forms of a tile that the automatic choice takes (launch_rules.h): KS_PLAIN and KS_SLICED, KS_GROUPED.
enum KsForms { KS_DENSE = 1, KS_MOE = 2 };

// The launch of `g` (a GemmParams whose tile fields are those of this tile shape) on this kernel.
template <bool SHARED, int BM, int BN, int X, int NST, int FORMS, bool KN = false, int WM = 1>
static hipError_t launch_ks(const GemmParams& g, bool grouped, int grid, hipStream_t stream)
{
    KsParams p{};
    p.A = g.A; p.A_local = g.A_local; p.B = g.B; p.C = g.C;
    p.lda = (int)g.lda; p.ldb = (int)g.ldb; p.ldc = (int)g.ldc;
    p.M = g.M; p.N = g.N; p.KC = g.K / BK;
    p.tiles_m = g.tiles_m;
    p.total_tiles = g.tiles_m * g.tiles_n;
    p.grid = grid;
    p.m_tile_start = g.m_tile_start;
    p.tiles_m_mul = div_mul(g.tiles_m);
    p.flag_mul = div_mul(g.rows_per_flag);
    p.local_lo = g.local_lo; p.local_hi = g.local_hi;
    p.flags = g.flags; p.epoch_ptr = g.epoch_ptr; p.err = g.err; p.wait_ticks = g.wait_ticks;
    p.epoch = g.epoch; p.n_flags = g.n_flags; p.c_is_f32 = g.c_is_f32;
    // Weights that the memory-side cache (256 MB) cannot hold come from HBM whatever the loads ask for, and are fetched
    // faster with the streaming hint: 64 tokens of Table 4 (1 GB of weights) 165 -> 155 us per call, 512 tokens 209 -> 199.
    // Weights that it may hold do not take the hint: 16 x 3584 x 4096 (29 MB) 8.5 without, 9.8 with it.
    p.b_streams = g.b_total_bytes >= (256ll << 20);
    if (grouped ? !(FORMS & KS_MOE) : !(FORMS & KS_DENSE)) return hipErrorInvalidValue;
    if constexpr ((FORMS & KS_MOE) != 0) {
        if (grouped) {
            p.row_index = g.row_index; p.tile_tab = g.tile_tab; p.n_tiles_dev = g.n_tiles_dev;
            p.b_group_stride = g.b_group_stride; p.a_bytes = g.a_bytes;
            return launch_ks_kind<SHARED, BM, BN, X, NST, KS_GROUPED>(p, KsNoSlices{}, stream);
        }
    }
    if constexpr ((FORMS & KS_DENSE) != 0) {
        if (g.n_slices == 0) return launch_ks_kind<SHARED, BM, BN, X, NST, KS_PLAIN, KN, WM>(p, KsNoSlices{}, stream);
        auto launch = [&](auto sl) {
            sl.M = g.M; sl.tiles_n = g.tiles_n; sl.slice_rows = g.slice_rows; sl.slice_chunks = g.slice_chunks;
            sl.chunk_rows = g.chunk_rows; sl.ldc_slice = (int)g.ldc_slice; sl.slice_mul = div_mul(g.slice_rows);
            sl.slice_ctr = g.slice_ctr;
            for (int w = 0; w < g.n_slices; ++w) { sl.slice_dst[w] = g.slice_dst[w]; sl.slice_flag[w] = g.slice_flag[w]; }
            return launch_ks_kind<SHARED, BM, BN, X, NST, KS_SLICED, KN, WM>(p, sl, stream);
        };
        return g.n_slices <= 8 ? launch(KsSlices<8>{}) : launch(KsSlices<kMaxWorld>{});
    }
    return hipErrorInvalidValue;
}

}  // namespace agg

// One launch function per tile shape (gemm_ks_*.hip); gemm_dispatch.hip names them.
#define AGG_KS_INSTANCE(SHARED, BM, BN, X, NST, FORMS)                                                      \
    namespace agg {                                                                                         \
    hipError_t launch_gemm_ks_##BM##x##BN(const GemmParams& p, bool grouped, int grid, hipStream_t s)       \
    {                                                                                                       \
        return launch_ks<SHARED, BM, BN, X, NST, FORMS>(p, grouped, grid, s);                               \
    }                                                                                                       \
    }
// ... for a B stored [K][N] and read in place
#define AGG_KN_INSTANCE(BM, BN, NW, NST, WM)                                                                \
    namespace agg {                                                                                         \
    hipError_t launch_gemm_kn_##BM##x##BN(const GemmParams& p, int grid, hipStream_t s)                     \
    {                                                                                                       \
        return launch_ks<true, BM, BN, NW, NST, KS_DENSE, true, WM>(p, false, grid, s);                     \
    }                                                                                                       \
    }
