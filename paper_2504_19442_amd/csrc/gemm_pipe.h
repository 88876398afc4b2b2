// Grouped GEMM (MoE, Section 4.1) as one stream of K stages over all of a workgroup's tiles.
//
// The main loop is that of gemm_kernel (four waves, wave w owns BM / 4 rows and all columns, 16x16x32 MFMAs in the same order: the same
// bits); what surrounds it differs, because what this GEMM waits for is its weights, of which every tile has its own.
//  * A and B have a ring each, of whole stages: two of A, three of B.  A batch of loads is A of the stage after the next one and then B of
//    the one after that; loads return in order, so the wait for A leaves B in flight, and B, which comes from HBM, has two stages to
//    arrive, A, which mostly hits the L2, one.
//  * The stream does not end with a tile: the last stages of a tile ask for the first ones of the next, whose list entry, token rows
//    and signals are looked at meanwhile, and the tile's rows are stored while those are on their way: from the registers (the rings are
//    in use), and counted (buffer stores whose descriptor holds back the rows that are not wanted), so that the first wait of the
//    next tile can leave them outstanding.  Signals that are not there yet hold nothing back but the next tile's rows of A: those are asked
//    for when the tile's rows have been stored and the signals waited for.
//  * The entries of the tile list and the token rows come through LDS as well: a load into registers would be waited for together with
//    every load in front of it.
// Shapes: 320x128 and 192x192 are there for segments that fill one tile but not two of a power of two (each weight then crosses the load
// path once, and no second tile is nearly empty), 128x192 and 128x224 for shorter and for much longer ones.  192x128, 256x160, 128x128 and
// 256x128 would add 0.3 % or less each over the ranges of launch_rules.h.
// Measured, Table 4 (8192 tokens, 222 to 298 rows per expert, 1 GB of weights), all shards there, routing and GEMM, us: 256x256 of gemm_kernel
// 382; 320x128 in that kernel 340, with the streaming hint on B 313; here 298 (another box: 335 and 291; kernel 280 to 300: 3.6 to 4 TB/s, 0.9
// to 1 PFLOP/s; 59 % of the cycles are MFMAs, at 1.9 GHz).  With the gather beside it the call takes 340.  What is left: the load path, 56 KiB per 1280 MFMA cycles (the loop of gemm_kernel without any loads takes 208 us,
// without those of A 268, without those of B 245), and power.  Table 5 (K = 192, rows in place, fp32), kernel: 54 -> 47.6, 3.9 TB/s;
// with whole lines per store (out_cols) the call is 108.6 -> 102.3 on one stream, Table 4 in fp32 341 -> 334 (routing and GEMM: 301).
#pragma once
#include "gemm_kernel.h"
#include "ks_stage.h"

namespace agg {

template <int BM, int BN>
struct PipeCfg : TileCfg<BM, BN> {
    using Base = TileCfg<BM, BN>;
    static constexpr int RA = 2, RB = 3;                    // stages of A and of B in LDS
    static constexpr int LA = BM / 32, LB = BN / 32;         // loads of a stage, per wave
    static constexpr int A_STAGE = BM * ROW_BYTES, B_STAGE = BN * ROW_BYTES;
    static constexpr int B_AT = RA * A_STAGE;                // where B's ring starts
    static constexpr int ROWS_AT = B_AT + RB * B_STAGE;      // rows of A of the next tile
    static constexpr int ROW_LOADS = (BM + 255) / 256;                   // a wave's loads of them
    static constexpr int ENTRY_AT = ROWS_AT + ROW_LOADS * 1024;          // an entry of the tile list, a copy per wave
    static constexpr int WORD_AT = ENTRY_AT + 1024;
    static constexpr int LDS_BYTES = WORD_AT + 16;
    static constexpr int MIN_STAGES = RB;                    // a tile has at least this many stages (empty ones, where K is shorter)
    static constexpr int N_ST_BF16 = Base::MB16 * 4 * out_cols<BN, 2>().n, N_ST_F32 = Base::MB16 * 4 * out_cols<BN, 4>().n;     // stores of a wave
    static_assert(RB == RA + 1, "what a stage's barrier waits for: all but the last stage of B");
    static_assert(Base::L == LA + LB && LDS_BYTES <= 159 * 1024, "tile");
};

// first MFMA of a tile's accumulator block: C = 0
template <int BLK>
__device__ __forceinline__ void mfma_acc16_first(const bf16x8& a, const bf16x8& b)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, 0" ::"v"(a), "v"(b), "n"(BLK * 4), "n"(BLK * 4 + 3));
}

template <int BM, int BN, bool B_NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_vgpr(192))) void gemm_pipe_kernel(const GemmParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using C_ = PipeCfg<BM, BN>;
    constexpr int LA = C_::LA, LB = C_::LB, TM = C_::TM, MB16 = C_::MB16, NB16 = C_::NB16, RA = C_::RA, RB = C_::RB;
    // naming the last accumulator register makes the compiler reserve a0..a(ACC-1) for this kernel
    static_assert(C_::ACC == 160 || C_::ACC == 144 || C_::ACC == 112 || C_::ACC == 96, "add a reservation line for this accumulator count");
    if constexpr (C_::ACC == 160) asm volatile("; accumulators a0..a159" ::: "a159");
    else if constexpr (C_::ACC == 144) asm volatile("; accumulators a0..a143" ::: "a143");
    else if constexpr (C_::ACC == 112) asm volatile("; accumulators a0..a111" ::: "a111");
    else asm volatile("; accumulators a0..a95" ::: "a95");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // load i of a wave covers rows 8 (wave + 4 i) + 0..7 of the stage; 16-byte chunk c of row r is kept in slot c ^ ((r >> 1) & 7)
    const int ld_row = wave * UNIT_ROWS + (lane >> 3);
    const unsigned ld_chunk = (unsigned)((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) * 16u;
    const unsigned lds_u = (unsigned)(unsigned long)(lds_byte*)LDS_PTR(lds);
    const unsigned lds_wave = lds_u + wave * 1024;
    typedef __attribute__((address_space(3))) volatile int lds_int;
    lds_int* const s_word = (lds_int*)(unsigned long)(lds_u + C_::WORD_AT);
    unsigned fr_a[2], fr_b[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const unsigned at = lds_u + (lane & 15) * ROW_BYTES + (((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) << 4);
        fr_a[h] = at + wave * MB16 * 2048;
        fr_b[h] = at + C_::B_AT;
    }
    const int KS = p.K / BK;
    const int KE = KS > C_::MIN_STAGES ? KS : C_::MIN_STAGES;
    const int epoch = p.epoch_ptr ? __hip_atomic_load(p.epoch_ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : p.epoch;
    const int total_tiles = *p.n_tiles_dev;
    const int G = gridDim.x, g = blockIdx.x;
    int t = (G & 7) == 0 ? (g & 7) * (G >> 3) + (g >> 3) : g;      // consecutive tiles of the list go to the workgroups of one XCD
    if (t >= total_tiles) return;
    const unsigned lda2 = (unsigned)p.lda * 2u, ldb2 = (unsigned)p.ldb * 2u;

    // ---- the list: the tile whose product is being computed, the next one, and (in flight) the entry of the one after that
    struct Tile { int expert, m0, m_lim, n0, f_lo, f_hi, st_lo, st_hi; bool valid; };
    // What is known of the list lies in LDS and comes there like the operands: a load that the compiler waited for would wait for
    // every load in front of it.  Asked for in one place between two tiles, it is there behind the next barrier but one.
    auto fetch_entry = [&](int at) {
        // (past the end of the list nothing is loaded)
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.tile_tab + at, at < total_tiles ? (unsigned)sizeof(MoeTile) : 0u);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_byte*)(unsigned long)(lds_u + C_::ENTRY_AT + wave * 256), 4, lane * 4, 0, 0, 0);
    };
    auto decode = [&](int at) {
        const lds_int* e = (const lds_int*)(unsigned long)(lds_u + C_::ENTRY_AT + wave * 256);
        Tile w;
        w.expert = __builtin_amdgcn_readfirstlane(e[0]);
        w.m0 = __builtin_amdgcn_readfirstlane(e[1]);
        w.m_lim = __builtin_amdgcn_readfirstlane(e[2]);
        w.n0 = __builtin_amdgcn_readfirstlane(e[3]) * BN;
        w.f_lo = __builtin_amdgcn_readfirstlane(e[4]);
        w.f_hi = __builtin_amdgcn_readfirstlane(e[5]);
        w.st_lo = __builtin_amdgcn_readfirstlane(e[6]);
        w.st_hi = __builtin_amdgcn_readfirstlane(e[7]);
        w.valid = at < total_tiles;
        return w;
    };
    auto fetch_rows = [&](const Tile& w) {
        if (!p.row_index) return;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(p.row_index + w.m0, w.valid ? (unsigned)(w.m_lim - w.m0) * 4u : 0u);
#pragma unroll
        for (int i = 0; i < C_::ROW_LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_byte*)(unsigned long)(lds_u + C_::ROWS_AT + wave * 256 + i * 1024), 4,
                                                     (tid + i * 256) * 4, 0, 0, 0);
    };
    unsigned off_a[LA], off_b[LB];
    auto rows_to_offsets = [&](const Tile& w) {
        // rows past the segment end get an offset outside the descriptor and load as zero
        const lds_int* rows = (const lds_int*)(unsigned long)(lds_u + C_::ROWS_AT);
        unsigned row[LA];
        if (p.row_index) {
#pragma unroll
            for (int i = 0; i < LA; ++i) row[i] = (unsigned)rows[ld_row + i * 32];
        } else {
#pragma unroll
            for (int i = 0; i < LA; ++i) row[i] = (unsigned)(w.m0 + ld_row + i * 32);
        }
#pragma unroll
        for (int i = 0; i < LA; ++i) off_a[i] = w.m0 + ld_row + i * 32 < w.m_lim ? row[i] * lda2 + ld_chunk : 0x80000000u;
    };
#pragma unroll
    for (int i = 0; i < LB; ++i) off_b[i] = (unsigned)(p.c_is_f32 ? out_col<BN, 4>(ld_row + i * 32) : out_col<BN, 2>(ld_row + i * 32)) * ldb2 + ld_chunk;

    // ---- the stream of loads.  The stages of a tile are followed by those of the next one; a stage past the end of K, or of the list,
    // loads nothing.
    const uint16_t* b_base;
    unsigned b_bytes;
    int ka, kb, kc_a = KS, kc_b = KS;        // next stage of A and of B, and how many there are
    auto point_b = [&](const Tile& w) {
        b_base = p.B + (long long)w.expert * p.b_group_stride + (long long)w.n0 * p.ldb;
        b_bytes = (unsigned)min(BN, p.N - w.n0) * ldb2;
        kb = 0;
        kc_b = w.valid ? KS : 0;
    };
    unsigned dst_a = 0, dst_b = 0;           // ring offsets of the batch under way
    __amdgpu_buffer_rsrc_t a_rs, b_rs;
    int a_off, b_off;
    auto batch_a = [&] {
        const KsStage s = ks_stage(ka, kc_a, ROW_BYTES, p.a_bytes);
        a_rs = make_rsrc(p.A, s.bytes);
        a_off = s.k_off;
        ++ka;
    };
    auto batch_b = [&] {
        const KsStage s = ks_stage(kb, kc_b, ROW_BYTES, b_bytes);
        b_rs = make_rsrc(b_base, s.bytes);
        b_off = s.k_off;
        ++kb;
    };
    auto load_a = [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rs, (lds_byte*)(unsigned long)(lds_wave + dst_a + i * 4096), 16, off_a[i], a_off, 0, 0);
    };
    auto load_b = [&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rs, (lds_byte*)(unsigned long)(lds_wave + C_::B_AT + dst_b + i * 4096), 16, off_b[i],
                                                 b_off, 0, B_NT ? 2 : 0);
    };
    auto load_op = [&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        if constexpr (j < LA) load_a(j_c);
        else load_b(std::integral_constant<int, j - LA>{});
    };

    // ---- signals: seen are those of [seen_lo, seen_hi]
    int seen_lo = 0x7FFFFFFF, seen_hi = -1;
    auto must_wait = [&](const Tile& w) { return p.flags && w.valid && w.f_hi >= w.f_lo && (w.f_lo < seen_lo || w.f_hi > seen_hi); };
    // wave 0, in front of a barrier: a look at the signals, or the wait for them
    auto look = [&](const Tile& w, auto wait_c) {
        if (wave == 0) {
            bool any;
            if constexpr (decltype(wait_c)::value) any = __ballot(poll_signals(p, w.f_lo, w.f_hi, epoch, lane)) != 0;
            else any = signals_missing(p, w.f_lo, w.f_hi, epoch, lane);
            if (lane == 0) *s_word = any;
        }
        asm volatile("" ::: "memory");
    };
    auto seen = [&](const Tile& w) {          // all waves, behind it; false: not all are there
        if (__builtin_amdgcn_readfirstlane(*s_word) != 0) return false;
        if (w.f_lo <= seen_hi + 1 && w.f_hi >= seen_lo - 1 && seen_hi >= 0) {
            seen_lo = min(seen_lo, w.f_lo);
            seen_hi = max(seen_hi, w.f_hi);
        } else {
            seen_lo = w.f_lo;
            seen_hi = w.f_hi;
        }
        return true;
    };

    // ---- start: the first tile's B is asked for before its signals are looked at
    auto arrived = [&](auto behind_c) {       // all that was asked for before the last `behind` loads
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(decltype(behind_c)::value));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    fetch_entry(t);
    arrived(std::integral_constant<int, 0>{});
    Tile cur = decode(t), nxt;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    fetch_rows(cur);
    fetch_entry(t + G);
    asm volatile("" ::: "memory");
    point_b(cur);
    static_for<RB>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        dst_b = s * C_::B_STAGE;
        batch_b();
        static_for<LB>([&](auto i_c) { load_b(i_c); });
    });
    if (must_wait(cur)) {
        look(cur, std::true_type{});
        __syncthreads();
        if (!seen(cur)) { __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); return; }
        __syncthreads();
    }
    arrived(std::integral_constant<int, RB * LB>{});
    rows_to_offsets(cur);
    ka = 0;
    static_for<RA>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        dst_a = s * C_::A_STAGE;
        batch_a();
        static_for<LA>([&](auto i_c) { load_a(i_c); });
    });
    nxt = decode(t + G);
    arrived(std::integral_constant<int, (RA - 1) * LA>{});
    fetch_rows(nxt);
    fetch_entry(t + 2 * G);

    bf16x8 fa[2][MB16], fb[NB16];
    unsigned at_a = 0, at_b = 0;             // ring offsets of the running stage
    unsigned ra, rb;                         // addresses of the fragments that are read now
    auto read_a = [&](auto i_c, int set) { fa[set][decltype(i_c)::value] = *(lds_frag*)(unsigned long)(ra + decltype(i_c)::value * 2048); };
    auto read_b = [&](auto j_c) { fb[decltype(j_c)::value] = *(lds_frag*)(unsigned long)(rb + decltype(j_c)::value * 2048); };

    ra = fr_a[0];
    rb = fr_b[0];
    static_for<MB16>([&](auto i_c) { read_a(i_c, 0); });
    static_for<NB16>([&](auto j_c) { read_b(j_c); });

    enum { WAIT_ALL, WAIT_BF16, WAIT_F32 };
    int first_wait = WAIT_ALL;               // what the first stage's barrier of a tile may leave outstanding

    // Stage ks of the running tile.  The next tile's signals are looked at two stages before its end.  Where some are still to come, its
    // rows of A are not asked for (`late`): they are waited for when this tile's rows have been stored.
    static_assert(C_::MIN_STAGES > RA, "the look at the signals is not in a tile's first stage");
    bool late = false;
    auto stage = [&](int ks, auto first_c) {
        constexpr bool first = decltype(first_c)::value;
        static_for<2>([&](auto h_c) {
            constexpr int h = decltype(h_c)::value;
            constexpr auto slots = C_::make_slots(h);
            if constexpr (h == 0) {
                ra = fr_a[1] + at_a;
                rb = fr_b[1] + at_b;
                asm volatile("" : "+v"(ra), "+v"(rb));
            }
            static_for<C_::NS>([&](auto s_c) {
                constexpr int sl = decltype(s_c)::value;
                constexpr int j = sl / MB16, i = sl % MB16;
                if constexpr (first && h == 0) mfma_acc16_first<i * NB16 + j>(fa[h][i], fb[j]);
                else mfma_acc16<i * NB16 + j>(fa[h][i], fb[j]);
                if constexpr (h == 1 && sl == C_::SB) {
                    // The running stage's fragments are all in registers, and the next stage has landed: of the loads behind it, those
                    // of B alone may be outstanding (and, in a tile's first stage, the stores of the tile before it).
                    const bool to_next_a = !first && ks == KE - RA;
                    const bool gate = to_next_a && must_wait(nxt);
                    if (gate) look(nxt, std::false_type{});
                    if constexpr (first) {
                        if (first_wait == WAIT_BF16) __builtin_amdgcn_s_waitcnt(vmcnt_imm(LB + C_::N_ST_BF16 < 63 ? LB + C_::N_ST_BF16 : 63) & ~(0xF << 8));
                        else if (first_wait == WAIT_F32) __builtin_amdgcn_s_waitcnt(vmcnt_imm(LB + C_::N_ST_F32 < 63 ? LB + C_::N_ST_F32 : 63) & ~(0xF << 8));
                        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & ~(0xF << 8));
                    } else {
                        __builtin_amdgcn_s_waitcnt(vmcnt_imm(LB) & ~(0xF << 8));
                    }
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    if (to_next_a) {
                        late = gate && !seen(nxt);
                        rows_to_offsets(nxt);
                        ka = 0;
                        kc_a = nxt.valid && !late ? KS : 0;
                    }
                    if (ks == KE - RB) point_b(nxt);
                    dst_a = at_a;
                    dst_b = at_b;
                    batch_a();
                    batch_b();
                    at_a = at_a == (RA - 1) * C_::A_STAGE ? 0 : at_a + C_::A_STAGE;
                    at_b = at_b == (RB - 1) * C_::B_STAGE ? 0 : at_b + C_::B_STAGE;
                    ra = fr_a[0] + at_a;
                    rb = fr_b[0] + at_b;
                    asm volatile("" : "+v"(ra), "+v"(rb), "+s"(dst_a), "+s"(dst_b));
                }
                static_for<C_::PER_SLOT>([&](auto k_c) {
                    constexpr auto op = slots.op[sl][decltype(k_c)::value];
                    if constexpr (op.type == 1) read_b(std::integral_constant<int, op.idx>{});
                    else if constexpr (op.type == 2) read_a(std::integral_constant<int, op.idx>{}, 1 - h);
                    else if constexpr (op.type == 3 && !(first && h == 0)) load_op(std::integral_constant<int, op.idx>{});
                });
            });
        });
    };

    for (;;) {
        stage(0, std::true_type{});
        for (int ks = 1; ks < KE; ++ks) stage(ks, std::false_type{});

        // ---- between two tiles.  What is asked for first: the list's entry after the next tile's, the rest of the batch of loads that
        // the last barrier released (all that the first stage of the next tile waits for), and then the stores.
        asm volatile("" ::: "memory");
        const Tile after = decode(t + 2 * G);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fetch_rows(after);
        fetch_entry(t + 3 * G);
        asm volatile("" ::: "memory");
        static_for<C_::LH0>([&](auto j_c) { load_op(std::integral_constant<int, C_::LH1 + decltype(j_c)::value>{}); });
        asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");       // (and the last MFMAs retire before the read-out)
        {
            int lane_e = lane;
            asm volatile("" : "+v"(lane_e));
            const int row_w = cur.m0 + wave * TM;
            const int n_valid = min(BN, p.N - cur.n0);
            auto stores = [&](auto tag) {
                using T = decltype(tag);
                constexpr int esz = sizeof(T);
                constexpr OutCols cols = out_cols<BN, esz>();
                char* const c_row0 = (char*)p.C + ((long long)row_w * p.ldc + cur.n0) * esz;
                const unsigned ldc_b = (unsigned)p.ldc * esz;
                // whole columns, rows that start on 16 bytes: a fixed number of stores, rows outside [st_lo, st_hi) held back by the
                // descriptor
                const bool whole = n_valid == BN && ((reinterpret_cast<uintptr_t>(p.C) | ((unsigned long long)p.ldc * esz)) & 15) == 0 && p.ldc < (1 << 22);
                first_wait = !whole ? WAIT_ALL : esz == 2 ? WAIT_BF16 : WAIT_F32;
                // rows in place (MoE + ReduceScatter): the next kernel reads them, they may stay in the caches
                const bool stream_out = esz == 2 || p.row_index;
                const __amdgpu_buffer_rsrc_t rs = make_rsrc(c_row0, (unsigned)TM * ldc_b);
                static_for<MB16 * 4>([&](auto iv_c) {
                    constexpr int i = decltype(iv_c)::value / 4, v = decltype(iv_c)::value % 4;
                    const int r = i * 16 + 4 * (lane_e >> 4) + v;
                    const bool in = row_w + r >= cur.st_lo && row_w + r < cur.st_hi;
                    const unsigned off = in ? (unsigned)r * ldc_b : 0x80000000u;
                    static_for<cols.n>([&](auto g_c) {
                        constexpr int s = cols.start[decltype(g_c)::value], g = cols.size[decltype(g_c)::value];
                        const auto x = acc_row<T, g, (i * NB16 + s) * 4 + v>();
                        const int col = 16 * s + g * (lane_e & 15);
                        if (whole) {
                            if (stream_out) buffer_store<2>(x, rs, off + col * esz);
                            else buffer_store<0>(x, rs, off + col * esz);
                        } else if (in) {
                            store_cols<false>((T*)(c_row0 + (long long)r * p.ldc * esz) + col, x, n_valid - col);
                        }
                    });
                });
            };
            if (p.c_is_f32) stores(float{}); else stores(__bf16{});
        }
        asm volatile("" ::: "memory");
        if (!nxt.valid) break;
        if (late) {
            // The next tile's first stages of A, into the places that nothing was loaded into; its first fragments of A again
            look(nxt, std::true_type{});
            __syncthreads();
            if (!seen(nxt)) break;
            ka = 0;
            kc_a = KS;
            static_for<RA>([&](auto s_c) {
                dst_a = at_a + decltype(s_c)::value * C_::A_STAGE;
                if (dst_a >= RA * C_::A_STAGE) dst_a -= RA * C_::A_STAGE;
                batch_a();
                static_for<LA>([&](auto i_c) { load_a(i_c); });
            });
            arrived(std::integral_constant<int, 0>{});
            static_for<MB16>([&](auto i_c) { read_a(i_c, 0); });
            late = false;
        }
        cur = nxt;
        nxt = after;
        t += G;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#else
    (void)p;
#endif
}

template <int BM, int BN, bool B_NT>
static hipError_t launch_pipe_nt(const GemmParams& p, int grid, hipStream_t stream)
{
    using C_ = PipeCfg<BM, BN>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)gemm_pipe_kernel<BM, BN, B_NT>, hipFuncAttributeMaxDynamicSharedMemorySize, C_::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((gemm_pipe_kernel<BM, BN, B_NT>), dim3(grid), dim3(256), C_::LDS_BYTES, stream, p);
    return hipGetLastError();
}

template <int BM, int BN>
static hipError_t launch_pipe(const GemmParams& p, int grid, hipStream_t stream)
{
    return p.b_total_bytes >= (256ll << 20) ? launch_pipe_nt<BM, BN, true>(p, grid, stream) : launch_pipe_nt<BM, BN, false>(p, grid, stream);
}

}  // namespace agg

// One launch function per tile shape (gemm_pipe_*.hip); gemm_dispatch.hip names them.
#define AGG_PIPE_INSTANCE(BM, BN)                                                                                         \
    namespace agg {                                                                                                       \
    hipError_t launch_gemm_pipe_##BM##x##BN(const GemmParams& p, bool grouped, int grid, hipStream_t s)                   \
    {                                                                                                                     \
        return grouped ? launch_pipe<BM, BN>(p, grid, s)     : hipErrorInvalidValue;                                      \
    }                                                                                                                     \
    }
