// Rules by which the host picks tiles and grids.  Plain C++, so that they can be checked without a GPU.
#pragma once
#include "moe_table.h"

#include <algorithm>
#include <cmath>

namespace agg {

// A tile configuration = a tile shape (bits 0-1) and the MFMA form of the main loop (bit 2): v_mfma_f32_32x32x16_bf16,
// or, with TILE_K32, v_mfma_f32_16x16x32_bf16 (half the accumulator traffic per flop: the chip holds a higher clock).
// Those are what agg_set_tile_config takes.  The tiles of gemm_pipe.h (grouped GEMM, 16x16x32 form: the same bits) belong to the
// automatic choice alone.
enum TileConfig { TILE_256x224 = 0, TILE_128x128 = 1, TILE_256x256 = 2, TILE_128x256 = 3, TILE_K32 = 4, TILE_NUMBERED = 8,
                  PIPE_128x192 = TILE_NUMBERED, PIPE_128x224, PIPE_192x192, PIPE_320x128, TILE_CONFIGS };

// Tile configurations of the K-split kernels (gemm_ks.h): what the automatic choice takes where the tiles above would leave
// most of the chip idle; not selectable by number.  KN_: the same for a B stored [K][N] and read in place.
enum KsTileConfig { KS_16x16 = TILE_CONFIGS, KS_16x32, KS_16x64, KS_32x32, KS_64x32, KS_64x64, KS_64x128, KN_64x64, KN_64x128, KN_128x128, KS_CONFIGS_END };

struct TileShape { int bm, bn; };
inline TileShape tile_shape(int cfg)
{
    switch (cfg) {
        case PIPE_128x192: return {128, 192};
        case PIPE_128x224: return {128, 224};
        case PIPE_192x192: return {192, 192};
        case PIPE_320x128: return {320, 128};
        case KS_16x16: return {16, 16};
        case KS_16x32: return {16, 32};
        case KS_16x64: return {16, 64};
        case KS_32x32: return {32, 32};
        case KS_64x32: return {64, 32};
        case KS_64x64: case KN_64x64: return {64, 64};
        case KS_64x128: case KN_64x128: return {64, 128};
        case KN_128x128: return {128, 128};
        default: break;
    }
    switch (cfg & 3) {
        case TILE_256x224: return {256, 224};
        case TILE_256x256: return {256, 256};
        case TILE_128x256: return {128, 256};
        default: return {128, 128};
    }
}

// Estimated time of one tile in a full round, in microseconds: what a tile takes whatever its K, and what it takes per 64
// of K.  From sweeps of M, N, K with every shape: what a tile costs follows the bytes it pulls through its compute unit's
// load path, (BM + BN) x 128 per 64 of K at about 70 KB/us, up to 128 x 128; the large tiles are bound by the matrix pipes
// at the clock the chip holds with all of them busy.  Over 60 shapes drawn from M 16..8192, N 96..7168, K 256..8192 (over
// their logarithms) the choice costs 1.4 % more than the best shape of each, and it is the best or within 2 % of it on 54
// (profiles/tile_choice.txt).  Where the line lies, both sides measured in
// us: 16x3584x4096 16x16 8.7, 128x128 24.9; 64x8192x3584 64x32 19.1, 64x64 22, 128x128 33; 128x7168x8192 64x64 42,
// 128x128 75; 999x1999x1984 64x128 17.2, 128x128 21; 1024x3584x4096 128x128 34, 64x128 51.
struct TileCost { int cfg; double fixed_us, us_per_k64; };
constexpr TileCost kTileCosts[] = {
    {TILE_256x224 | TILE_K32, 4.0, 1.25}, {TILE_256x256 | TILE_K32, 4.0, 1.42}, {TILE_128x256 | TILE_K32, 4.0, 0.83},
    {TILE_128x128 | TILE_K32, 4.0, 0.46},
    {KS_64x128, 3.5, 0.37}, {KS_64x64, 3.0, 0.24}, {KS_64x32, 4.0, 0.20}, {KS_32x32, 3.0, 0.125}, {KS_16x32, 3.0, 0.09},
    {KS_16x16, 3.0, 0.07},
};
constexpr TileCost kTileCostsKn[] = {{KN_64x64, 3.9, 0.299}, {KN_64x128, 4.0, 0.38}, {KN_128x128, 4.6, 0.556}};
constexpr double kTransposeUs = 7.6, kTransposeBytesPerUs = 5.6e6;        // tile_kn
constexpr double kPublishUs = 0.009, kStoreUs256 = 10.0, kStoreUs128x256 = 4.0;     // best_tile, slices
// the K-split kernels divide row and tile numbers with 32-bit multipliers, exact while rows x divisor < 2^32
constexpr int kKsMaxRows = 65535;

inline long long tile_count(TileShape t, int M, int N) { return (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

inline double tile_cost(int num_cus, const TileCost& k, int M, int N, int K, bool slices)
{
    const TileShape t = tile_shape(k.cfg);
    const long long tiles = tile_count(t, M, N);
    const long long rounds = (tiles + num_cus - 1) / num_cus;
    double cost = (double)rounds * (k.fixed_us + k.us_per_k64 * (K / 64));
    if (slices) {
        cost += kPublishUs * (double)tiles;
        cost += (double)rounds * (t.bm == 256 ? kStoreUs256 : t.bn == 256 ? kStoreUs128x256 : 0.0);
    }
    return cost;
}

// Pick the tile shape with the smallest estimated time: rounds of tiles over the CUs times the cost of a tile.  The
// 16x16x32 form of the main loop everywhere: the same work at a lower power per flop, so the chip holds a higher clock
// (measured 5 to 8 % faster on every shape); the 32x32x16 form stays selectable (configurations 0 to 3).
// slices: GEMM + ReduceScatter's epilogue, which adds two things.  Every tile publishes itself (a release fence, an atomic add to
// a counter that the tiles of a slice share): 9 ns each, one after the other, whatever their size.  And it stores fp32, which at
// the end of a round all CUs do at once while nothing multiplies; with four 128x128 tiles in place of one large one the stores of
// some fall behind the loads of others.  Over 450 problems drawn from 4 to 8192 rows, N 96 to 8192, K 128 to 3584 the choice costs
// 1.4 % more than the best tile (2.5 % without the two), and 3 are more than 2 % slower than with the numbered tiles alone (14).
// On one stream nothing is published (gemm_rs), and it is counted all the same: the tile, and with it the order of the sums, follows from the
// sizes alone.
// Both sides, us per call: 8 x 3300 x 128 16x16 12.7, 32x32 10.4, 128x128 10.5; 4232 x 4060 x 2368 256x224 174, 128x128 148.
// large_only: without the K-split tiles.
inline int best_tile(int num_cus, int M, int N, int K, bool slices = false, bool large_only = false)
{
    int best = kTileCosts[0].cfg;
    double best_cost = 1e300;
    for (const TileCost& k : kTileCosts) {
        if (k.cfg >= TILE_CONFIGS && (large_only || M > kKsMaxRows)) continue;
        const double cost = tile_cost(num_cus, k, M, N, K, slices);
        if (cost < best_cost) {
            best_cost = cost;
            best = k.cfg;
        }
    }
    return best;
}

// Tile for a B stored [K][N] that can be read in place (its rows on 16 bytes, whole 16-byte chunks of columns), or -1: it is transposed first
// and `cfg`, best_tile's choice for the transposed one, is taken.  Transposing costs its bytes, read and written, and 7.6 us: a kernel more and the
// event behind the GEMM.  Over 200 problems drawn from M 4..8192, N 96..7168, K 256..8192 the choice takes 30 % less time than transposing
// always, is slower by more than 2 % on none, and costs 0.8 % more than the better of both (by more than 5 % on 12, all transposed: the costs
// are those of in-place tiles 4 to 10 % slower than they were then, and they have become faster since).  Both sides, us: 1024 x 3584 x 4096
// 128x128 in place 38.6, transposed 49.6; 57 x 96 x 320 5.8 and 11.2; 30 x 336 x 2624 15.0 and 13.3; two rounds, weights in no cache: 2048 x 3584 x
// 4096 103 and 77, x 1024 33.0 and 33.1.
// Where `cfg` is a numbered tile and the problem has more than one round of them, it is taken: those follow the order that the rows arrive in or
// that the slices are wanted in (agg_set_tile_order, first_slice), the small tiles do not, and the bits must not depend on the order.  In a
// single round all tiles start at once.  (One in a thousand problems of those ranges, by the costs 10 % slower than in place.)
// cfg = -1: the best of the tiles that read in place (they all give the same bits).
inline int tile_kn(int num_cus, int cfg, int M, int N, int K, bool slices = false)
{
    int best = -1;
    double best_cost = 1e300;
    for (const TileCost& k : kTileCosts)
        if (k.cfg == cfg) best_cost = tile_cost(num_cus, k, M, N, K, slices) + kTransposeUs + 4.0 * N * K / kTransposeBytesPerUs;
    if (M > kKsMaxRows || (cfg >= 0 && cfg < TILE_CONFIGS && tile_count(tile_shape(cfg), M, N) > num_cus)) return -1;
    for (const TileCost& k : kTileCostsKn) {
        const double cost = tile_cost(num_cus, k, M, N, K, slices);
        if (cost < best_cost) {
            best_cost = cost;
            best = k.cfg;
        }
    }
    return best;
}

// Upper bound of the grouped GEMM's tile table for one tile shape: sum over experts of ceil(rows / bm) <= P / bm + E, times
// the n-tiles.
inline long long moe_table_entries(long long P, int E, int N, TileShape t) { return (P / t.bm + E) * ((N + t.bn - 1) / t.bn); }
// ... and over the shapes that can be selected by number (128 x 128 is the smallest)
inline long long moe_table_bound(long long P, int E, int N) { return moe_table_entries(P, E, N, {128, 128}); }

// The shape, among those that can be selected by number, that decides whether a reserved table is large enough for a call:
// rounds of tiles over the CUs times the cost of a tile (the small tile is bound by the global->LDS path: about 0.6 of the
// large tile's rate per flop), with segments 15 % above the mean.
inline int table_tile_grouped(int num_cus, long long wanted_rows, int E, int N)
{
    const int cand[3] = {TILE_256x224, TILE_256x256, TILE_128x128};
    const double eff[3] = {1.0, 1.0, 0.6};
    const double rows = 1.15 * (double)wanted_rows / E;
    double best = 1e300;
    int cfg = cand[0];
    for (int i = 0; i < 3; ++i) {
        const TileShape ts = tile_shape(cand[i]);
        const long long mt = (long long)((rows + ts.bm - 1) / ts.bm);
        const long long tiles = (long long)E * mt * ((N + ts.bn - 1) / ts.bn);
        const long long waves = (tiles + num_cus - 1) / num_cus;
        const double cost = (double)waves * ts.bm * ts.bn / eff[i];
        if (cost < best) { best = cost; cfg = cand[i]; }
    }
    return cfg | TILE_K32;
}

// Expected number of tiles of `bm` rows of a segment of `mean` rows on average, its length spread around that like that of a
// random routing (standard deviation sqrt(mean)): sum over k of P(length > k * bm).
inline double expected_m_tiles(double mean, int bm)
{
    const double sd = std::sqrt(mean);
    // up to nine standard deviations below the mean a term is 1 (to the last bit): those are counted, not computed -- of a
    // segment of 4 M rows the sum took 0.3 ms of host time per call
    const long long whole = std::max(0ll, (long long)((mean - 9.0 * sd) / bm));
    double n = 1.0 + (double)whole;
    for (long long k = whole + 1; k * (double)bm < mean + 3.0 * sd; ++k) n += 0.5 * std::erfc((k * (double)bm - mean) / (sd * std::sqrt(2.0)));
    return n;
}

// The same for the grouped GEMM, where every tile has a weight matrix of its own to pull.  Fitted to the measured times of every
// tile for 740 problems drawn from 4 to 8192 tokens, 4 to 64 experts, top-1 to 4, N 96 to 2048, K 64 to 4096 (gathered rows in bf16
// and fp32, rows in place): the choice costs 0.7 % more than the best tile of each (geometric mean; 0.8 % on 370 other draws) and takes
// 12 % less time than the choice among 256x224, 256x256 and 128x128 alone, which is faster by more than 5 % on 12 of the 1110, by
// more than 10 % on two.  The costs of the tiles of gemm_pipe.h are fitted to 800 further draws.  On 1226 others, all such that the choice
// without them is a numbered tile, they take the place of one in 333 of 766 for gathered rows, which then take 6.3 % less time (all: 2.8 %), and
// in 31 of 460 for rows in place (3.8 % less); 37 of the 333 are slower by more than 5 %, 20 by more than 10 % (1168 tokens x 4,
// 6 x 1695 x 384: 32.9 and 24.8): of those about half have tiles that are estimated to just fill their last round and do not quite fit into
// it, which depends on the routing.  (An estimate with the spread of the number of tiles does no better on average.)
constexpr TileCost kTileCostsGrouped[] = {
    {KS_16x32, 3.4, 0.113}, {KS_16x64, 3.4, 0.179}, {KS_32x32, 2.6, 0.142}, {KS_64x64, 3.3, 0.267}, {KS_64x128, 3.5, 0.40},
    {TILE_128x128 | TILE_K32, 3.0, 0.60}, {TILE_128x256 | TILE_K32, 2.9, 0.94}, {TILE_256x224 | TILE_K32, 4.1, 1.50},
    {TILE_256x256 | TILE_K32, 4.0, 1.73},
    {PIPE_128x192, 3.7, 0.742}, {PIPE_128x224, 3.2, 0.894}, {PIPE_192x192, 2.7, 1.013}, {PIPE_320x128, 3.5, 0.997},
};
constexpr double kGroupedStoreBytesPerUs = 82e3;     // fp32 rows, per compute unit
constexpr double kGroupedWeightBytesPerUs = 7.2e6;   // weights of the experts that have rows, whole chip

// Tile shape of a grouped GEMM: `rows` rows of A spread over E experts, [N][K] weights per expert.  Rounds of tiles times
// the cost of a tile, as in best_tile, but not less than the weights of the experts that have rows take from HBM; where they
// bound it, a last round that fills only part of the chip costs its share of that time, and the smaller tile wins.  Measured,
// us per call with routing, bf16 out, Table 4: 64 tokens (two rows per expert) 16x64 149, 16x32 154, 64x64 158, 128x128 196; 512
// tokens 64x64 190, 64x128 197, 32x32 197, 128x128 226; 2048 tokens 128x128 232, 64x128 277.  Rows in place with K = 192 and fp32
// out (the GEMM of Table 5, kernel alone, cold): 256x256 70, 128x256 63, 128x128 71.  Gathered rows never take the 128x256 tile of the large
// kernel: at 8192 tokens of Table 4 the whole call is 1 % faster in bf16 (374 against 376) but its first pass on new weights 5 % slower
// (457 against 435), and in fp32 it is 5 % slower throughout (392 against 371); where it would be the best of the numbered tiles, that
// of gemm_pipe.h is faster.  There, with routing, weights beyond the memory-side cache, us: 8192 tokens 320x128 291, 128x256 330, 256x256 335,
// 256x224 368; 4096 tokens 192x192 232, 320x128 254, 256x256 267.
// A tile of gemm_pipe.h takes the place of a numbered one, whose bits it gives, never of a K-split one.
// Which K-split tile is taken, or that another one is, follows from the problem alone: the small tiles and those of gemm_pipe.h are left
// out where their table (P pairs) would have more entries than the static one, whatever table is used.  Among the numbered ones, which all give
// the same bits, those are left out whose table would have more than `tab_base` entries; -1 if that is all of them.
inline int best_tile_grouped(int num_cus, long long rows, int E, int N, int K, bool gathered, bool f32, long long P,
                             long long tab_base, bool large_only = false)
{
    const double active = E * (1.0 - std::pow(1.0 - 1.0 / E, (double)rows));       // experts with at least one row
    const double hbm_us = active * N * K * 2.0 / kGroupedWeightBytesPerUs;
    int best = -1, best_that_fits = -1, best_pipe = -1;
    double best_cost = 1e300, fits_cost = 1e300, pipe_cost = 1e300;
    for (const TileCost& k : kTileCostsGrouped) {
        const TileShape t = tile_shape(k.cfg);
        const bool small = k.cfg >= TILE_CONFIGS, numbered = k.cfg < TILE_NUMBERED, pipe = !small && !numbered;
        const long long entries = moe_table_entries(P, E, N, t);
        if ((small && large_only) || (!numbered && entries > kStaticTabEntries) || (gathered && numbered && t.bm == 128 && t.bn == 256)) continue;
        // a tile of gemm_pipe.h that is nearly empty: the weights' bytes are what counts, and the small tiles ask for more of them at a
        // time (48 tokens, 3 rows per expert, 29 x 1659 x 2304: 128x192 72 us, 16x64 50)
        if (pipe && (double)rows < active * t.bm / 8) continue;
        const double tiles = active * expected_m_tiles((double)rows / active, t.bm) * ((N + t.bn - 1) / t.bn);
        const double rounds = std::ceil(tiles / num_cus);
        // ... or, rows in place (short K, fp32 out), a single round of them: there is no next tile whose loads could be under way beside the
        // stores, and the numbered tiles start and end sooner.  Over 460 draws the call with them takes, in one round, 3.5 % longer than with
        // the numbered choice (1064 tokens x 2, 25 x 1308 x 192: 32.6 and 29.2), in more 4 % less (7896 x 4, 9 x 576 x 512: 71.4 and 84.5)
        if (pipe && !gathered && rounds < 2.0) continue;
        const double tile_us = k.fixed_us + k.us_per_k64 * (K / 64) + (f32 ? t.bm * t.bn * 4 / kGroupedStoreBytesPerUs : 0.0);
        const double cost = std::max(rounds * tile_us, hbm_us * rounds * num_cus / std::max(tiles, (double)num_cus));
        if (!pipe && cost < best_cost) {
            best_cost = cost;
            best = k.cfg;
        }
        if (pipe && cost < pipe_cost) {
            pipe_cost = cost;
            best_pipe = k.cfg;
        }
        if (numbered && entries <= tab_base && cost < fits_cost) {
            fits_cost = cost;
            best_that_fits = k.cfg;
        }
    }
    if (best >= TILE_CONFIGS) return best;
    return pipe_cost < best_cost ? best_pipe : best_that_fits;
}

// Worlds and slots (below 2 GiB, for 32-bit offsets) of reduce_flow_kernel, whose loads never stop.  Above, two slots of 2 GiB take 1157 us
// with the kernel for any world, eight 3790.
inline bool reduce_flows(int W, long long n_vec4) { return (W == 8 || (W >= 2 && W <= 4)) && n_vec4 < (1ll << 27); }

// Workgroups, and threads of one, of a reducer launch over n_vec4 float4 whose caller leaves the size to the library.  Persistent, each walking
// many blocks of a float4 per thread (one acquire per workgroup, not per block).  (Of a size that the caller names: 256 threads.)  A reducer may have to wait for a GEMM that is launched after it,
// which has to find room: of 512 registers per SIMD lane a workgroup of any of the reducers takes 64, a large GEMM tile 448, a K-split tile up
// to 384 (128x128 with a [K][N] operand; 288 and less the others).  A GEMM that finds none runs into the time limit of the reducer's wait.
//   Loads that never stop: what counts is that few streams are in flight, and beside a GEMM that every CU has the same share of them (the
//     GEMM's tiles wait for the slowest CU).  One workgroup of three waves per CU; two to four slots with nothing beside them take seven
//     of four waves per eight CUs.  Room for any GEMM on every CU.
//     Eight slots of 1024 x 8192, us per call, slots not touched lately, by workgroups of four waves, 128 / 192 / 224 / 256 / 512 of them, and 256 of
//     three: 60.7 / 52.9 / 53.4 / 58.6 / 59.0 and 50.8; 200 x 4000 9.4 / 9.2 / . / 9.5 / 11.3 and 9.1.  224 of four waves and 256 of three: four of
//     1024 x 8192 32.1 and 32.4, three 26.9 and 27.5, two 22.1 and 22.8.
//     Beside the next call's GEMM (8192 x 8192 x 3584 on 8 ranks, calls that do not wait for the one before), us per call: 192 of four waves 388,
//     256 of three 380, a loop that drains at every block, 256 of four waves, 375; own slice first 391, 380 and 375; in four chunks 393, 387 and 383.
//     Behind its own GEMM, calls that wait: 421, 417 and 430; 8192 x 8192 x 1024 222, 218 and 233.
//   Any world: three per two CUs, room for a K-split tile on every CU and for a large one on half of them; beside a GEMM one per CU.  At 1 /
//     1.25 / 1.5 / 2 per CU six slots of 1024 x 8192 take 46.2 / 48.4 / 46.4 / 46.3, sixteen 95.5 / 109 / 104 / 99.1; at 1 and 1.5 nine of 300 x 2000
//     10.9 and 9.8, six of 1024 x 8192 in sixteen chunks 64.9 and 56.4, two of 2 GiB 1302 and 1157.
struct ReduceShape {
    int workgroups, threads;
};
inline ReduceShape reduce_shape(int W, int num_cus, long long n_vec4, bool beside_gemm)
{
    const bool flows = reduce_flows(W, n_vec4), three_waves = flows && (W == 8 || beside_gemm);
    const int threads = three_waves ? 192 : 256;
    const long long need = (n_vec4 + threads - 1) / threads;
    const long long want = three_waves || beside_gemm ? num_cus : flows ? num_cus * 7ll / 8 : num_cus * 3ll / 2;
    const long long n = need < want ? need : want;
    return {n < 1 ? 1 : (int)n, threads};
}

}  // namespace agg
