// The host-side rules of the library behind plain C functions, for the tests that check them without a GPU.
#include "delivered.h"
#include "ks_stage.h"
#include "launch_rules.h"
#include "moe_table.h"

#include <cstdlib>
#include <map>

using namespace agg;

extern "C" {

// Plays agg_reserve_moe(entries[0]), ..(entries[n - 1]) on one context; allocation number k fails where fails[k] is set.  For
// each call: its return code, whether there is a table, the entries that can really be stored in it, and what the calls
// may assume of it (the reservation, and the fixed size that the small tiles go by).
void moe_reserve_play(int n, const long long* entries, int n_allocs, const int* fails, int* rc, int* has_table, long long* room,
                      long long* base, int* leaked)
{
    MoeWorkspace w{};
    std::map<char*, size_t> live;
    int k = 0;
    auto take = [&](void** p, size_t bytes) {
        if (k < n_allocs && fails[k++]) return -6;
        *p = std::malloc(64);                     // an address of its own; nothing is stored there
        live[(char*)*p] = bytes;
        return 0;
    };
    for (int i = 0; i < n; ++i) {
        rc[i] = moe_workspace_reserve(w, entries[i], take, take, [&](void* p) { live.erase((char*)p); std::free(p); });
        has_table[i] = w.tab != nullptr;
        base[i] = w.base;
        room[i] = 0;
        for (const auto& a : live)
            if ((char*)w.tab == a.first) room[i] = (long long)(a.second / kMoeTileBytes);
            else if (w.ctrl && (char*)w.ctrl == a.first && (char*)w.tab == a.first + kStaticTabOffset)
                room[i] = (long long)((a.second - kStaticTabOffset) / kMoeTileBytes);
    }
    const size_t held = (w.ctrl ? 1u : 0u) + (w.tab_large ? 1u : 0u);
    *leaked = (int)(live.size() - held);
    for (const auto& a : live) std::free(a.first);
}

// Every 16-byte access of stages 0 .. KC + past - 1 of a tile of `tile_rows` rows, of which `rows` exist, each `ld` bytes apart and
// 64 KC elements long: the number of accesses that a bounds check lets through outside the rows, for both ways in which it
// may treat the scalar offset (added to the lane's, or taken from the size, modulo 2^32), plus those it holds back inside.
int ks_stage_bad_accesses(int KC, int past, int rows, int tile_rows, unsigned ld)
{
    int bad = 0;
    const unsigned bytes = (unsigned)rows * ld;
    for (int s = 0; s < KC + past; ++s) {
        const KsStage st = ks_stage(s, KC, 128, bytes);
        for (int row = 0; row < tile_rows; ++row)
            for (unsigned chunk = 0; chunk < 8; ++chunk) {
                const unsigned lane = (unsigned)row * ld + chunk * 16;
                const bool wanted = s < KC && row < rows;
                const bool added = (unsigned long long)lane + (unsigned)st.k_off < st.bytes;
                const bool taken = lane < (unsigned)(st.bytes - (unsigned)st.k_off);
                bad += (added != wanted) + (taken != wanted);
            }
    }
    return bad;
}

int reduce_grid(int W, int num_cus, long long n_vec4, int beside_gemm) { return reduce_shape(W, num_cus, n_vec4, beside_gemm != 0).workgroups; }

int reduce_threads(int W, int num_cus, long long n_vec4, int beside_gemm) { return reduce_shape(W, num_cus, n_vec4, beside_gemm != 0).threads; }

// n calls on one context: kind[i] 0 = a copy of the shards ranks[i] launched with epoch[i] on stream[i], 1 = a GEMM.  kept[i]: that stream keeps
// order.  answer[i]: the GEMM is behind all of them; asked[i]: how often the runtime was asked about the stream.
void delivered_play(int W, int n, const int* kind, const unsigned long long* ranks, const int* epoch, const long long* stream, const int* kept,
                    int* answer, int* asked)
{
    Delivered d;
    for (int i = 0; i < n; ++i) {
        asked[i] = 0;
        auto ask = [&] { ++asked[i]; return kept[i] != 0; };
        answer[i] = 0;
        if (kind[i] == 0) d.note(ranks[i], epoch[i], (const void*)stream[i], ask);
        else answer[i] = d.all(W, epoch[i], (const void*)stream[i], ask);
    }
}

double m_tiles(double mean, int bm) { return expected_m_tiles(mean, bm); }

// The same sum term by term, as it is defined.
double m_tiles_plain(double mean, int bm)
{
    const double sd = std::sqrt(mean);
    double n = 1.0;
    for (long long k = 1; k * (double)bm < mean + 3.0 * sd; ++k) n += 0.5 * std::erfc((k * (double)bm - mean) / (sd * std::sqrt(2.0)));
    return n;
}

int tile_plain(int num_cus, int M, int N, int K, int slices) { return best_tile(num_cus, M, N, K, slices != 0); }

// The tile of a [K][N] operand that can be read in place, -1 = transposed first.
int tile_of_kn(int num_cus, int M, int N, int K, int slices) { return tile_kn(num_cus, best_tile(num_cus, M, N, K, slices != 0), M, N, K, slices != 0); }

int tile_rows_and_columns(int tile) { return tile_shape(tile).bm << 16 | tile_shape(tile).bn; }

// The K-split tiles that the automatic choice can take; returns how many.
int ks_tiles(int grouped, int* out)
{
    int n = 0;
    auto add = [&](const TileCost& k) {
        if (k.cfg >= TILE_CONFIGS) out[n++] = k.cfg;
    };
    if (grouped) for (const TileCost& k : kTileCostsGrouped) add(k);
    else for (const TileCost& k : kTileCosts) add(k);
    return n;
}

int tile_grouped(int num_cus, long long rows, int E, int N, int K, int gathered, int f32, long long P, long long tab_base, int large_only)
{
    return best_tile_grouped(num_cus, rows, E, N, K, gathered != 0, f32 != 0, P, tab_base, large_only != 0);
}

long long static_table_entries() { return kStaticTabEntries; }

}
