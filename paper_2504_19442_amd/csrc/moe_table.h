// The tile table of the grouped GEMM as a context holds it: how large it has to be for a problem, and what agg_reserve_moe
// does to it.  Plain C++, so that an allocation that fails can be played through without a GPU.
#pragma once
#include <stddef.h>

namespace agg {

struct MoeTile;

constexpr int kMoeMaxExperts = 4096;
// Control block of the MoE routing: the tile count (int, read by the grouped GEMM), the number of finished routing
// calls, the ticket counter, and two tagged counts per expert (its pairs; those of them that get tiles).
constexpr size_t kMoeCtrlCall = 8, kMoeCtrlTicket = 16, kMoeCtrlCounts = 256;
constexpr size_t kMoeCtrlKept = kMoeCtrlCounts + (size_t)kMoeMaxExperts * 8;
constexpr size_t kMoeCtrlBytes = kMoeCtrlKept + (size_t)kMoeMaxExperts * 8;

// The table behind the control block, of a fixed size.  The K-split tiles of the automatic choice are taken up to this many
// entries whatever was reserved, so every table that is in use holds at least as many.
constexpr size_t kMoeTileBytes = 32;
constexpr long long kStaticTabEntries = 32760;
constexpr size_t kStaticTabOffset = kMoeCtrlBytes;
constexpr size_t kStaticScratchBytes = kStaticTabOffset + kStaticTabEntries * kMoeTileBytes;   // 1088 KiB

struct MoeWorkspace {
    int* ctrl;            // the control block (its first word is the tile count of the launch under way), the fixed table behind it
    MoeTile* tab;         // the table in use: the fixed one, or tab_large
    MoeTile* tab_large;
    long long cap;        // entries of the table in use: at least kStaticTabEntries, and at least ...
    long long base;       // ... as many as agg_reserve_moe was asked for
};

// A table of `entries`.  alloc(void**, bytes) and alloc_ctrl(void**, bytes) (control block zeroed) return 0 or an error code;
// release(void*) gives back what alloc gave.  An error leaves the workspace as usable as it was.
template <class AllocCtrl, class Alloc, class Release>
int moe_workspace_reserve(MoeWorkspace& w, long long entries, AllocCtrl&& alloc_ctrl, Alloc&& alloc, Release&& release)
{
    void* p = nullptr;
    if (!w.ctrl) {
        if (int rc = alloc_ctrl(&p, kStaticScratchBytes)) return rc;
        w.ctrl = (int*)p;
        w.tab = (MoeTile*)((char*)p + kStaticTabOffset);
        w.cap = kStaticTabEntries;
    }
    if (w.cap < entries) {
        if (int rc = alloc(&p, (size_t)entries * kMoeTileBytes)) return rc;      // (the table in use stays until there is a larger one)
        if (w.tab_large) release(w.tab_large);
        w.tab = w.tab_large = (MoeTile*)p;
        w.cap = entries;
    }
    if (w.base < entries) w.base = entries;
    return 0;
}

}  // namespace agg
