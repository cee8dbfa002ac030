// The batched products' work list (batched_plan.h), exported for the host tests.
#include "../../paper_1709_02410_amd/csrc/batched_plan.h"

using namespace rpyw;

// Items {begin, end, target, share} of S systems: returns their
// number, *parts the most shares of a system.  whole: items with one part.
extern "C" int64_t host_batched_plan(const int64_t* offsets, int S, int span, int tile, int mat, int64_t whole,
                                     int* parts, int* out, int64_t room) {
    int64_t nmax = 0;
    for (int s = 0; s < S; ++s) nmax = std::max(nmax, offsets[s + 1] - offsets[s]);
    std::vector<BatchedItem> items;
    *parts = batched_items(offsets, S, span, tile, batched_parts(whole, mat != 0),
                           split_from(whole, mat != 0, nmax, span), whole, items);
    for (size_t i = 0; i < items.size() && (int64_t)(4 * i + 3) < room; ++i) {
        out[4 * i] = items[i].begin;
        out[4 * i + 1] = items[i].end;
        out[4 * i + 2] = items[i].target;
        out[4 * i + 3] = items[i].share;
    }
    return (int64_t)items.size();
}

extern "C" int host_share_tiles(int tiles, int parts) { return share_tiles(tiles, parts); }
extern "C" int host_used_parts(int tiles, int parts) { return used_parts(tiles, parts); }
