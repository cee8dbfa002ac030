// Work list of the batched products.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace rpyw {

// An item: the targets from `target` on of the system of blobs [begin, end),
// against a share of its sources, `share` = number of the share + 256 times the
// number of the system's shares (the kernels read it as an int4).
struct BatchedItem {
    int begin, end, target, share;
};

// A system's sources are shared out at whole tiles of the kernel: `parts` shares
// or fewer of share_tiles tiles (the same with used_parts for parts).
constexpr int share_tiles(int tiles, int parts) { return (tiles + parts - 1) / parts; }
constexpr int used_parts(int tiles, int parts) {
    return (tiles + share_tiles(tiles, parts) - 1) / share_tiles(tiles, parts);
}

// Parts into which the sources are split, so that there are about
// kBatchedItems items of work: 1024 to 1280 run at a time, and the large
// systems' items are long (few systems are a serial pass over all sources on a
// few workgroups; many end unevenly).  A call, before and now: two
// systems of up to 5000 blobs, FP32C, 80 -> 30 us; 14 of up to 11000, 8
// right-hand sides, FP64, 4.9 -> 2.4 ms; 64 of up to 12000, 4 right-hand sides,
// FP64, 5.7 -> 3.4 ms; 64 of up to 17000, 16 right-hand sides, FP32C, 11.1 ->
// 10.9 ms.  Twice as many items lose up to 12%.
constexpr int64_t kBatchedItems = 8192;
constexpr int kBatchedMaxParts = 64;
// items: with one part, which is at least `blobs` / span.
inline int batched_parts(int64_t items, bool mat) {
    // (rounded down where the partial sums of a part are the larger: span 256)
    return (int)std::max<int64_t>(
        1, std::min<int64_t>(kBatchedMaxParts, (kBatchedItems + (mat ? items - 1 : 0)) / items));
}

// Systems of fewer than split_from(...) blobs stay whole: those below
// kBatchedShort once the items fill the GPU (kBatchedFull), for then the sums of
// the parts and their epilogue cost more than the split gives; from one item for
// each of 256 compute units on if that is all of them and an item's sums are
// large for its work (matrix cores, systems of one span).  A call, split into
// all tiles and whole: 480 systems of 200, FP64, 122 and 101 us; 2000 of 80 169
// and 154; 300 of 300, 8 right-hand sides, FP32C, 204 and 171; 100 of 200 69 and
// 54.  200 of 300 (400 items), FP64, 130 and 140.
constexpr int64_t kBatchedShort = 768;
constexpr int64_t kBatchedFull = 416;
inline int64_t split_from(int64_t items, bool mat, int64_t nmax, int span) {
    const bool few = items < kBatchedFull && !(items >= 256 && nmax < kBatchedShort && (mat || nmax <= span));
    return few ? 0 : kBatchedShort;
}

// Work list, longest items first (LPT order): spans of targets against each
// share of each system.  Returns the most shares of a system.  Small
// systems have one or few shares, whatever the largest one has: an item costs
// some 25 ns here and in its upload and 12 ns of the work counter (an item for
// each part of each of 20000 systems of 1 to 4 blobs beside one of 2000 took 8.0
// ms, one item for each 0.7).
inline int batched_items(const int64_t* sys_offsets, int S, int span, int tile, int parts, int64_t from,
                         int64_t whole, std::vector<BatchedItem>& items) {
    auto size = [&](int s) { return sys_offsets[s + 1] - sys_offsets[s]; };
    auto used = [&](int s) {
        return parts > 1 && size(s) >= from ? used_parts((int)((size(s) + tile - 1) / tile), parts) : 1;
    };
    std::vector<int> order(S);
    for (int s = 0; s < S; ++s) order[s] = s;
    if (parts == 1)
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return size(x) > size(y); });
    else
        std::stable_sort(order.begin(), order.end(),
                         [&](int x, int y) { return size(x) * used(y) > size(y) * used(x); });
    items.clear();
    items.reserve((size_t)whole);
    int most = 1;
    for (int s : order) {
        const int b0 = (int)sys_offsets[s], b1 = (int)sys_offsets[s + 1], n = used(s);
        most = std::max(most, n);
        for (int p = 0; p < n; ++p)
            for (int t = b0; t < b1; t += span) items.push_back({b0, b1, t, p + 256 * n});
    }
    return most;
}

}  // namespace rpyw
