// When the expansion (expand_kernels.hip) takes a call, and how it cuts the
// call's x entries into workgroup tiles.  Plain host C++: the rule is tested
// without a GPU.  Not installed.
#pragma once

#include <algorithm>
#include <stdint.h>

namespace spv {

constexpr int kLongCol = 2047;   // longest column it takes

struct ExpandTiles {
    bool taken;    // else scan and scatter
    int per;       // x entries per tile (f known on the host)
    int per_min;   // bounds of a tile whose f is known on the device only
    int per_max;
    int grid;      // workgroups
};

// A tile's products are one workgroup's work, chunk after chunk, whatever
// columns x lists, where the scatter cuts all products into equal chunks.  So a
// tile of `per` entries may hold at most 8192 products or two chunks more than
// twice its mean (10 us or less), whichever columns x lists.  Matrices whose
// columns are about equally long (grids) pass at any size; others while there
// are workgroups enough for tiles that small.  Past that, tiles that small are
// dealt out in turn where they still fill a chunk on average, and the call
// goes to scan and scatter where they do not.
//
// Measured on 1M columns of 4 to 2047 entries, the longest first, 60M in all:
// with the longest column as the only limit the 16 / 256 / 32768 heaviest
// columns took 85 / 91 / 263 us, PageRank 49.2 ms and a push BFS 1.29 ms; with
// this rule 45 / 47 / 105 us, 19.0 and 0.53 ms.  4096 random columns of it
// take 38 us expanded and 52 with scan and scatter, where they go now because
// the heaviest 4096 take 129 and 100.  Columns of 10 to 50 entries: 59 us for
// 20000 of them, as before.
//
// A tile takes slots with one counter update per bucket that it touches, for a
// thin tile about one per product: beyond one tile per compute unit, tiles are
// as wide as fills a chunk.  A multiply of 16384 / 65536 random columns of 1M
// with 8 entries each, back to back: 33.7 / 42.9 us with a tile for every
// workgroup that could be resident, 18.5 / 24.3 this way, 23.3 / 32.3 with scan
// and scatter; sixteen columns of 300 entries 20.0 us in one tile, 13.4 in eight.
// With a device-known f every workgroup gets the same number of tiles:
// PageRank over 300,000 columns of 50, whose tiles of 1024 entries left one
// round in eight to 37 of 256 workgroups, 5.8 -> 4.6 ms.
//
// f < 0: known on the device only, at most n.  gmax: workgroups resident at once.
inline ExpandTiles expand_tiles(int64_t n, int64_t nnz, int64_t longest, int64_t f, int block, int chunk, int gmax,
                                int num_cu) {
    const double mean = std::max(1.0, n > 0 ? (double)nnz / (double)n : 1.0);   // products per x entry
    // one chunk's worth, with room for uneven columns
    const int64_t one = std::min<int64_t>(block, std::max<int64_t>(1, (int64_t)(0.85 * chunk / mean)));
    const double uneven = (double)longest - 2.0 * mean, extra = std::max(8192.0, 2.0 * chunk);
    const int64_t most =
        uneven > 0.0 ? std::max<int64_t>(1, (int64_t)std::min((double)block, extra / uneven)) : block;
    const bool fill = most >= one;   // several tiles per workgroup are no loss
    auto parts = [](int64_t count, int64_t size) { return (count + size - 1) / size; };
    ExpandTiles t{};
    t.per_min = (int)std::min<int64_t>({16, one, most});
    t.per_max = (int)most;
    if (f < 0) {   // a tile per workgroup, if x is no longer than that
        t.taken = fill || std::min<int64_t>(block, parts(n, gmax)) <= most;
        t.per = t.per_min;
        t.grid = gmax;
    } else {
        int64_t per = std::min(std::max<int64_t>(parts(f, num_cu), t.per_min), one);
        if (parts(f, per) > gmax) per = std::min<int64_t>(block, parts(parts(f, gmax), one) * one);   // several chunks
        per = std::min(per, most);
        t.taken = fill || parts(f, per) <= num_cu;
        t.per = (int)per;
        t.grid = (int)std::max<int64_t>(1, std::min<int64_t>(parts(f, per), gmax));
    }
    t.taken = t.taken && longest <= kLongCol;
    return t;
}

}  // namespace spv
