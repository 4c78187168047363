// Groups of representatives that a frame keeps a K-means bound for (k_lloyd_assign).  Plain C++: tests/test_lloyd_groups.py compiles it for the host.
#pragma once

namespace mosaic {

constexpr int kLloydGroups = 7;     // groups
constexpr int kLloydTiles = 64;     // tiles of 16 ids in the table of a context's 1024 clusters at most

// A frame's candidates -- the Cs ids of its visual partition, or all C without partitions (P = 0) -- span `span` tiles of 16 ids at most, counted from the
// tile of its first candidate; group g has tiles lo(g) .. lo(g + 1) - 1 of them.
struct LloydGroups {
    int span;
    constexpr LloydGroups(int P, int Cs, int C) : span(0) {
        const int table = (C + 15) / 16;            // (no candidate lies beyond it: a single partition of 1015 ids has 64 tiles, wherever it begins)
        span = P <= 0 ? table : Cs % 16 == 0 ? Cs / 16 : (Cs + 14) / 16 + 1;
        if (span > table) span = table;
    }
    constexpr int lo(int g) const { return span <= kLloydGroups ? (g < span ? g : span) : (g * span + kLloydGroups - 1) / kLloydGroups; }
    constexpr int of(int t) const { return span <= kLloydGroups ? t : t * kLloydGroups / span; }
    // tiles of group g of a frame whose candidates lie in tiles t0 .. t1 - 1, as a mask
    constexpr unsigned long long tiles(int g, int t0, int t1) const {
        const int a = t0 + lo(g), e = t0 + lo(g + 1), b = e < t1 ? e : t1;
        return a < b ? (~0ull >> (64 - (b - a))) << a : 0ull;
    }
};

} // namespace mosaic
