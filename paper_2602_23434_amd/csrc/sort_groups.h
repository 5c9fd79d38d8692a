// Which items of a sort call share one radix sort (SortGroup in k_sort.hip):
// the rules that the launcher goes by.  Host arithmetic only, so that a plain
// C++ compiler takes it.
#pragma once

#include <stdint.h>

namespace pl {

constexpr int kGroup = 8;            // items sorted together at most

inline int bits_for(uint64_t count)
{
    int b = 0;
    while (b < 32 && ((uint64_t)1 << b) < count) ++b;
    return b;
}

// 8-bit digits of `keys` distinct keys.
inline int sort_passes(uint64_t keys)
{
    const int b = bits_for(keys);
    return ((b > 1 ? b : 1) + 7) / 8;
}

// A group under construction: its particles, its distinct keys, and the most
// keys of one of its items.
struct GroupSize {
    int64_t np = 0;
    uint64_t keys = 0, most = 0;
};

// Whether an item of np particles and `keys` distinct keys joins a group:
// while the scratch holds the particles (cap), the keys stay below the run
// table's sentinel 2^32 - 1 (k_runs_build marks "no neighbour" with it, so no
// particle may have it as its key), and the group takes at most one pass more
// than its largest item.
inline bool group_takes(const GroupSize &g, int64_t np, uint64_t keys, int64_t cap)
{
    const uint64_t most = g.most > keys ? g.most : keys;
    return g.np + np <= cap && g.keys + keys <= 0xffffffffull && sort_passes(g.keys + keys) <= sort_passes(most) + 1;
}

}  // namespace pl
