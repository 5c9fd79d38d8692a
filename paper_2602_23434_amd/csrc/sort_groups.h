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
//  * the scratch holds the particles (cap);
//  * the keys stay below the run table's sentinel 2^32 - 1 (k_runs_build marks "no
//    neighbour" with it, so no particle may have it as its key);
//  * the digits' passes stay as many as its largest item's, or the group is small:
//    one pass more over all its particles costs more than the launches that
//    sorting the item by itself takes.  us per sort, together and apart: 256^3 cells,
//    whose 2^24 keys take three passes and with any other item four, 1e6 particles
//    with 5000 on 32^3 602 and 627, 4e6 802 and 823, 2^24 1810 and 1774; 1e6 with 5e5
//    979 and 1115.
constexpr int64_t kExtraPass = 1 << 22;
inline bool group_takes(const GroupSize &g, int64_t np, uint64_t keys, int64_t cap)
{
    const uint64_t most = g.most > keys ? g.most : keys;
    if (g.np + np > cap || g.keys + keys > 0xffffffffull) return false;
    return sort_passes(g.keys + keys) <= sort_passes(most) + (g.np + np <= kExtraPass ? 1 : 0);
}

// Memory that the items of a group read and write.  Sorted one after another,
// an item may write what an earlier one has read (a spare set of arrays handed
// from item to item) or written; in one launch it may not.
struct GroupMemory {
    static constexpr int kPerItem = 32;
    struct Range {
        uintptr_t beg, end;
        int item;
        bool write;
    };
    Range all[kGroup * kPerItem];        // by address
    int n = 0;

    // Add an item's ranges (at most kPerItem); false, and nothing added, when a
    // byte that it writes is used by another item of the group, or it uses one
    // that another writes.
    bool add(int item, const Range *mine, int count)
    {
        const int before = n;
        for (int k = 0; k < count; ++k) {
            if (mine[k].end <= mine[k].beg) continue;
            int at = n++;
            for (; at > 0 && all[at - 1].beg > mine[k].beg; --at) all[at] = all[at - 1];
            all[at] = mine[k];
            all[at].item = item;
        }
        bool clash = false;
        for (int a = 0; a < n && !clash; ++a)
            for (int b = a + 1; b < n && all[b].beg < all[a].end && !clash; ++b)
                clash = all[a].item != all[b].item && (all[a].write || all[b].write);
        if (!clash) return true;
        int kept = 0;
        for (int k = 0; k < n; ++k)
            if (all[k].item != item) all[kept++] = all[k];
        n = before;
        return false;
    }
};

}  // namespace pl
