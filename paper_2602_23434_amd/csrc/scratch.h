// Size of the context's one allocation for the sort's keys and indices (four
// 4-byte words per particle), which between sorts also holds the spectral update's
// fluid records, 64 bytes for every cell of a box.  With four particles per cell or
// more the records need nothing beyond the keys.  With fewer, down to one, the
// allocation grows for them, but by no more than kRecordsExtra: a context that
// never touches a spectrum would otherwise take up to four times the sort's
// scratch (1024^3 cells and as many particles: 69 GB instead of 17).  Boxes
// beyond it sample the fields.  Host arithmetic only, so that a plain C++ compiler
// takes it.
#pragma once

#include <stdint.h>

namespace pl {

constexpr int64_t kRecordsExtra = 64ll << 20;

inline int64_t keys_bytes(int64_t max_np) { return 16 * ((max_np + 63) & ~(int64_t)63); }

// Bytes to ask for; keys_bytes alone does where there is no room for more.
inline int64_t slab_bytes(int64_t max_np, int64_t max_cells)
{
    const int64_t keys = keys_bytes(max_np), records = 64 * max_cells;
    return max_cells <= max_np && records > keys && records <= keys + kRecordsExtra ? records : keys;
}

}  // namespace pl
