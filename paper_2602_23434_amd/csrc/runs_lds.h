// LDS layout of the run kernel.  Host and device arithmetic without HIP's types,
// so that a plain C++ compiler takes it (constexpr: for both sides).
#pragma once

#include <stddef.h>

namespace pl {

constexpr size_t runs_section(size_t b) { return (b + 15) & ~(size_t)15; }

// Capacity of the queue of particles that need the HBM gather: with a
// two-cell field halo only particles two cells out of their tile land there.
constexpr int gq_cap(int hf) { return hf == 2 ? 64 : 256; }

// Threads of the small blocks, and capacity of the queue of deposits outside
// their batch's cell: float32, what the LDS leaves beside every channel and a
// two-cell field halo on 8^3 tiles; float64, 128 less what the control words below
// take, so that no tile is refused for them.
constexpr int kRunsSmall = 256;
constexpr int runs_queue(size_t real, int threads) { return threads == kRunsSmall ? 64 : real == 4 ? 192 : 116; }

constexpr int kRunsGroups = 64;        // entries of the launch's unit table
constexpr int kRunsCtlBytes = 64 + 4 * kRunsGroups;

// Sections of one work unit (offs): field records of `rec` reals for Lf cells,
// float64 deposit tile of Ld cells and nslot channels, the two queues, sums;
// control words at the end.  Bytes in all.
constexpr size_t runs_lds_layout(size_t real, int rec, int Lf, int Ld, int nslot, int hf, int threads, size_t offs[6])
{
    const int dq = runs_queue(real, threads);
    size_t o = 0;
    offs[0] = o; o += runs_section((size_t)Lf * rec * real);
    offs[1] = o; o += runs_section((size_t)Ld * nslot * sizeof(double));
    offs[2] = o; o += runs_section((size_t)gq_cap(hf) * sizeof(int));
    offs[3] = o; o += runs_section((size_t)dq * sizeof(int));
    offs[4] = o; o += runs_section((size_t)dq * (3 + nslot) * real);
    offs[5] = o; o += 8 * sizeof(double);
    return o + kRunsCtlBytes;
}

}  // namespace pl
