// Which tiles the run kernel takes in the float32 form, and which particles of a
// batch join its deposit sums: a rule on sizes alone.  The kernel sums up to four
// particles' deposits in float32 before a float64 LDS atomic; the kernels that
// take what it leaves add float64 products one by one or in float64 sums.  So
// the grids' last bits depend on which of them runs, and on which particles join
// a batch.  Both go by this fixed footprint, not by what the kernel needs today,
// so that a leaner kernel does not change a grid: 32-byte field records of charged
// particles (16 bytes of others), queues of 256 deposits.
//  * with a two-cell field halo: particles up to one cell outside the tile join
//    the sums where this footprint fits the LDS, else those inside the tile only;
//  * with a one-cell halo: the run kernel takes the tile where this fits.
// Host arithmetic only, so that a plain C++ compiler takes it.
#pragma once

#include <stddef.h>

namespace pl {

// Bytes for one item's tile T (cells per dimension) with `nslot` channels.
inline size_t runs_sums_bytes(bool charged, const int T[3], int ndim, int nslot, int hf)
{
    auto section = [](size_t b) { return (b + 15) & ~(size_t)15; };
    auto cells = [&](int h) { return (size_t)(T[0] + 2 * h) * (T[1] + 2 * h) * (ndim >= 3 ? T[2] + 2 * h : 1); };
    const size_t queue = 256, far = hf == 2 ? 64 : 256;
    return section(cells(hf) * (charged ? 32 : 16)) + section(cells(2) * nslot * 8) + far * 4 + queue * 4 +
           queue * (size_t)(3 + nslot) * 4 + 80;
}

}  // namespace pl
