// When a plain call bins an item's particle indices by tile and advances them
// tile by tile, and when it leaves them to the direct kernel (one particle per
// thread, deposits as global atomics): a rule on the call as a whole.  Host
// arithmetic only, so that a plain C++ compiler takes it.
//
// The items of a species kind share one direct launch, whose cost is a chain of
// A = 27 (9 in 2D) x channels atomics per lane, half a microsecond each, once, and
// A atomics per particle at 2.4e10 per second.  A binned item has a chain of its
// own: keys, one scatter per 8 bits of its tiles, tile offsets and step (26 us
// with the gaps between them), the longer the more of its tiles a CU takes.  So a
// large item is binned by itself; small ones only where the chains of all of
// them cost less than the one direct chain.  Measured in us per call, binned and
// direct, fused steps on MI355X (float64 unless said; the model agrees to 30 %):
//   charged, one item: 600 on 16^3 42 and 99, 2048 on 64^3 112 and 126, 20000 on 16^3
//     60 and 206, 131079 on 64^3 162 and 1190; 2D 2055 on 32^2 54 and 30, 8199 47 and
//     37, 20000 on 128^2 (float32) 54 and 76;
//   dust, one item: 2048 on 32^3 52 and 68; 2D 8199 on 32^2 46 and 23;
//   charged, k items: 600 on 16^3, k = 2 69 and 102, 4 130 and 103, 64 1890 and 334;
//     20000 on 16^3, k = 2 111 and 365, 64 3312 and 10132; 2D 2048 on 64^2, k = 2 81 and
//     46, 256 9624 and 1407.
#pragma once

#include <stdint.h>

#include "../../include/pl.h"

namespace pl {

// An item of a plain call that deposits, as far as the rule looks.
struct PlainItem {
    int64_t np, tiles;           // tiles of its bins
    int channels;
    bool fits;                   // the bins' scratch and the tile kernel's LDS hold it
    bool binned;                 // the rule's answer
};

constexpr int kBinMinDeposit = 512;

// us of an item's binned chain, and of its atomics in the direct kernel.
inline double bins_us(const PlainItem &i, int ndim, int prec, int kind, int num_cu)
{
    const double unit = ndim == 2 ? 12.0 : (prec == PL_F64 ? 14.0 : 25.0) * (kind == PL_DUST ? 0.7 : 1.0);
    const double units = (double)(i.tiles < i.np ? i.tiles : i.np) / num_cu;
    return 26.0 + (i.tiles > 256 ? 8.0 : 0.0) + unit * (units > 1.0 ? units : 1.0) + 4e-4 * (double)i.np;
}
inline double atoms_us(const PlainItem &i, int ndim) { return (ndim == 2 ? 9.0 : 27.0) * i.channels * (double)i.np / 24000.0; }

// The items of one species kind.
inline void choose_bins(PlainItem *it, int n, int ndim, int prec, int kind, int num_cu)
{
    constexpr double kMargin = 1.05;
    int left = 0, small = 0;     // items that stay direct so far, those of them that could be binned
    double chains = 0.0, atoms = 0.0, first = 0.0;
    for (int k = 0; k < n; ++k) {
        PlainItem &i = it[k];
        i.binned = false;
        if (i.np <= 0) continue;
        const double b = bins_us(i, ndim, prec, kind, num_cu), a = atoms_us(i, ndim);
        const bool can = i.fits && i.np >= kBinMinDeposit;
        if (can && kMargin * b < a) {
            i.binned = true;
            continue;
        }
        ++left;
        if (can) ++small;
        chains += b;
        atoms += a;
        const double chain = 0.5 * (ndim == 2 ? 9.0 : 27.0) * i.channels;
        if (chain > first) first = chain;
    }
    if (small == 0 || small < left) return;
    const double hi = first > atoms ? first : atoms, lo = first > atoms ? atoms : first;
    if (kMargin * chains < hi + 0.5 * lo)
        for (int k = 0; k < n; ++k)
            if (it[k].np > 0) it[k].binned = true;
}

// A push alone (no deposit): binning saves scattered field reads.  Direct and
// binned in us: tracers 3D 131072 on 32^3 88 and 80, on 64^3 112 and 92, 2D float64
// 524295 on 512^2 146 and 149, 1048583 302 and 210, 600000 on 256^2 137 and 117; charged 64^3
// 131079 189 and 116, 512^2 524295 287 and 207; dust, which reads three components
// and pushes cheaply, 64^3 131079 60 and 94, 524295 232 and 212, 128 x 96 x 64 393223 212 and
// 195, 512^2 at any count slower binned (2097159 345 and 550).  On 16^3, whose fields
// stay in the caches, the direct kernel is the faster.
constexpr int kBinMinPush = 131072, kBinMinPushDust = 393216, kBinMinPush2D = 524288;
constexpr int kBinMinPushCells = 20000, kBinMinPushPerTile = 32;
inline bool push_bins(int64_t np, int64_t cells, int64_t tiles, int ndim, int prec, int kind)
{
    if (cells < kBinMinPushCells || np / kBinMinPushPerTile < tiles) return false;
    if (ndim == 3) return np >= (kind == PL_DUST ? kBinMinPushDust : kBinMinPush);
    if (kind == PL_DUST || np < kBinMinPush2D) return false;
    return !(kind == PL_TRACER && prec == PL_F64) || np >= 4 * cells;
}

}  // namespace pl
