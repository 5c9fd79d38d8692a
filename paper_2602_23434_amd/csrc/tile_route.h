// Where the self-grouping tile kernels (k_local_impl.h) pay: the rules by which
// a call takes them or the one-particle-per-thread kernel (k_step_impl.h).
// Host arithmetic only, so that a plain C++ compiler takes it.
//
// Grouping a chunk by cell costs three passes over its particles' positions
// and as many barriers, and saves LDS atomics: a quarter (float32) to a half
// (float64) of them remain, and lanes of one cell no longer meet on one address.
// So it pays by what the deposit costs without it: 27 points and 7 or 8 channels
// in 3D, not 9 points in 2D or the 4 channels of dust; particles stored cell by
// cell (lanes of one cell), not rank by rank (lanes of distinct cells); and where
// few tiles hold many particles, since a tile of several chunks takes several
// CUs.  Times below are us per call on MI355X, one particle per thread and
// grouped, 64^3 cells (512^2 in 2D) and TSC unless said, p particles per cell.
#pragma once

#include <stdint.h>

#include "../../include/pl.h"

namespace pl {

enum LocalMode { LM_FUSED = 0, LM_PUSH = 1, LM_DEP = 2 };

// A launch's items: particles, tiles and cells in all.
struct TileLoad {
    int64_t np, nt, cells;
};

inline bool local_pays(int mode, int ndim, int prec, int kind, int key, int num_cu, const TileLoad &w)
{
    const int64_t pt = w.nt > 0 ? w.np / w.nt : 0;                 // particles per tile
    const bool f64 = prec == PL_F64, charged = kind == PL_LORENTZ, d2 = ndim == 2;
    const bool by_cell = key == PL_KEY_TILE_CELL || key == PL_KEY_TILE_RUN;
    auto per_cell = [&](double p) { return (double)w.np >= p * (double)w.cells; };
    if (mode == LM_PUSH) {
        // The gather from 16-byte records against one LDS read per component;
        // larger blocks, which cost where there are many small tiles.
        //  a tile per CU or fewer: charged 32^3 float32 p 8 113 and 36, 32 x 32 float64
        //    p 256 96 and 30
        //  2D: float32 charged p 8 102 and 89, dust 105 and 85, on 1024^2 (16384
        //    tiles) 306 and 325, 267 and 307; float64 charged 145 and 167
        //  3D float32: charged p 8 187 and 86; dust p 2 44 and 49 (two blocks a CU,
        //    two particles a thread), p 4 62 and 55, 128^3 p 2 185 and 164
        //  3D float64: charged p 8 250 and 196, 128^3 p 2 642 and 655, p 4 1063
        //    and 984; dust 136 and 129, 128^3 940 and 1133; tracers 177 and 139
        if (w.nt <= num_cu) return true;
        if (d2) return (!f64 || !charged) && w.cells >= 64 * w.nt && w.nt <= 4096;
        if (!f64) return charged || pt >= 2048 || w.nt > 1024;
        if (kind == PL_DUST) return w.nt <= 1024;
        return w.nt <= 4096 || per_cell(3.5);
    }
    const bool fused = mode == LM_FUSED, few = w.nt <= num_cu / 4;
    // Few tiles of many particles each: 32 x 32 float32 charged p 32 57 and 35,
    // 16^3 float64 dust p 16 by rank 71 and 50, float32 deposit p 2 by rank 39 and 28.
    if (few && pt >= (f64 || d2 ? 2048 : 1024)) return true;
    if (by_cell) {
        // Stored cell by cell or run by run.  3D: float32 charged deposit p 4 by
        // cell 383 and 115, by run 296 and 115, dust deposit p 2 89 and 80; fused
        // charged p 2 184 and 143, dust p 2 104 and 151, p 4 239 and 128.
        if (!d2) return !fused || charged || per_cell(3.5);
        // 2D: deposit charged by cell p 4 164 and 139, by run 136 and 139, p 8 216 and
        // 152; dust by cell p 8 245 and 140, by run float32 p 16 239 and 191, float64
        // 232 and 223 (1024^2 808 and 860); fused charged p 8 413 and 246 (128 x 128
        // float64 42 and 46), dust float64 p 8 260 and 310, p 16 629 and 443.
        if (!fused) {
            if (charged) return per_cell(key == PL_KEY_TILE_CELL ? 3.5 : 7.0);
            if (key != PL_KEY_TILE_CELL) return !f64 && per_cell(14.0);
            return per_cell(f64 && w.nt < 1024 ? 14.0 : 7.0);
        }
        const double p = charged || !f64 ? 7.0 : 14.0;
        return per_cell(w.nt < 1024 ? 2.0 * p : p);
    }
    // Stored in any order within the tile, or rank by rank.  2D: fused float32
    // charged p 8 179 and 242, by rank 151 and 237, dust 137 and 207, float64 charged 216
    // and 363; deposit 151 and 151, 118 and 152, 115 and 139, 175 and 234.
    if (d2) return false;
    if (!f64) {
        // charged fused p 2 153 and 143 (128^3 939 and 1010, 48^3 98 and 108), p 4 246
        // and 195, by rank 222 and 193; deposit p 2 109 and 101 (24 x 40 x 20, 640 a
        // tile, 35 and 39), by rank 91 and 95, p 4 161 and 113; dust fused p 8 228 and 279,
        // 32^3 p 4 75 and 43; 48^3 (216 tiles) p 16 128 and 111; dust deposit p 2 65 and 69,
        // p 4 105 and 82.  Tiles between a quarter of the CUs' number and it leave some
        // CUs two chunks of a tile and others one: 48^3 by rank p 4 76 and 86.
        const bool between = !few && w.nt <= num_cu;
        if (charged && fused) return pt >= 1280 || few;
        if (charged) return pt >= (between ? 2560 : key == PL_KEY_TILE_RANK ? 1280 : 1024);
        if (fused) return between && pt >= 4096;
        return pt >= (between ? 2560 : 2048);
    }
    // Float64: tiles of 8 x 4 x 4 and blocks of 256 threads up to 2048 particles a
    // tile.  Charged fused p 2 176 and 178, p 4 191 and 181, p 8 328 and 250, p 16 812
    // and 804; by rank p 4 162 and 176, p 8 270 and 243, p 16 740 and 871; 32^3 (256
    // tiles) p 8 98 and 92, p 16 167 and 172; 24 x 40 x 20 (150 tiles) p 2 45 and 42.
    // Deposit p 4 158 and 128, p 8 244 and 156, p 16 557 and 530; by rank p 8 241 and
    // 218.  Dust fused p 8 276 and 286; deposit p 8 184 and 147, by rank 158 and 153.
    const bool small = pt < 2048 && w.nt >= 512;
    const bool fill = w.nt < num_cu * 3 / 4;
    const bool rank = key == PL_KEY_TILE_RANK;
    if (!charged) return !fused && !rank && pt >= 1024 && (small || fill);
    if (rank) return pt >= 1024 && (small || (fused && fill));
    return fill || (small && pt >= 512);
}

}  // namespace pl
