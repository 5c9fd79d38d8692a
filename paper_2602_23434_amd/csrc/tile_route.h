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
// CUs.  Where a launch has more units than the chip holds blocks, its blocks
// claim them from one counter, about 20 ns a claim: 2D float32 pushes of 600
// particles a tile take 11 us on 192 tiles, 36 on 500 and 48 on 1024, which one
// particle per thread, with more and smaller blocks resident, does in 19, 20 and 29.
// So the lines lie at the tiles that are resident, too.  Times below are us per call on MI355X, one particle per thread and
// grouped, 64^3 cells (512^2 in 2D), TSC and the default tiles (8^3 in float32,
// 8 x 4 x 4 in float64, 8 x 8 and 8 x 4 in 2D) unless said, p particles per cell.
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
    const int64_t ct = w.nt > 0 ? w.cells / w.nt : 0;              // cells per tile
    const bool f64 = prec == PL_F64, charged = kind == PL_LORENTZ, d2 = ndim == 2;
    const bool by_cell = key == PL_KEY_TILE_CELL || key == PL_KEY_TILE_RUN;
    auto per_cell = [&](double p) { return (double)w.np >= p * (double)w.cells; };
    if (mode == LM_PUSH) {
        // The gather from 16-byte records against one LDS read per component;
        // larger blocks, which cost where there are many small tiles.
        //  a tile per CU or fewer: charged 32^3 float32 p 8 113 and 36, 32 x 32 float64
        //    p 256 96 and 30
        //  2D: float32 charged p 8 102 and 89, dust 105 and 85, on 1024^2 (16384
        //    tiles) 306 and 325, 267 and 307; float64 charged 145 and 167; 16 x 8 tiles
        //    97 and 72, 98 and 69, float64 dust 100 and 78; 16 x 16 float32 charged 58 and
        //    67, float64 74 and 128, tracers p 4 25 and 52
        //  3D float32: charged p 8 187 and 86; dust p 2 44 and 49 (two blocks a CU,
        //    two particles a thread), p 4 62 and 55, 128^3 p 2 185 and 164
        //  3D float64: charged p 8 250 and 196, 128^3 p 2 642 and 655, p 4 1063
        //    and 984, 8 x 8 x 4 tiles p 8 263 and 196, but 8^3, whose 48-byte records
        //    leave two blocks a CU a field halo of one cell only, 235 and 391, 16 x 8 x 4
        //    243 and 338; dust 136 and 129, 128^3 940 and 1133, 8^3 tiles 125 and 181, on 48^3
        //    (216 tiles) 97 and 65, 48^3 in 8 x 8 x 4 80 and 67; tracers 177 and 139, 8 x 8 x 4
        //    p 1 40 and 56, p 2 61 and 67, p 4 100 and 92, 8^3 p 1 44 and 50, p 2 68 and 58
        //  resident or not (two blocks of 512 per CU): float64 charged 480 tiles of 280
        //    particles 38 and 26, of 400 44 and 49; dust 23 and 19, of 520 29 and 42, 800 tiles
        //    66 and 56; float32 dust 384 tiles of 900 32 and 22, 512 38 and 48, of 2000 66 and
        //    58; 2D dust 1024 tiles of 600 20 and 48, float64 2048 tiles 78 and 59
        const bool resident = w.nt <= num_cu || w.nt + w.np / 4096 <= 2 * num_cu;
        if (f64 && charged && ct >= 512) return false;
        if (resident) return true;
        if (d2) return w.nt >= 7 * num_cu && w.nt <= 16 * num_cu && ct < (f64 && charged ? 64 : 256);
        if (!f64) return charged || pt >= 1800 || w.nt > 1024;
        if (kind == PL_DUST) return ct < 256 && 2 * w.nt >= 5 * num_cu && w.nt <= 1600;
        if (kind == PL_TRACER && ct >= 256) return pt >= 768;
        if (2 * w.nt < 5 * num_cu && pt < 512) return false;
        return w.nt <= 4096 || per_cell(3.5);
    }
    const bool fused = mode == LM_FUSED, few = w.nt <= num_cu / 4, half = w.nt <= num_cu / 2;
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
        // 8 x 8 x 4 tiles: charged fused p 4 250 and 224, by rank 212 and 223; 32^3 (128
        // tiles) p 4 84 and 53, by rank 78 and 52, dust 48 and 39, deposits 50 and 32, 33
        // and 24, by rank p 8 62 and 58, 41 and 42; 16 x 8 x 4 dust deposit by rank p 4 82 and
        // 90, p 8 123 and 114.
        // Chunks are of 1024 particles or more, so between a quarter of the CUs' number of
        // tiles and it a tile of a few more becomes two: 200 tiles of 900 charged fused 81 and
        // 74, of 1200 99 and 114, of 2000 143 and 129, deposit 55 and 50, 66 and 80, 90 and 85.
        // More: 512 tiles of 900 charged fused 146 and 140, by rank 136 and 139, deposit 106
        // and 98, by rank of 1200 105 and 102, dust of 1200 75 and 72; 96 tiles of 700 charged
        // 63 and 57, deposit 41 and 35.
        const bool between = !few && w.nt <= num_cu;
        const bool rank = key == PL_KEY_TILE_RANK;
        if (half && pt >= (charged ? 700 : 1024)) return true;
        if (charged && fused) return between ? pt >= 1600 || (pt >= 800 && pt <= 1000) : pt >= 1280 || few;
        if (charged) return between ? pt >= 2560 || (!rank && pt >= 850 && pt <= 1000) : pt >= (rank ? 1150 : 850);
        if (fused) return between && pt >= 4096;
        return pt >= (between || rank ? 2560 : 1150);
    }
    // Float64.  Blocks of 256 threads up to 2048 particles a tile, one of 512 per CU
    // beyond, which pays on tiles of 256 cells or more.  8 x 4 x 4 tiles:
    // charged fused p 2 176 and 178, p 4 191 and 181, p 8 328 and 250, p 16 812
    // and 804; by rank p 4 162 and 176, p 8 270 and 243, p 16 740 and 871; 32^3 (256
    // tiles) p 8 98 and 92, p 16 167 and 172; 24 x 40 x 20 (150 tiles) p 2 45 and 42.
    // Deposit p 4 158 and 128, p 8 244 and 156, p 16 557 and 530; by rank p 8 241 and
    // 218, p 12 333 and 333.  Dust fused p 8 276 and 286; deposit p 8 184 and 147, by rank
    // 158 and 153.
    // 8 x 8 x 4: charged fused p 4 290 and 250, p 8 524 and 403, p 16 973 and 973, by
    // rank p 4 241 and 246, p 8 406 and 366, p 12 596 and 501; deposit p 8 313 and 227, p
    // 16 580 and 592, by rank p 8 256 and 208, p 16 476 and 517, 64 x 64 x 32 (512 tiles) p 4
    // 77 and 88; dust fused p 8 278 and 312, deposit p 4 110 and 120, p 8 184 and 156, by
    // rank 140 and 146, 32^3 (128 tiles) fused p 8 87 and 78, deposit p 4 32 and 38, p 8 53
    // and 47, by rank 40 and 46, p 16 70 and 61; 48^3 (432 tiles) charged fused p 4 152 and
    // 127, deposit 88 and 79.
    // 8^3: charged fused p 8 521 and 417, by rank 450 and 375, 48^3 (216 tiles) p 2 103
    // and 107, p 8 286 and 215; deposit p 8 301 and 239, p 16 565 and 642, by rank 226 and
    // 193, 64 x 64 x 32 (256 tiles) by rank 126 and 136; dust deposit p 8 176 and 148.
    // 4^3: charged fused p 8 502 and 523, p 16 950 and 896, by rank 790 and 868; deposit p
    // 8 364 and 289, by rank 253 and 288; dust 219 and 231.
    // Few of the smaller tiles, 8 x 4 x 4: 320 of 280 charged fused 57 and 52, by rank 50 and
    // 51, of 1100 149 and 105, 117 and 103, deposit 33 and 31, 97 and 57, by rank of 700 48 and
    // 41, dust deposit of 520 33 and 28, by rank 27 and 28; 480 of 280 charged fused 65 and 68,
    // of 700 109 and 93, by rank 98 and 92, deposit of 400 45 and 53, of 700 66 and 62, by rank
    // 52 and 64; 800 of 280 109 and 102, of 700 185 and 148, by rank 152 and 145, deposit of 280
    // 73 and 70, by rank of 700 105 and 93.
    const bool flat = ct < 256;
    const bool fill = 4 * w.nt < (flat ? 6 : 3) * num_cu, many = 2 * w.nt >= 3 * num_cu, lots = 2 * w.nt >= 5 * num_cu;
    const bool big = pt >= 2048;
    const bool rank = key == PL_KEY_TILE_RANK;
    const bool thin = !per_cell(14.0);
    if (!charged) {
        if (half && pt >= (fused || !rank ? 2048 : 4096)) return true;
        if (fused || rank) return false;
        if (flat && fill && 4 * w.nt >= 3 * num_cu) return pt >= 500;
        return (many || (fill && big)) && ct >= 128 && per_cell(7.0) && thin && pt >= 1024;
    }
    if (fused) {
        if (big) return !flat || (fill && !rank);
        if (fill) return flat || !rank || pt >= 1024;
        if (rank) return many && ct >= 128 && pt >= (flat ? 650 : 1024);
        return many && pt >= (ct < 128 ? 1024 : lots ? 272 : 512);
    }
    if (rank) {
        if (half && pt >= 4096) return true;
        if (big) return !flat && thin && w.nt >= 2 * num_cu;
        if (flat && fill) return 4 * w.nt >= 3 * num_cu && pt >= 600;
        return ct >= 128 && thin && (flat ? lots && pt >= 650 : pt >= 1024 && w.nt >= 4 * num_cu);
    }
    return fill || (big ? !flat && thin : many && pt >= (ct < 128 ? 512 : lots ? 272 : 650));
}

}  // namespace pl
