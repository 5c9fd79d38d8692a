"""Which kernel a tiled call takes, compiled for the CPU from the header that the
launcher uses.  Each line is a call timed with both kernels on the GPU (us with
one particle per thread, us grouped): the rule takes the faster one."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include "tile_route.h"
extern "C" int pays(int mode, int ndim, int prec, int kind, int key, int64_t np, int64_t nt, int64_t cells)
{
    const pl::TileLoad w{np, nt, cells};
    return pl::local_pays(mode, ndim, prec, kind, key, 256, w);
}
"""
FUSED, PUSH, DEP = 0, 1, 2
F64, F32 = 0, 1
CHARGED, DUST, TRACER = 0, 1, 2
TILE, CELL, RANK, RUN = 0, 1, 2, 3


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    L.pays.argtypes = [C.c_int] * 5 + [C.c_int64] * 3
    return L


CASES = [
    # mode, prec, kind, key, box, tiles, particles per cell, step us, grouped us
    (FUSED, F32, CHARGED, TILE, (512, 512, 1), 4096, 8, 179, 242),
    (FUSED, F32, CHARGED, RANK, (440, 288, 1), 1980, 6, 62, 83),
    (FUSED, F32, DUST, TILE, (40, 48, 80), 300, 11, 171, 215),
    (FUSED, F32, DUST, TILE, (64, 64, 64), 512, 8, 228, 279),
    (FUSED, F32, DUST, TILE, (32, 32, 32), 64, 4, 75, 43),
    (FUSED, F64, DUST, RANK, (80, 84, 100), 10500, 10, 860, 885),
    (FUSED, F64, CHARGED, RANK, (64, 64, 64), 2048, 16, 740, 871),
    (FUSED, F64, CHARGED, TILE, (64, 64, 64), 2048, 8, 328, 250),
    (FUSED, F64, CHARGED, TILE, (64, 64, 64), 2048, 2, 176, 178),
    (FUSED, F32, CHARGED, TILE, (64, 64, 64), 512, 16, 595, 480),
    (FUSED, F32, CHARGED, RANK, (64, 64, 64), 512, 8, 395, 271),
    (FUSED, F32, CHARGED, CELL, (64, 64, 64), 512, 8, 1130, 295),
    (FUSED, F64, DUST, CELL, (512, 512, 1), 8192, 8, 260, 310),
    (DEP, F64, DUST, RANK, (64, 64, 64), 2048, 16, 285, 384),
    (DEP, F32, DUST, TILE, (64, 64, 64), 512, 2, 65, 69),
    (DEP, F32, CHARGED, RUN, (64, 64, 64), 512, 8, 538, 148),
    (DEP, F32, DUST, RUN, (512, 512, 1), 4096, 4, 106, 128),
    (DEP, F64, CHARGED, TILE, (32, 32, 1), 32, 16, 20, 23),
    (PUSH, F64, CHARGED, TILE, (1024, 1024, 1), 32768, 8, 446, 708),
    (PUSH, F64, DUST, TILE, (128, 128, 128), 16384, 8, 940, 1133),
    (PUSH, F32, CHARGED, TILE, (64, 64, 64), 512, 8, 187, 86),
    (PUSH, F64, TRACER, TILE, (64, 64, 64), 2048, 8, 177, 139),
    (PUSH, F32, DUST, TILE, (64, 64, 64), 512, 2, 44, 49),
    # tiles other than the default ones
    (FUSED, F64, CHARGED, TILE, (64, 64, 64), 1024, 8, 524, 403),      # 8 x 8 x 4
    (FUSED, F64, CHARGED, RANK, (64, 64, 64), 1024, 12, 596, 501),
    (FUSED, F64, CHARGED, RANK, (64, 64, 64), 512, 8, 450, 375),       # 8^3
    (FUSED, F64, CHARGED, TILE, (48, 48, 48), 216, 8, 286, 215),
    (FUSED, F64, CHARGED, TILE, (48, 48, 48), 216, 2, 103, 107),
    (FUSED, F64, CHARGED, RANK, (64, 64, 64), 4096, 16, 790, 868),     # 4^3
    (FUSED, F64, DUST, TILE, (32, 32, 32), 128, 8, 87, 78),
    (FUSED, F64, DUST, TILE, (64, 64, 64), 1024, 8, 278, 312),
    (FUSED, F32, CHARGED, TILE, (32, 32, 32), 128, 4, 84, 53),
    (DEP, F64, CHARGED, RANK, (64, 64, 64), 1024, 8, 256, 208),
    (DEP, F64, CHARGED, RANK, (64, 64, 64), 1024, 16, 476, 517),
    (DEP, F64, CHARGED, RANK, (64, 64, 32), 512, 4, 77, 88),
    (DEP, F64, CHARGED, TILE, (64, 64, 64), 512, 16, 565, 642),
    (DEP, F64, DUST, TILE, (64, 64, 64), 512, 8, 176, 148),
    (DEP, F64, DUST, TILE, (32, 32, 32), 128, 4, 32, 38),
    (DEP, F32, DUST, RANK, (64, 64, 64), 512, 4, 82, 90),              # 16 x 8 x 4
    (PUSH, F64, CHARGED, TILE, (64, 64, 64), 512, 8, 235, 391),
    (PUSH, F64, CHARGED, RANK, (48, 48, 48), 216, 8, 177, 192),
    (PUSH, F64, CHARGED, TILE, (64, 64, 64), 1024, 8, 263, 196),
    (PUSH, F64, DUST, TILE, (64, 64, 64), 512, 8, 125, 181),
    (PUSH, F64, DUST, TILE, (48, 48, 48), 216, 8, 97, 65),
    (PUSH, F64, TRACER, TILE, (64, 64, 64), 1024, 1, 40, 56),
    (PUSH, F64, TRACER, TILE, (64, 64, 64), 512, 2, 68, 58),
    (PUSH, F32, CHARGED, TILE, (512, 512, 1), 1024, 8, 58, 67),        # 16 x 16
    (PUSH, F32, DUST, TILE, (512, 512, 1), 2048, 8, 98, 69),           # 16 x 8
    (PUSH, F32, TRACER, TILE, (512, 512, 1), 1024, 4, 25, 52),
]

# The same for calls of few tiles, by particles per tile.
FEW = [
    # mode, ndim, prec, kind, key, cells per tile, tiles, particles per tile, step us, grouped us
    (FUSED, 3, F64, CHARGED, RANK, 128, 320, 900, 103, 87),
    (FUSED, 3, F64, CHARGED, TILE, 128, 320, 1100, 149, 105),
    (FUSED, 3, F64, CHARGED, TILE, 128, 480, 280, 65, 68),
    (FUSED, 3, F64, CHARGED, RANK, 128, 480, 700, 98, 92),
    (FUSED, 3, F64, CHARGED, RANK, 128, 800, 520, 123, 132),
    (DEP, 3, F64, CHARGED, TILE, 128, 320, 1100, 97, 57),
    (DEP, 3, F64, CHARGED, RANK, 128, 480, 700, 52, 64),
    (DEP, 3, F64, CHARGED, RANK, 128, 800, 700, 105, 93),
    (DEP, 3, F64, DUST, TILE, 128, 320, 520, 33, 28),
    (DEP, 3, F64, DUST, TILE, 128, 480, 520, 34, 45),
    (FUSED, 3, F32, CHARGED, TILE, 512, 200, 900, 81, 74),
    (FUSED, 3, F32, CHARGED, TILE, 512, 200, 1200, 99, 114),
    (DEP, 3, F32, CHARGED, TILE, 512, 200, 1200, 66, 80),
    (DEP, 3, F32, DUST, TILE, 512, 512, 1200, 75, 72),
    (DEP, 3, F32, CHARGED, TILE, 512, 96, 700, 41, 35),
    (PUSH, 2, F32, CHARGED, TILE, 64, 192, 600, 19, 13),
    (PUSH, 2, F32, CHARGED, TILE, 64, 500, 600, 21, 36),
    (PUSH, 2, F32, DUST, TILE, 64, 1024, 600, 20, 48),
    (PUSH, 2, F64, DUST, TILE, 32, 2048, 520, 78, 59),
    (PUSH, 3, F64, DUST, TILE, 128, 480, 280, 24, 20),
    (PUSH, 3, F64, DUST, TILE, 128, 480, 520, 30, 43),
    (PUSH, 3, F64, DUST, TILE, 128, 800, 520, 67, 58),
    (PUSH, 3, F64, CHARGED, TILE, 128, 480, 400, 45, 49),
    (PUSH, 3, F32, DUST, TILE, 512, 384, 900, 35, 22),
    (PUSH, 3, F32, DUST, TILE, 512, 512, 900, 39, 49),
]


@pytest.mark.parametrize("mode,prec,kind,key,box,tiles,ppc,step,grouped", CASES)
def test_the_faster_kernel(rule, mode, prec, kind, key, box, tiles, ppc, step, grouped):
    cells = box[0] * box[1] * box[2]
    got = rule.pays(mode, 2 if box[2] == 1 else 3, prec, kind, key, cells * ppc + 7, tiles, cells)
    assert bool(got) == (grouped < step)


@pytest.mark.parametrize("mode,ndim,prec,kind,key,ct,tiles,pt,step,grouped", FEW)
def test_few_tiles(rule, mode, ndim, prec, kind, key, ct, tiles, pt, step, grouped):
    got = rule.pays(mode, ndim, prec, kind, key, pt * tiles + 7, tiles, ct * tiles)
    assert bool(got) == (grouped < step)
