"""LDS of the run kernel's float64 form, compiled for the CPU from the header that
the kernel uses: every tile that fits with queues of 128 deposits and 16 bytes of
control words fits with the present ones too."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include "runs_lds.h"
extern "C" long bytes(int real, int rec, int Lf, int Ld, int nslot, int hf, int threads)
{
    size_t offs[6];
    return (long)pl::runs_lds_layout(real, rec, Lf, Ld, nslot, hf, threads, offs);
}
// tiles of up to 1024 cells that fit the plain layout and not this one
extern "C" int refused(int rec, int nslot, int hf, long lds)
{
    auto sec = [](long b) { return (b + 15) / 16 * 16; };
    int n = 0;
    for (int x = 1; x <= 64; ++x)
        for (int y = 1; y <= 64; ++y)
            for (int z = 1; z <= 64 && x * y * z <= 1024; ++z)
                for (int ndim = z == 1 ? 2 : 3; ndim <= 3; ++ndim) {
                    const int Lf = (x + 2 * hf) * (y + 2 * hf) * (ndim == 3 ? z + 2 * hf : 1);
                    const int Ld = (x + 4) * (y + 4) * (ndim == 3 ? z + 4 : 1);
                    const long plain = sec(8L * rec * Lf) + sec(8L * Ld * nslot) + (hf == 2 ? 256 : 1024) + 512 +
                                       sec(128L * (3 + nslot) * 8) + 64 + 16;
                    n += plain <= lds && bytes(8, rec, Lf, Ld, nslot, hf, 512) > lds;
                }
    return n;
}
"""


@pytest.fixture(scope="module")
def lds(tmp_path_factory):
    d = tmp_path_factory.mktemp("lds")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    L.bytes.restype = C.c_long
    L.refused.argtypes = [C.c_int, C.c_int, C.c_int, C.c_long]
    return L


@pytest.mark.parametrize("hf", [1, 2])
@pytest.mark.parametrize("rec,nslot", [(6, 0), (6, 1), (6, 3), (6, 4), (6, 7), (6, 8), (4, 0), (4, 1), (4, 3), (4, 4)])
def test_no_tile_is_refused_for_the_control_words(lds, rec, nslot, hf):
    assert lds.refused(rec, nslot, hf, 160 * 1024) == 0


def test_footprints(lds):
    # 8^3, float32, seven channels, two-cell halo: 24-byte records, 192 queued deposits
    assert lds.bytes(4, 6, 1728, 1728, 7, 2, 512) == 1728 * 24 + 1728 * 56 + 256 + 768 + 7680 + 64 + 320
    # 4 x 9 x 12 in float64 with eight channels fits the 160 KB
    assert lds.bytes(8, 6, 6 * 11 * 14, 8 * 13 * 16, 8, 1, 512) <= 160 * 1024
