"""The footprint by which the float32 run kernel takes a tile, compiled for the
CPU from the header that the launcher uses: the tiles whose grids it sums in
float32 are the ones it has always taken."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")
LDS = 160 * 1024

PROBE = r"""
#include "runs_sums.h"
extern "C" long bytes(int charged, int tx, int ty, int tz, int ndim, int nslot, int hf)
{
    const int T[3] = {tx, ty, tz};
    return (long)pl::runs_sums_bytes(charged != 0, T, ndim, nslot, hf);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("sums")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    L.bytes.restype = C.c_long
    return L


@pytest.mark.parametrize("tile,nslot,takes", [
    ((8, 8, 8), 7, True), ((8, 8, 8), 8, True), ((8, 8, 4), 8, True), ((16, 8, 4), 7, True),
    ((16, 8, 4), 8, False), ((8, 16, 4), 8, False), ((8, 8, 9), 8, False), ((12, 8, 6), 8, False),
    ((9, 9, 8), 7, False), ((12, 12, 4), 7, False), ((16, 8, 5), 7, False),
])
def test_tiles_taken(rule, tile, nslot, takes):
    """Charged particles, one-cell field halo, 160 KB of LDS."""
    assert (rule.bytes(1, *tile, 3, nslot, 1) <= LDS) == takes


def test_halo_and_kind(rule):
    # 8^3 tiles: with every channel only the particles inside the tile join (two-cell halo), with seven all do
    assert rule.bytes(1, 8, 8, 8, 3, 8, 2) > LDS >= rule.bytes(1, 8, 8, 8, 3, 7, 2)
    # by hand: 12^3 records of 32 bytes and 12^3 x 7 sums, 64 + 256 queue words, 256 x 10 floats, 80 bytes
    assert rule.bytes(1, 8, 8, 8, 3, 7, 2) == 1728 * 32 + 1728 * 56 + 256 + 1024 + 10240 + 80
    assert rule.bytes(0, 8, 8, 1, 2, 4, 1) == 100 * 16 + 144 * 32 + 1024 + 1024 + 7168 + 80
