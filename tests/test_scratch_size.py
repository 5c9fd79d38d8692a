"""Size of the sort's scratch, compiled for the CPU from the header that
pl_part_init uses: four words per particle, and little more for the spectral
update's records."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include "scratch.h"
extern "C" int64_t slab(int64_t np, int64_t cells) { return pl::slab_bytes(np, cells); }
extern "C" int64_t keys(int64_t np) { return pl::keys_bytes(np); }
"""


@pytest.fixture(scope="module")
def size(tmp_path_factory):
    d = tmp_path_factory.mktemp("scratch")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    for f in (L.slab, L.keys):
        f.restype = C.c_int64
    L.slab.argtypes = [C.c_int64, C.c_int64]
    L.keys.argtypes = [C.c_int64]
    return L


@pytest.mark.parametrize("np,cells", [(1024 ** 3, 1024 ** 3), (512 ** 3, 512 ** 3), (3 * 256 ** 3, 256 ** 3), (1, 1),
                                      (64, 64), (1000, 4096), (2 ** 24, 128 ** 3), (4096, 1024), (2 ** 31 - 1, 1024 ** 3)])
def test_bound(size, np, cells):
    assert size.keys(np) >= 16 * np
    assert size.keys(np) <= size.slab(np, cells) <= size.keys(np) + (64 << 20)


def test_records_fit_where_it_says(size):
    assert size.slab(64 ** 3, 64 ** 3) == 64 * 64 ** 3               # one particle per cell: 16.8 MB instead of 4.2
    assert size.slab(4 * 64 ** 3, 64 ** 3) == size.keys(4 * 64 ** 3)
    assert size.slab(512 ** 3, 512 ** 3) == size.keys(512 ** 3)      # 8.6 GB of records: not for them
    assert size.slab(1000, 64 ** 3) == size.keys(1000)
