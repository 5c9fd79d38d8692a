"""The rules by which the items of a sort call share one radix sort, compiled
for the CPU from the header that the launcher uses."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include "sort_groups.h"
extern "C" int takes(int64_t gnp, uint64_t gkeys, uint64_t gmost, int64_t np, uint64_t keys, int64_t cap)
{
    pl::GroupSize g;
    g.np = gnp;
    g.keys = gkeys;
    g.most = gmost;
    return pl::group_takes(g, np, keys, cap);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    L.takes.argtypes = [C.c_int64, C.c_uint64, C.c_uint64, C.c_int64, C.c_uint64, C.c_int64]
    return L


@pytest.mark.parametrize("cells,items", [(1024 ** 3, 4), (1024 * 1024 * 512, 8)])
def test_no_key_is_the_run_tables_sentinel(rules, cells, items):
    """The largest key of a group is its number of keys less one; the run table's
    builder takes 2^32 - 1 for "no neighbour", so it must stay below that: items
    whose cells add up to 2^32 are not sorted together, and one fewer are."""
    keys = cells
    taken = 1
    while taken < items and rules.takes(100 * taken, keys, cells, 100, cells, 1 << 20):
        keys += cells
        taken += 1
    assert keys - 1 < 2 ** 32 - 1
    assert taken == items - 1


def test_keys_up_to_the_sentinel_join(rules):
    assert rules.takes(10, 2 ** 31, 2 ** 31, 10, 2 ** 31 - 1, 100)
    assert not rules.takes(10, 2 ** 31, 2 ** 31, 10, 2 ** 31, 100)
    assert not rules.takes(10, 2 ** 31, 2 ** 31, 91, 1, 100)      # the scratch's particles
