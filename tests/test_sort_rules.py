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
// ranges: (item, begin, end, write) of items in turn, n of them; the items that join the first one's group
extern "C" int joined(const int64_t *r, int n)
{
    static pl::GroupMemory m;
    m.n = 0;
    int items = 0;
    for (int k = 0; k < n;) {
        pl::GroupMemory::Range mine[pl::GroupMemory::kPerItem];
        int c = 0;
        const int64_t it = r[4 * k];
        for (; k < n && r[4 * k] == it; ++k)
            mine[c++] = pl::GroupMemory::Range{(uintptr_t)r[4 * k + 1], (uintptr_t)r[4 * k + 2], 0, r[4 * k + 3] != 0};
        if (!m.add((int)it, mine, c)) break;
        ++items;
    }
    return items;
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
    L.joined.argtypes = [C.POINTER(C.c_int64), C.c_int]
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


@pytest.mark.parametrize("cells,np,small_cells,small_np,want", [
    (256 ** 3, 1 << 24, 32 ** 3, 1000, False),      # 2^24 keys, three passes: a fourth over 16 million particles
    (255 ** 3, 1 << 24, 32 ** 3, 1000, True),       # three passes with both
    (256 ** 3, 500_000, 32 ** 3, 1000, True),       # a fourth pass over half a million
    (16 ** 3, 60_000, 4096 * 15, 4000, True),
    (96 ** 3, 5_000_000, 96 ** 3, 1_000_000, True),
])
def test_no_further_pass_over_many_particles(rules, cells, np, small_cells, small_np, want):
    assert bool(rules.takes(np, cells, cells, small_np, small_cells, 1 << 30)) == want


def _joined(rules, ranges):
    flat = [int(v) for r in ranges for v in r]
    return rules.joined((C.c_int64 * len(flat))(*flat), len(ranges))


@pytest.mark.parametrize("name,ranges,want", [
    # (item, begin, end, write): each item reads its set and writes its other one
    ("own sets", [(0, 0, 10, 0), (0, 20, 30, 1), (1, 10, 20, 0), (1, 30, 40, 1)], 2),
    ("a read-only array of both", [(0, 0, 10, 0), (0, 20, 30, 1), (1, 0, 10, 0), (1, 30, 40, 1)], 2),
    ("the second writes what the first has read", [(0, 0, 10, 0), (0, 20, 30, 1), (1, 10, 20, 0), (1, 0, 10, 1)], 1),
    ("the second reads what the first writes", [(0, 0, 10, 0), (0, 20, 30, 1), (1, 29, 39, 0), (1, 40, 50, 1)], 1),
    ("one table for both", [(0, 0, 10, 0), (0, 20, 30, 1), (1, 10, 20, 0), (1, 30, 40, 1), (1, 25, 26, 1)], 1),
    ("an array inside another's", [(0, 0, 100, 1), (1, 200, 210, 0), (1, 50, 60, 0)], 1),
    ("a long range before a short one", [(0, 0, 100, 0), (1, 10, 20, 0), (2, 90, 95, 1)], 2),
    ("its own arrays in any order", [(0, 0, 10, 1), (0, 5, 8, 0), (1, 10, 12, 1)], 2),
    ("empty ranges", [(0, 5, 5, 1), (0, 6, 8, 1), (1, 5, 6, 1), (1, 7, 7, 1)], 2),
])
def test_items_that_share_memory_are_sorted_one_after_another(rules, name, ranges, want):
    assert _joined(rules, ranges) == want
