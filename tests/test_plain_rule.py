"""When a plain call bins an item's particles, compiled for the CPU from the
header that the launcher uses.  Calls timed both ways on the GPU (us with every
item binned, us with none): the rule takes the faster way for the call as a
whole, and large items are binned beside small ones that are not."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include "plain_cost.h"
extern "C" void choose(int n, const int64_t *np, const int64_t *tiles, const int *fits, int channels, int ndim, int prec,
                       int kind, int *binned)
{
    static pl::PlainItem it[4096];
    for (int i = 0; i < n; ++i) it[i] = pl::PlainItem{np[i], tiles[i], channels, fits[i] != 0, false};
    pl::choose_bins(it, n, ndim, prec, kind, 256);
    for (int i = 0; i < n; ++i) binned[i] = it[i].binned;
}
extern "C" int push(int64_t np, int64_t cells, int64_t tiles, int ndim, int prec, int kind)
{
    return pl::push_bins(np, cells, tiles, ndim, prec, kind);
}
"""
F64, F32 = 0, 1
CHARGED, DUST, TRACER = 0, 1, 2


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("plain")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    L = C.CDLL(str(so))
    L.push.argtypes = [C.c_int64] * 3 + [C.c_int] * 3

    def choose(items, channels, ndim, prec, kind):
        """items: (particles, tiles, fits)"""
        n = len(items)
        out = (C.c_int * n)()
        L.choose(n, (C.c_int64 * n)(*[i[0] for i in items]), (C.c_int64 * n)(*[i[1] for i in items]),
                 (C.c_int * n)(*[i[2] for i in items]), channels, ndim, prec, kind, out)
        return [bool(v) for v in out]

    return choose, L.push


@pytest.mark.parametrize("count,np,box,ndim,tiles,prec,kind,binned,direct", [
    (1, 600, 16, 3, 16, F64, CHARGED, 42, 99), (2, 600, 16, 3, 16, F64, CHARGED, 69, 102),
    (4, 600, 16, 3, 16, F64, CHARGED, 130, 103), (64, 600, 16, 3, 16, F64, CHARGED, 1890, 334),
    (1000, 600, 16, 3, 16, F64, CHARGED, 31600, 4900),
    (8, 2048, 16, 3, 8, F32, CHARGED, 328, 164), (1, 2048, 64, 3, 1024, F64, CHARGED, 112, 126),
    (2, 2048, 64, 3, 1024, F64, CHARGED, 215, 150), (2, 2048, 64, 2, 8, F64, CHARGED, 81, 46),
    (1, 2048, 32, 3, 128, F64, DUST, 52, 68), (4, 2048, 32, 3, 128, F64, DUST, 176, 72),
    (64, 20000, 16, 3, 16, F64, CHARGED, 3312, 10132), (64, 20000, 128, 2, 16, F32, CHARGED, 2970, 3461),
    (16, 200000, 32, 3, 128, F64, CHARGED, 1480, 25822), (1, 8199, 32, 2, 2, F64, DUST, 46, 23),
    (1, 8199, 32, 2, 2, F64, CHARGED, 47, 37), (1, 2055, 32, 2, 1, F32, CHARGED, 44, 29),
])
def test_the_faster_way(rule, count, np, box, ndim, tiles, prec, kind, binned, direct):
    choose, _ = rule
    got = choose([(np, tiles, 1)] * count, 7 if kind == CHARGED else 4, ndim, prec, kind)
    assert got == [binned < direct] * count


def test_a_large_item_beside_small_ones(rule):
    choose, _ = rule
    got = choose([(200000, 128, 1)] + [(600, 16, 1)] * 40 + [(0, 16, 1), (3, 16, 1)], 7, 3, F64, CHARGED)
    assert got == [True] + [False] * 42


def test_one_that_must_stay_direct_keeps_the_small_ones(rule):
    choose, _ = rule
    # alone the small item is binned; beside one of too few particles, whose chain is paid anyway, it is not
    assert choose([(600, 16, 1)], 7, 3, F64, CHARGED) == [True]
    assert choose([(600, 16, 1), (511, 16, 1)], 7, 3, F64, CHARGED) == [False, False]
    assert choose([(600, 16, 0)], 7, 3, F64, CHARGED) == [False]


@pytest.mark.parametrize("np,n,ndim,tiles,prec,kind,binned,direct", [
    (131079, 64, 3, 1024, F64, TRACER, 92, 112), (131079, 64, 3, 1024, F64, DUST, 103, 61),
    (524295, 64, 3, 512, F32, DUST, 212, 232), (2097159, 512, 2, 256, F32, DUST, 554, 338),
    (524295, 512, 2, 512, F64, TRACER, 149, 146), (1048583, 512, 2, 512, F64, TRACER, 210, 302),
    (524295, 512, 2, 256, F32, TRACER, 106, 141), (524295, 512, 2, 512, F64, CHARGED, 207, 287),
    (32775, 16, 3, 16, F64, CHARGED, 28, 28 - 1),
])
def test_push(rule, np, n, ndim, tiles, prec, kind, binned, direct):
    _, push = rule
    assert bool(push(np, n ** ndim, tiles, ndim, prec, kind)) == (binned < direct)
