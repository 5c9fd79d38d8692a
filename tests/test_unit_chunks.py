"""The deal of a run-kernel launch's parts to its chunks, compiled for the CPU
from the header that the kernel uses: every part in one chunk, and the crowded
pieces, which a list has first, spread over all of them."""

import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include "unit_chunks.h"
extern "C" int queues() { return pl::kQueues; }
extern "C" int deal() { return pl::kDeal; }
extern "C" int size(int q, int parts) { return pl::chunk_size(q, parts); }
extern "C" int part(int q, int k) { return pl::chunk_part(q, k); }
"""


@pytest.fixture(scope="module")
def chunks(tmp_path_factory):
    d = tmp_path_factory.mktemp("chunks")
    src, so = d / "probe.cpp", d / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(so)], check=True)
    return C.CDLL(str(so))


@pytest.mark.parametrize("parts", [0, 1, 15, 16, 17, 127, 128, 129, 257, 512, 1000, 4096, 5121])
def test_every_part_in_one_chunk(chunks, parts):
    nq = chunks.queues()
    got = [chunks.part(q, k) for q in range(nq) for k in range(chunks.size(q, parts))]
    assert sorted(got) == list(range(parts))


@pytest.mark.parametrize("heavy,parts", [(64, 1088), (128, 1088), (500, 4600), (1024, 5000)])
def test_first_parts_are_spread(chunks, heavy, parts):
    """Each chunk has its share of the first parts, to within one deal, and has them first."""
    nq, deal = chunks.queues(), chunks.deal()
    for q in range(nq):
        mine = [chunks.part(q, k) < heavy for k in range(chunks.size(q, parts))]
        n = sum(mine)
        assert abs(n - heavy / nq) <= deal
        assert all(mine[:n])
