"""The cache of resident block counts under threads, compiled for the CPU from the
header that the launchers use: contexts of one process may be on any thread."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23434_amd", "csrc")

PROBE = r"""
#include <stdio.h>
#include <atomic>
#include <thread>
#include <vector>
#include "launch_cache.h"
int main()
{
    static pl::LaunchCache<long> cache;
    std::atomic<long> made{0}, wrong{0};
    std::vector<std::thread> t;
    for (int w = 0; w < 8; ++w)
        t.emplace_back([&, w] {
            for (long k = 0; k < 40000; ++k) {
                const long key = w % 2 ? k : 39999 - k;
                const int v = cache.get(key, [&]() { ++made; return (int)(3 * key); });
                if (v != 3 * key) ++wrong;
            }
        });
    for (auto &x : t) x.join();
    printf("%ld %ld\n", made.load(), wrong.load());
    return 0;
}
"""


def test_every_value_made_once(tmp_path):
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout.split()
    assert out == ["40000", "0"]
