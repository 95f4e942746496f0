"""The sizes of the workspace's arrays (csrc/capacity.h, compiled for the host) over
every body count and bucket size a context accepts: what the blocks of a build reserve
of the subtree lists fits the buffer and 64-bit counters, down to the last block."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <random>
#include <type_traits>
#include "capacity.h"

int main()
{
    using namespace bhx;
    static_assert(std::is_same<decltype(subtree_splits(1, 1, 1)), int64_t>::value, "64 bits");
    std::mt19937_64 rng(1);
    for (int64_t n : {(int64_t)1, (int64_t)2, (int64_t)5000, (int64_t)1 << 20, (int64_t)307000000,
                      (int64_t)306783379, ((int64_t)1 << 30) - 1, (int64_t)1 << 30})
        for (int leaf : {1, 2, 3, 16, 64})
            for (int level = 1; level <= kMaxLevel; level++) {
                const int64_t words = kInnerWords * n;
                // all bodies in one block, and in about a thousand uneven ones
                if (subtree_splits(level, n, leaf) > words) return puts("one block"), 1;
                int64_t left = n, top = 0;
                while (left > 0) {
                    int64_t b = 1 + (int64_t)(rng() % (2 * (n / 1000 + 1)));
                    if (b > left) b = left;
                    const int64_t need = subtree_splits(level, b, leaf);
                    // clusters of leaf + 1 bodies that split on every level down to 20
                    if (need < (20 - level) * (b / (leaf + 1))) return puts("need"), 1;
                    if (need < 0 || top + need > words) return puts("past the buffer"), 1;
                    top += need;
                    left -= b;
                }
            }
    // the sum that a 32-bit counter could not hold
    printf("%d\n", subtree_splits(7, (int64_t)1 << 30, 1) > INT32_MAX);
    return 0;
}
"""


def test_subtree_lists_fit(tmp_path):
    (tmp_path / "cap.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I",
                    os.path.join(ROOT, "paper_1912_04197_amd", "csrc"),
                    str(tmp_path / "cap.cpp"), "-o", str(tmp_path / "cap")], check=True)
    r = subprocess.run([str(tmp_path / "cap")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert r.stdout == "1\n"
