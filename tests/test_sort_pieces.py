"""The pieces in which a block of the bucket sort sorts its range (csrc/sort_pieces.h,
compiled for the host): whatever a piece's passes through global memory have done so
far, another block finds its own range where it was, every range is sorted once and
the order is the stable sort's."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "sort_pieces.h"

using Key = uint64_t;
static std::vector<Key> keys;       // as other blocks see them
static std::vector<int> vals;

static int64_t bucket_end(int64_t from, Key top, int shift)
{
    int64_t i = from;
    while (i < (int64_t)keys.size() && (keys[i] >> shift) == top) i++;
    return i;
}
// The whole buckets that start in the tile [t0, t1).
static std::pair<int64_t, int64_t> range(int64_t t0, int64_t t1, int shift)
{
    return {t0 ? bucket_end(t0, keys[t0 - 1] >> shift, shift) : 0,
            bucket_end(t1, keys[t1 - 1] >> shift, shift)};
}

int main(int argc, char **argv)
{
    const int64_t tile = atoi(argv[1]), cap = tile + atoi(argv[2]);
    const int shift = atoi(argv[3]);
    std::mt19937_64 rng(atoi(argv[4]));
    // buckets of 1 key to several tiles, large ones one after another too
    std::vector<int> sizes;
    for (int k = 0; k < 60; k++)
        sizes.push_back(rng() % 4 == 0 ? 1 + rng() % (5 * cap) : 1 + rng() % (tile / 8));
    Key top = 0;
    for (int sz : sizes) {
        top += 1 + rng() % 3;
        for (int j = 0; j < sz; j++) {
            keys.push_back(top << shift | (rng() % 64) * 0x0101010101010101ull % (1ull << shift));
            vals.push_back((int)vals.size());
        }
    }
    const int64_t n = (int64_t)keys.size();
    std::vector<std::pair<Key, int>> want(n);
    for (int64_t i = 0; i < n; i++) want[i] = {keys[i], vals[i]};
    std::stable_sort(want.begin(), want.end(),
                     [](const auto &a, const auto &b) { return a.first < b.first; });
    std::vector<std::pair<int64_t, int64_t>> ranges;
    for (int64_t t0 = 0; t0 < n; t0 += tile) ranges.push_back(range(t0, std::min(t0 + tile, n), shift));
    std::vector<char> seen(n, 0);
    std::vector<size_t> order(ranges.size());
    for (size_t k = 0; k < order.size(); k++) order[k] = k;
    std::shuffle(order.begin(), order.end(), rng);
    int64_t global = 0;
    for (size_t blk : order) {
        const auto [ra, rb] = ranges[blk];
        if (ra >= std::min<int64_t>((blk + 1) * tile, n)) continue;
        for (int64_t a = ra; a < rb;) {
            const int64_t b = bhx::piece_end(keys.data(), a, rb, cap, shift);
            if (b <= a || b > rb) return puts("piece outside the range"), 1;
            for (int64_t i = a; i < b; i++)
                if (seen[i]++) return puts("sorted twice"), 1;
            global += b - a > cap;
            // stable passes on one byte each; beyond cap every pass's result can be seen
            for (int p = 0; p < 8; p++) {
                std::vector<std::pair<Key, int>> t;
                for (int64_t i = a; i < b; i++) t.push_back({keys[i], vals[i]});
                std::stable_sort(t.begin(), t.end(), [p](const auto &x, const auto &y) {
                    return (x.first >> 8 * p & 255) < (y.first >> 8 * p & 255);
                });
                for (int64_t i = a; i < b; i++) keys[i] = t[i - a].first, vals[i] = t[i - a].second;
                if (b - a <= cap && p < 7) continue;  // in LDS until the last pass
                for (size_t k = 0; k < ranges.size(); k++)
                    if (range((int64_t)k * tile, std::min<int64_t>((k + 1) * tile, n), shift) != ranges[k])
                        return puts("a block finds another range"), 1;
            }
            a = b;
        }
    }
    for (int64_t i = 0; i < n; i++)
        if (!seen[i] || keys[i] != want[i].first || vals[i] != want[i].second)
            return puts("not the stable order"), 1;
    printf("%lld\n", (long long)global);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    (d / "pieces.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I",
                    os.path.join(ROOT, "paper_1912_04197_amd", "csrc"), str(d / "pieces.cpp"),
                    "-o", str(d / "pieces")], check=True)
    return str(d / "pieces")


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("tile,over,shift", [(64, 96, 39), (128, 32, 47)])
def test_ranges_stay_where_they_were(program, tile, over, shift, seed):
    """Tiles and capacities of a scaled-down block; buckets larger than the capacity
    occur in every run."""
    r = subprocess.run([program, str(tile), str(over), str(shift), str(seed)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 0
