"""What a build makes of the previous build's launch hints (csrc/build_plan.h, compiled
for the host): which levels get launches, where whole subtrees start and how many
passes sort, on either side of each rule's line."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LEVELS = 22

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "build_plan.h"
int main(int argc, char **argv)  // n, scenes, hint words
{
    using namespace bhx;
    if (argc != 3 + kHintWords) return 2;
    int32_t hint[kHintWords];
    for (int k = 0; k < kHintWords; k++) hint[k] = atoi(argv[3 + k]);
    const LevelPlan p = plan_levels(hint, atoll(argv[1]), atoi(argv[2]));
    bool even;
    const int passes = sort_passes(hint, atoll(argv[1]), atoi(argv[2]), &even);
    printf("%d %d %lld %d %d %d\n", p.deep, p.sub, (long long)p.sub_nodes, (int)p.prefix, passes,
           (int)even);
}
"""


RECAPTURE = r"""
#include <cstdio>
#include "build_plan.h"
using namespace bhx;
static int captures(int calls, int period, int most)  // the wanted level turns every `period` calls
{
    int32_t hint[kHintWords] = {};
    Recapture r;
    int sub = 5, n = 0;
    for (int k = 0; k < calls; k++) {
        const int now = 5 + (k / period) % 2;
        hint[kHintMost + 5] = hint[kHintMost + 6] = most;
        if (r.due(hint, 2, sub, 2, now)) sub = now, n++;
    }
    return n;
}
int main()
{
    int32_t hint[kHintWords] = {};
    Recapture r;
    // nothing new; a first change at once; a lasting one after at most kLongest calls
    printf("%d", r.due(hint, 2, 5, 2, 5));
    printf("%d", r.due(hint, 2, 5, 3, 5));
    int waited = 0;
    for (int k = 0; k < 10; k++)
        for (int w = 0; !r.due(hint, 3, 5, 2, 5); w++) waited = w + 1 > waited ? w + 1 : waited;
    printf(" %d", waited);
    // what has stopped to fit: at once, whatever the wait
    printf(" %d", r.due(hint, 2, 5, 0, 5));
    hint[kHintMost + 5] = 1025;
    printf("%d", r.due(hint, 2, 5, 2, 6));
    hint[kHintMost + 5] = 1024;
    printf("%d", r.due(hint, 2, 5, 2, 6));
    printf(" %d %d\n", captures(1000, 1, 256), captures(1000, 1, 2000));
}
"""


def test_recapture(tmp_path):
    (tmp_path / "r.cpp").write_text(RECAPTURE)
    subprocess.run(["g++", "-std=c++17", "-D__host__=", "-D__device__=", "-I",
                    os.path.join(ROOT, "paper_1912_04197_amd", "csrc"), str(tmp_path / "r.cpp"),
                    "-o", str(tmp_path / "r")], check=True)
    out = subprocess.run([str(tmp_path / "r")], capture_output=True, text=True,
                         check=True).stdout.split()
    assert out[:3] == ["01", "64", "110"]
    assert int(out[3]) <= 30  # a level that hovers: not a capture a call
    assert int(out[4]) == 999  # subtrees that are too large: each time


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__host__=", "-D__device__=", "-I",
                    os.path.join(ROOT, "paper_1912_04197_amd", "csrc"), str(d / "plan.cpp"),
                    "-o", str(d / "plan")], check=True)

    def call(n, hint, scenes=1):
        out = subprocess.run([str(d / "plan"), str(n), str(scenes), *map(str, hint)],
                             capture_output=True, text=True, check=True).stdout.split()
        return dict(zip(("deep", "sub", "sub_nodes", "prefix", "passes", "even"), map(int, out)))

    return call


def _hint(bodies, count, most, scenes=1):
    """The words that a build of `count` nodes and `most` bodies in a node per level leaves."""
    count = list(count) + [0] * (LEVELS - len(count))
    most = list(most) + [0] * (LEVELS - len(most))
    depth = max(k for k, c in enumerate(count) if c) if any(count) else 0
    return [depth, most[5], *count, *most, bodies, scenes]


NONE = [-1] * (4 + 2 * LEVELS)
SMALL = _hint(5000, [1, 8, 64, 500, 800], [5000, 800, 120])
BALL = _hint(5000, [1, 8, 64, 370, 1996, 709], [0] * 5 + [4])  # leaf 4
TINY = _hint(4097, [1, 8, 64, 300], [4097, 700, 100])
LARGE = _hint(1 << 20, [1, 8, 64, 512, 4096, 30000, 200000, 600000, 60000, 3000],
              [0, 0, 0, 0, 0, 90])


def test_without_hints(plan):
    assert plan(100000, NONE) == dict(deep=21, sub=-1, sub_nodes=0, prefix=1, passes=0, even=0)


def test_from_the_same_scene(plan):
    assert plan(5000, SMALL) == dict(deep=5, sub=2, sub_nodes=64, prefix=0, passes=2, even=1)
    got = plan(1 << 20, LARGE)
    assert got == dict(deep=10, sub=5, sub_nodes=30000, prefix=1, passes=3, even=1)


def test_a_large_scene_after_a_small_one(plan):
    """Levels are added for the growth (a factor of 210: four), and the subtrees start
    where nodes of 120 * 210 / 8^k bodies are small."""
    assert plan(1 << 20, SMALL) == dict(deep=9, sub=5, sub_nodes=8 ** 5, prefix=1, passes=2, even=1)
    assert plan(10000, SMALL)["deep"] == 5 and plan(10000, SMALL)["sub"] == 2
    assert plan(10001, SMALL)["deep"] == plan(40000, SMALL)["deep"] == 6
    assert plan(9000, SMALL)["sub_nodes"] == 64
    assert plan(40001, SMALL)["deep"] == 7
    assert plan(1 << 30, SMALL)["deep"] == 14
    # four launched levels or five: level 2 while 100 bodies grow to 256 at most
    assert plan(10488, TINY)["sub"] == 2 and plan(10489, TINY)["sub"] == 3
    assert plan(10489, TINY)["sub_nodes"] == 8 ** 3
    # as many blocks as the level's cells need, not those of the small scene's nodes
    assert plan(40000, BALL) == dict(deep=7, sub=5, sub_nodes=8 ** 5, prefix=1, passes=2, even=1)
    assert plan(9000, BALL)["sub_nodes"] == 709


def test_a_small_scene_after_a_large_one(plan):
    for n in (5000, 300000):
        assert plan(n, LARGE) == dict(deep=10, sub=5, sub_nodes=min(30000, n), prefix=1, passes=2,
                                      even=1)


def test_unknown_levels_after_large_nodes(plan):
    """Levels that the previous build did not look at are guessed only below small nodes."""
    h = _hint(50000, [1, 8, 64, 512, 4096], [50000, 9000, 1500, 300])
    assert plan(50000, h)["sub"] == -1
    assert plan(500000, h)["sub"] == -1


def test_scenes(plan):
    many = _hint(51200, [64, 500, 4000], [800, 120, 16], scenes=64)
    assert plan(51200, many, 64)["sub"] == 1
    assert plan(51200, many, 32)["sub"] == 1
    # one scene of 64 times a scene's bodies
    assert plan(51200, many, 1) == dict(deep=6, sub=5, sub_nodes=8 ** 5, prefix=1, passes=2, even=1)
    assert plan(51200, many, 300)["passes"] == 0  # more scenes than a block's offsets


def test_third_pass(plan):
    def at(nodes, n, most=1024, of=None):
        return plan(n, _hint(of or n, [1, 8, 64, 512, 4096, nodes], [0] * 5 + [most]))["passes"]

    assert at(10000, 240000) == 2
    assert at(10000, 240001) == 3
    # few level-5 nodes because most bodies are in leaves above: all buckets are small
    assert at(500, 20000, most=32) == 2 and at(500, 20000, most=33) == 3
    assert at(500, 40001, most=32, of=20000) == 3  # grown past it
    # crowded level-5 nodes: a level of small nodes down to 8
    for most, passes in (([1025, 1024], 3), ([1025, 1025, 1024], 3), ([4000, 4000, 4000, 1024], 3),
                         ([4000, 4000, 4000, 1025, 900], 0), ([1025], 0)):
        h = _hint(100000, [1, 8, 64, 512, 4096] + [9000] * 6, [0] * 5 + most)
        assert plan(100000, h)["passes"] == passes
        assert plan(200000, h)["passes"] == passes  # up to twice as many bodies
        assert plan(800001, h)["passes"] == 0
        assert not plan(100000, h)["even"]


def test_after_a_one_block_build(plan):
    h = [7, -1] + [1] * 8 + [0] * 14 + [-1] * 22 + [4096, 1]
    assert plan(5000, h) == dict(deep=8, sub=-1, sub_nodes=0, prefix=1, passes=0, even=0)
