// What a build makes of the launch hints that the previous build left: plain
// functions of the hint words that the host code and a host program share. The
// hints only choose launches and a sort; any choice builds the same tree.
#pragma once

#include <cstdint>

#include "capacity.h"

namespace bhx {

// The pinned words, -1 before the first build.
enum HintWord : int {
    kHintDepth = 0,                  // deepest non-empty level
    kHintMost5 = 1,                  // most bodies in one node of level kHintLevel (-1: no sort hint)
    kHintCount = 2,                  // [kLevels] nodes per level
    kHintMost = 2 + kLevels,         // [kLevels] most bodies in one node per level (0 or less: not known)
    kHintBodies = 2 + 2 * kLevels,   // bodies of that build, all scenes together
    kHintScenes = 3 + 2 * kLevels,   // its scenes
    kHintWords = 4 + 2 * kLevels,
};

constexpr int64_t kSmallBuild = 4096;  // a single scene this small is built by one block
// The level whose largest node the build reports for the choice of sort.
constexpr int kHintLevel = 5;
// The levels 1..kPrefixLevels of a single scene's tree are read off the
// sorted keys: a level-kPrefixLevels cell is the key's top 3 kPrefixLevels
// bits, and the first body of each such cell gives every cell range above it.
constexpr int kPrefixLevels = 5;
// The buckets of two passes lie inside cells of level kHintLevel, of three of:
constexpr int kBucketLevel3 = 8;
constexpr int kBucketMax = 1024;  // bucket bound the bucket sort's blocks are sized for
// A range whose buckets all hold at most kRankMax keys is sorted by comparison
// instead of radix passes (200,000 bodies, 18 a level-5 node: builds of 108 us, not
// 132). Each key's comparisons walk its bucket in LDS, so the cost grows with the
// bucket.
constexpr int kRankMax = 32;
// From this mean number of bodies per level-5 node (two buckets) most ranges hold a
// larger bucket, and a third pass costs less than radix passes in LDS: builds of
// 2^20 evenly spread bodies (32 a node) take 194 us with it and 211 without, of 2^21
// 315 and 357; 500,000 (15) 146 and 140, 200,000 of a ball (18) 118 and 108. Where no
// level-5 node is larger than a comparison takes, the mean is high because most bodies
// are in leaves above, and the pass would be lost (20,000 bodies of a ball, leaf 16: 98
// us with it, 83 without; 131,072, leaf 64: 124 and 113).
constexpr int64_t kThirdPassFrom = 24;
constexpr int kLdsScenes = 256;   // scenes whose offsets a sorting block holds
constexpr int kSubBodies = 256;   // see k_build_subtrees

// By how much the scenes of a build of n bodies are larger than those of the build that
// left the hints, when it is more than twice (1 otherwise: a hint of a similar or a
// larger scene is used as it is, its nodes hold as many bodies or more).
inline double hint_growth(const volatile int32_t *hint, int64_t n, int scenes)
{
    const double from = (double)hint[kHintBodies] * scenes, to = (double)n * hint[kHintScenes];
    return hint[kHintBodies] > 0 && to > 2.0 * from ? to / from : 1.0;
}

// How a build launches its levels, read once from the previous build's hints:
// levels 0..deep-1 get a launch each (the deeper ones share one block): one more than
// that build had, and another for each factor of four of growth. With
// `prefix` a single scene's levels 1..kPrefixLevels are read off the
// sorted keys instead (the gather writes the marks k_prefix_levels reads).
// With sub >= 0 the levels below it, and its moments, are left to one launch
// of k_build_subtrees for about sub_nodes nodes: sub is the first level (from the
// first that is launched) whose nodes held at most kSubBodies bodies in the
// previous build; of a scene that has grown, the level on which they would, if nodes
// grow alike and each level's hold an eighth of those above. The previous build's
// own level and node count gave 2^20 bodies after 5000 twelve blocks for all below level
// 5: 1.09 ms, now 0.29 (repeated builds 0.23); 40,000 after 5000 0.20, now 0.11 (0.10).
struct LevelPlan {
    int deep = kMaxLevel, prev = -1, sub = -1;
    int64_t sub_nodes = 0;
    bool prefix = false;
};

inline LevelPlan plan_levels(const volatile int32_t *hint, int64_t n, int scenes)
{
    LevelPlan p;
    if (!hint || hint[kHintDepth] < 0) {
        p.prefix = scenes == 1;
        return p;
    }
    const double growth = hint_growth(hint, n, scenes);
    p.prev = hint[kHintDepth];
    int64_t deep = p.prev + 1;
    for (double g = growth; g > 2.0; g /= 4.0) deep++;
    if (deep < p.deep) p.deep = (int)deep;
    p.prefix = scenes == 1 && p.deep > kPrefixLevels;
    const int first = p.prefix ? kPrefixLevels : 1;  // (the root's moments launch reports the hints)
    double most = 0.0, cells = scenes;  // largest node of level l (guessed from above); its cells
    for (int l = 1; l < kMaxLevel; l++) {
        cells *= 8.0;
        if (hint[kHintMost + l] > 0)
            most = hint[kHintMost + l];
        else if (most > 0.0 && most <= kSubBodies)  // the previous subtrees began above
            most /= 8.0;
        else if (most > 0.0 || l >= first)
            break;
        if (l < first || most * growth > kSubBodies) continue;
        p.sub = l;
        // (a scene that has grown: as many as there can be; a block too many ends at once)
        if (growth == 1.0 && hint[kHintMost + l] > 0) cells = hint[kHintCount + l];
        p.sub_nodes = cells < (double)n ? (int64_t)cells : n;
        break;
    }
    return p;
}

// How a build sorts: by buckets after 2 or 3 passes on the top key bits or, 0, by
// passes over the whole keys. even: whether level kHintLevel's nodes allow buckets.
// A range is a tile plus at most one bucket, and a bucket lies inside one cell of
// level kHintLevel or kBucketLevel3; a cell that is no node holds at most a leaf's
// bodies, and a level's bound holds for the levels below it.
inline int sort_passes(const volatile int32_t *hint, int64_t n, int scenes, bool *even)
{
    *even = false;
    if (!hint || scenes > kLdsScenes || n <= kSmallBuild || hint[kHintMost5] < 0) return 0;
    const double growth = hint_growth(hint, n, scenes);
    const int64_t nodes = hint[kHintCount + kHintLevel];
    if (hint[kHintMost5] <= kBucketMax) {
        *even = true;
        return nodes > 0 && n > kThirdPassFrom * nodes && hint[kHintMost5] * growth > kRankMax ? 3
                                                                                               : 2;
    }
    for (int l = kHintLevel + 1; l <= kBucketLevel3; l++)
        if (hint[kHintMost + l] > 0 && hint[kHintMost + l] * growth <= kBucketMax) return 3;
    return 0;
}

// When a captured step, whose build froze the sort (`passes`) and subtree level (`sub`)
// of its time, is captured again because the hints now give others. Both still build
// the same tree; a capture costs about 50 us (one-step calls of 50,000 bodies: 290 us
// replayed, 337 captured each). A choice that has stopped to
// fit (a bucket beyond the sort's blocks, subtrees of several times kSubBodies bodies)
// is replaced at once; others after a wait that doubles with each capture, so that a
// largest node that hovers about a rule's line costs a few captures, not one a call.
struct Recapture {
    static constexpr int kLongest = 64;  // calls
    int hold = 0, next = 1;

    bool due(const volatile int32_t *hint, int passes, int sub, int passes_now, int sub_now)
    {
        if (passes == passes_now && sub == sub_now) return false;
        const bool fits = !(passes > 0 && passes_now == 0) &&
                          !(sub >= 0 && hint && hint[kHintMost + sub] > 4 * kSubBodies);
        if (fits && hold > 0) {
            hold--;
            return false;
        }
        hold = next;
        next = next < kLongest ? 2 * next : kLongest;
        return true;
    }
};

}  // namespace bhx
