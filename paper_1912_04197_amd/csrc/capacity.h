// Sizes of a workspace's arrays: plain functions that the device code, the host
// code and a host program share.
#pragma once

#include <cstdint>

namespace bhx {

constexpr int kMaxLevel = 21;           // cells on a 2^21 grid per axis
constexpr int kLevels = kMaxLevel + 1;  // levels 0..21

// Upper bound on the node count of the trees of n bodies in up to `scenes`
// scenes with the given bucket size: one root per scene, and every level
// below holds at most min(n, 8 n / (leaf + 1)) nodes, because its nodes are
// disjoint non-empty children of cells holding more than `leaf` bodies.
inline int64_t node_capacity(int64_t n, int leaf, int scenes = 1)
{
    if (n <= 0) return scenes > 1 ? scenes : 1;
    int64_t internal = n / (leaf + 1);
    int64_t per_level = 8 * internal < n ? 8 * internal : n;
    return (int64_t)(scenes > 1 ? scenes : 1) + (int64_t)kMaxLevel * per_level;
}

// The nodes that split below level `level` in subtrees of `bodies` bodies: their
// level holds at most bodies / (leaf + 1) of them, and level kMaxLevel splits none.
__host__ __device__ inline int64_t subtree_splits(int level, int64_t bodies, int leaf)
{
    return (kMaxLevel - level) * (bodies / (leaf + 1));
}

// 32-bit words of the buffer that lists them (Workspace::inner), which holds any
// build's: subtrees start below level 0, and a leaf holds one body at least. It is
// also the contact search's table, which takes less than 16 words a body.
constexpr int64_t kInnerWords = 16;  // a body
static_assert(kInnerWords >= (kMaxLevel - 1) / 2, "lists of subtrees");

}  // namespace bhx
