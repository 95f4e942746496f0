// Aggregate identification (subsection "Post-processing: aggregate
// identification"): bodies are the vertices of a graph whose edges are the
// contacts, and aggregates are its connected components with more than one
// body. The paper fills a contact container from its contact model and
// traverses the graph depth first; here the contacts are sphere overlaps
// found on the GPU with the Morton-sorted bodies of the tree build, and the
// components come from a lock-free union-find over those edges.
//
//   1. the cell level: the deepest tree level whose cell side is at least the
//      largest contact distance 2 r_max + skin, so every contact joins two
//      bodies in the same or adjacent cells of that level;
//   2. one thread per sorted body scans the bodies of its own cell and of the
//      neighbouring cells later in the Morton order (the earlier ones hold
//      earlier bodies only) and, for every body later in the sorted order
//      within r_s + r_t + skin, counts the contact and unites the two bodies'
//      sets. A cell is a contiguous key range; a table of the ranges of the cells
//      of level min(cell level, table level) gives it in one load, or bounds the
//      search for it. The radii are first gathered into sorted order;
//   3. union-find on caller indices: a set is named by its smallest index,
//      the larger of two roots is linked under the smaller with a
//      compare-and-swap, finds halve paths; parent[i] <= i always, so every
//      find ends, and a failed link is always another thread's success;
//   4. every body takes its root as label; roots of sets larger than one
//      body are counted.
#include "bhx_impl.h"

namespace bhx {
namespace {

__device__ inline int32_t load_fresh(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline int32_t uf_find(int32_t *parent, int32_t x)
{
    for (;;) {
        const int32_t p = load_fresh(parent + x);
        if (p == x) return x;
        const int32_t gp = load_fresh(parent + p);
        if (gp != p) atomicCAS(parent + x, p, gp);  // path halving
        x = gp;
    }
}

__device__ inline void uf_union(int32_t *parent, int32_t a, int32_t b)
{
    for (;;) {
        a = uf_find(parent, a);
        b = uf_find(parent, b);
        if (a == b) return;
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        if (atomicCAS(parent + a, a, b) == a) return;  // larger root under the smaller
    }
}

// counters: [0] contacts, [1] aggregates, [2] bits of the largest radius (a
// non-negative double, so its bits order like the value)
__global__ __launch_bounds__(64) void k_contact_init(unsigned long long *__restrict__ counters)
{
    if (threadIdx.x < 3) counters[threadIdx.x] = 0ull;
}

// Every block ends in atomics on a shared counter, which take some 10 ns each
// one after another, so the kernels below that do little else run few large
// blocks (k_uf_finish of 200,000 bodies: 35 us with an atomic a wave, 6 with one
// for 1024 bodies).
constexpr int kWide = 1024;

// The sum, or the largest, of a 1024-thread block's values, on thread 0.
template <bool MAX>
__device__ inline unsigned long long block_reduce(unsigned long long v)
{
    __shared__ unsigned long long red[kWide / 64];
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long u = __shfl_xor(v, o);
        v = MAX ? (u > v ? u : v) : u + v;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kWide / 64; w++) {
            const unsigned long long u = red[w];
            v = MAX ? (u > v ? u : v) : u + v;
        }
    return v;
}

// The largest radius, and an empty cell table.
__global__ __launch_bounds__(kWide) void k_radius_max(const double *__restrict__ radius, int64_t n,
                                                      unsigned long long *__restrict__ counters,
                                                      int32_t *__restrict__ table, int64_t entries)
{
    const int64_t t = (int64_t)blockIdx.x * kWide + threadIdx.x, stride = (int64_t)gridDim.x * kWide;
    for (int64_t i = t; i < entries; i += stride) table[i] = 0;
    double r = 0.0;  // fmax ignores NaN; negative radii never exceed 0
    for (int64_t i = t; i < n; i += stride) r = fmax(r, radius[i]);
    const unsigned long long most =
        block_reduce<true>((unsigned long long)__double_as_longlong(r));
    if (threadIdx.x == 0) atomicMax(counters + 2, most);
}

// The deepest level whose cell side is at least the largest contact distance.
__device__ inline int contact_level(double skin, const SceneBox &box,
                                    const unsigned long long *__restrict__ counters)
{
    const double r = __longlong_as_double((long long)counters[2]);
    const double reach = 2.0 * r + skin;
    int level = 0;
    while (level < kMaxLevel && ldexp(box.L, -(level + 1)) >= reach) level++;
    return level;
}

// Radii in sorted order (rs[s] = radius[idx[s]]), so the contact test reads them
// next to the bodies; every body its own set; the set sizes; and the sorted
// positions [table[2c], table[2c + 1]) of every non-empty cell c of the table's
// level.
__global__ __launch_bounds__(256) void k_contact_prep(
    const double *__restrict__ radius, const uint32_t *__restrict__ idx,
    const uint64_t *__restrict__ keys, int64_t n, double skin, const SceneBox *__restrict__ box,
    const unsigned long long *__restrict__ counters, int table_level, double *__restrict__ rs,
    int32_t *__restrict__ label, int32_t *__restrict__ size, int32_t *__restrict__ table)
{
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    rs[s] = radius[idx[s]];
    label[s] = (int32_t)s;
    size[s] = 0;
    const int shift = 3 * (kMaxLevel - min(contact_level(skin, box[0], counters), table_level));
    const uint64_t c = keys[s] >> shift;
    if (s == 0 || keys[s - 1] >> shift != c) table[2 * c] = (int32_t)s;
    if (s == n - 1 || keys[s + 1] >> shift != c) table[2 * c + 1] = (int32_t)s + 1;
}

// First position in [lo, hi) whose key is >= k, or hi.
__device__ inline int64_t lower_bound(const uint64_t *__restrict__ keys, int64_t lo, int64_t hi,
                                      uint64_t k)
{
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < k)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// A chain of dependent loads a cell bounds it (a thread's searches), so the
// table replaces them: 200,000 bodies of a rubble pile took 188 us with a search
// over all keys for each of 27 cells, 57 us with the table and the later cells.
__global__ __launch_bounds__(256) void k_contacts(const Body *__restrict__ body,
                                                  const uint64_t *__restrict__ keys,
                                                  const uint32_t *__restrict__ idx,
                                                  const double *__restrict__ rsort, int64_t n,
                                                  double skin, const SceneBox *__restrict__ box,
                                                  int table_level,
                                                  const int32_t *__restrict__ table,
                                                  int32_t *__restrict__ parent,
                                                  unsigned long long *__restrict__ counters)
{
#pragma clang fp contract(off)
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned long long found = 0;
    if (s < n) {
        const int level = contact_level(skin, box[0], counters);
        const int coarse = 3 * (level - min(level, table_level));  // bits below the table's cells
        const int drop = kMaxLevel - level;  // bits below the level's cell coordinate
        const uint64_t key = keys[s];
        const uint64_t own = key >> (3 * drop);
        const int32_t c[3] = {(int32_t)(compact3(key >> 2) >> drop),
                              (int32_t)(compact3(key >> 1) >> drop),
                              (int32_t)(compact3(key) >> drop)};
        const int32_t nside = 1 << level;
        const Body me = body[s];
        const double rs = rsort[s];
        int32_t is = -1;  // caller index, loaded at the first contact
        for (int dx = -1; dx <= 1; dx++) {
            const int32_t x = c[0] + dx;
            if (x < 0 || x >= nside) continue;
            for (int dy = -1; dy <= 1; dy++) {
                const int32_t y = c[1] + dy;
                if (y < 0 || y >= nside) continue;
                for (int dz = -1; dz <= 1; dz++) {
                    const int32_t z = c[2] + dz;
                    if (z < 0 || z >= nside) continue;
                    const uint64_t nb = (spread3((uint64_t)x) << 2) |
                                        (spread3((uint64_t)y) << 1) | spread3((uint64_t)z);
                    if (nb < own) continue;  // earlier bodies only
                    int64_t lo = table[2 * (nb >> coarse)], hi = table[2 * (nb >> coarse) + 1];
                    if (coarse) {
                        lo = lower_bound(keys, lo, hi, nb << (3 * drop));
                        hi = lower_bound(keys, lo, hi, (nb + 1) << (3 * drop));
                    }
                    for (int64_t t = lo > s + 1 ? lo : s + 1; t < hi; t++) {
                        const Body o = body[t];
                        const double ex = o.x - me.x, ey = o.y - me.y, ez = o.z - me.z;
                        const double d2 = ex * ex + ey * ey + ez * ez;
                        const double R = rs + rsort[t] + skin;
                        if (d2 <= R * R) {
                            found++;
                            if (is < 0) is = (int32_t)idx[s];
                            uf_union(parent, is, (int32_t)idx[t]);
                        }
                    }
                }
            }
        }
    }
    // one atomic per block on the contact counter
    __shared__ unsigned long long red[4];
    for (int o = 32; o > 0; o >>= 1) found += __shfl_xor(found, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = found;
    __syncthreads();
    if (threadIdx.x == 0) {
        found = red[0] + red[1] + red[2] + red[3];
        if (found) atomicAdd(counters, found);
    }
}

__global__ __launch_bounds__(256) void k_uf_flatten(int32_t *__restrict__ label, int64_t n,
                                                    int32_t *__restrict__ size)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t r = uf_find(label, (int32_t)i);
    atomicAdd(size + r, 1);
}

__global__ __launch_bounds__(kWide) void k_uf_finish(int32_t *__restrict__ label, int64_t n,
                                                     const int32_t *__restrict__ size,
                                                     unsigned long long *__restrict__ counters)
{
    unsigned long long sets = 0;  // of more than one body, by their roots
    for (int64_t i = (int64_t)blockIdx.x * kWide + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kWide) {
        label[i] = uf_find(label, (int32_t)i);
        sets += size[i] > 1 ? 1 : 0;
    }
    sets = block_reduce<false>(sets);
    if (threadIdx.x == 0 && sets) atomicAdd(counters + 1, sets);
}

inline unsigned grid(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_contacts(const Workspace &w, hipStream_t s, const double *radius, int64_t n,
                           double skin, int32_t *label, int32_t *size,
                           unsigned long long *counters)
{
    if (n <= 0) return hipSuccess;
    // the build's list buffer is free after it: the cell table, of the deepest
    // level that fits (two words a cell) and has at most about eight cells a body
    int table_level = 0;
    while (table_level < kMaxLevel && (2ll << (3 * (table_level + 1))) <= w.inner_words &&
           (1ll << (3 * table_level)) < n)
        table_level++;
    int32_t *table = w.inner;
    const int64_t entries = 2ll << (3 * table_level);
    const unsigned wide = (unsigned)((n + kWide - 1) / kWide < 256 ? (n + kWide - 1) / kWide : 256);
    // the sort's second key buffer is free too: sorted radii
    double *rsort = reinterpret_cast<double *>(w.keys[1]);
    k_contact_init<<<1, 64, 0, s>>>(counters);
    k_radius_max<<<wide, kWide, 0, s>>>(radius, n, counters, table, entries);
    k_contact_prep<<<grid(n), 256, 0, s>>>(radius, w.idx[0], w.keys[0], n, skin, w.box, counters,
                                           table_level, rsort, label, size, table);
    k_contacts<<<grid(n), 256, 0, s>>>(w.body, w.keys[0], w.idx[0], rsort, n, skin, w.box,
                                       table_level, table, label, counters);
    k_uf_flatten<<<grid(n), 256, 0, s>>>(label, n, size);
    k_uf_finish<<<wide, kWide, 0, s>>>(label, n, size, counters);
    return hipGetLastError();
}

}  // namespace bhx
