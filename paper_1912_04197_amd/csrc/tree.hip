// Octree construction on the device, rebuilt on every force evaluation
// (subsection "Hierarchical treecode algorithm"; the five GPU stages of
// subsection "CUDA implementation of GPU-parallel Barnes-Hut" are prior art,
// this is a Morton-key design for CDNA4):
//   1. bounding box of each scene's bodies -> its root cube (and input
//      validation); a call may hold many independent scenes, stored as
//      contiguous body ranges, each with its own root,
//   2. 63-bit Morton keys on a 2^21 grid,
//   3. stable sort of (key, index): radix passes on 8-bit digits over the whole
//      key, or on its top digits and the rest in LDS; for several scenes passes on
//      the scene index too,
//   4. gather of positions, masses and softening into Morton order,
//   5. top-down octree, one launch per level: each split cell finds its
//      octant ranges by binary search in the sorted keys,
//   6. bottom-up moments, one launch per level: mass and centre of mass from
//      the children by eq. (COMinternal), leaves from their bodies; from the
//      level where nodes are small one launch makes whole subtrees, 5 and 6 both.
// A single scene of at most kSmallBuild bodies takes one launch for all of it.
// Every launch reads its sizes from the device tree header, so the sequence
// needs no host round trip and can be captured in a graph.
#include <cmath>
#include <cstddef>

#include "bhx_impl.h"
#include "sort_pieces.h"

namespace bhx {
namespace {

constexpr double kInf = __builtin_huge_val();

__device__ inline uint64_t lanemask_lt(int lane) { return (1ull << lane) - 1ull; }

template <typename T>
__device__ inline T wave_min(T v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}
template <typename T>
__device__ inline T wave_max(T v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

// The smallest and largest of a row's 16 lanes' values, on every lane of the row,
// by DPP lane moves (a lane permute goes through the LDS unit, which the 16
// waves of a block share).
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128;
__device__ inline double row_min(double v)
{
    v = fmin(v, dpp_f64<kDppXor1>(v));
    v = fmin(v, dpp_f64<kDppXor2>(v));
    v = fmin(v, dpp_f64<kDppRor4>(v));
    return fmin(v, dpp_f64<kDppRor8>(v));
}
__device__ inline double row_max(double v)
{
    v = fmax(v, dpp_f64<kDppXor1>(v));
    v = fmax(v, dpp_f64<kDppXor2>(v));
    v = fmax(v, dpp_f64<kDppRor4>(v));
    return fmax(v, dpp_f64<kDppRor8>(v));
}

// Inclusive scan over a 256-thread block (4 waves).
__device__ inline uint32_t block_incl_scan_256(uint32_t v, uint32_t *lds4, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_incl_scan(v);
    if (lane == 63) lds4[wave] = v;
    __syncthreads();
    uint32_t add = 0, tot = 0;
    for (int w = 0; w < 4; w++) {
        uint32_t x = lds4[w];
        if (w < wave) add += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return v + add;
}

// ---------------------------------------------------------------- 1. box

// Order-preserving map of doubles to unsigned integers, so integer atomics
// give the exact minimum and maximum whatever the order of the updates.
__device__ inline unsigned long long order_enc(double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ inline double order_dec(unsigned long long e)
{
    const unsigned long long b = (e >> 63) ? (e & 0x7fffffffffffffffull) : ~e;
    return __longlong_as_double((long long)b);
}

// Encodings of a box without bodies. A context's boxes hold these from its creation
// and between builds: a build's last kernel sets them again (a launch of its own at
// the build's start cost 5 us).
__device__ inline void reset_box(SceneBox *box)
{
    for (int a = 0; a < 3; a++) box->lo_enc[a] = box->hi_enc[a] = ~0ull;
    box->mild_acc = ~0u;
}

// Whether a body's mass and softening (squared) leave the ranges of kMild*.
__device__ inline bool wild_body(double m, double e2)
{
    return !(mild_mass(m) && e2 <= kMildEps2);
}

// One work item: a chunk of at most kBoxChunk bodies of one scene (for one
// scene, chunk c is the `per` bodies from c*per on). Reduces its box in the block
// and merges it into the scene's with integer atomics; flags bad input.
constexpr int kBoxThreads = 1024;  // one block per chunk: up to 4 bodies per thread

// Bodies per chunk of a single scene: one a thread while that leaves no more
// blocks than CUs (each block ends in six atomics on shared words).
// 50,000 bodies: 13 blocks of 4096 took 13 us for the kick and drift, 49 of 1024
// take 8.7; 2^20: 256 blocks either way.
inline int box_chunk(int64_t n)
{
    int per = kBoxThreads;
    while (per < kBoxChunk && n > 256 * (int64_t)per) per *= 2;
    return per;
}

__global__ __launch_bounds__(kBoxThreads) void k_box_chunk(const double *__restrict__ pos,
                                                   const double *__restrict__ mass,
                                                   const double *__restrict__ eps, int64_t n,
                                                   int per, const int32_t *__restrict__ chunks,
                                                   SceneBox *__restrict__ box,
                                                   TreeHeader *__restrict__ hdr)
{
    int sc = 0;
    int64_t first = (int64_t)blockIdx.x * per, end = first + per;
    if (chunks) {
        sc = chunks[3 * blockIdx.x];
        first = chunks[3 * blockIdx.x + 1];
        end = chunks[3 * blockIdx.x + 2];
    }
    if (end > n) end = n;
    double lo[3] = {kInf, kInf, kInf}, hi[3] = {-kInf, -kInf, -kInf};
    bool bad = false, wild = false;
    for (int64_t i = first + threadIdx.x; i < end; i += kBoxThreads) {
        double x[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
        double m = mass[i], e = eps ? eps[i] : 0.0;
        bad |= !(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]));
        bad |= !(isfinite(m) && m >= 0.0);
        bad |= !(isfinite(e) && e >= 0.0);
        wild |= wild_body(m, e * e);
        for (int a = 0; a < 3; a++) {
            lo[a] = fmin(lo[a], x[a]);
            hi[a] = fmax(hi[a], x[a]);
        }
    }
    if (__ballot(bad) && (threadIdx.x & 63) == 0) flag_status(hdr->status, ST_NONFINITE);
    if (__ballot(wild) && (threadIdx.x & 63) == 0) atomicAnd(&box[sc].mild_acc, 0u);
    __shared__ double red[kBoxThreads / 64][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int a = 0; a < 3; a++) {
        double l = wave_min(lo[a]), h = wave_max(hi[a]);
        if (lane == 0) {
            red[wave][a] = l;
            red[wave][3 + a] = h;
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        double v = red[0][a];
        for (int w = 1; w < kBoxThreads / 64; w++)
            v = a < 3 ? fmin(v, red[w][a]) : fmax(v, red[w][a]);
        if (a < 3)
            atomicMin(&box[sc].lo_enc[a], order_enc(v));
        else
            atomicMin(&box[sc].hi_enc[a - 3], ~order_enc(v));
    }
}

// The same work items for one step of a multi-step call, on the sorted state
// of the previous build: kick and drift each body (v = v + (dt/2) a, then
// x = x + dt v, each one fused multiply-add as the caller-order step rounds
// it), write the new state in the same order to the S buffers with its mass,
// softening and caller index, and reduce the box of the new positions.
__global__ __launch_bounds__(kBoxThreads) void k_state_kick_drift(
    const Body *__restrict__ body, const double *__restrict__ tvel,
    const double *__restrict__ tacc, const double *__restrict__ beps2,
    const uint32_t *__restrict__ cidx, int64_t n, double h, double dt, int per,
    const int32_t *__restrict__ chunks, Body *__restrict__ sbody, double *__restrict__ svel,
    double *__restrict__ seps2, uint32_t *__restrict__ scidx, SceneBox *__restrict__ box,
    TreeHeader *__restrict__ hdr)
{
    int sc = 0;
    int64_t first = (int64_t)blockIdx.x * per, end = first + per;
    if (chunks) {
        sc = chunks[3 * blockIdx.x];
        first = chunks[3 * blockIdx.x + 1];
        end = chunks[3 * blockIdx.x + 2];
    }
    if (end > n) end = n;
    double lo[3] = {kInf, kInf, kInf}, hi[3] = {-kInf, -kInf, -kInf};
    bool bad = false, wild = false;
    for (int64_t i = first + threadIdx.x; i < end; i += kBoxThreads) {
        const Body b = body[i];
        const double x0[3] = {b.x, b.y, b.z};
        double x[3], v[3];
        for (int a = 0; a < 3; a++) {
            v[a] = fma(h, tacc[3 * i + a], tvel[3 * i + a]);
            x[a] = fma(dt, v[a], x0[a]);
        }
        sbody[i] = Body{x[0], x[1], x[2], b.m};
        for (int a = 0; a < 3; a++) svel[3 * i + a] = v[a];
        const double e2 = seps2 ? beps2[i] : 0.0;
        if (seps2) seps2[i] = e2;
        wild |= wild_body(b.m, e2);
        scidx[i] = cidx[i];
        bad |= !(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]));
        for (int a = 0; a < 3; a++) {
            lo[a] = fmin(lo[a], x[a]);
            hi[a] = fmax(hi[a], x[a]);
        }
    }
    if (__ballot(bad) && (threadIdx.x & 63) == 0) flag_status(hdr->status, ST_NONFINITE);
    if (__ballot(wild) && (threadIdx.x & 63) == 0) atomicAnd(&box[sc].mild_acc, 0u);
    __shared__ double red[kBoxThreads / 64][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int a = 0; a < 3; a++) {
        double l = wave_min(lo[a]), hv = wave_max(hi[a]);
        if (lane == 0) {
            red[wave][a] = l;
            red[wave][3 + a] = hv;
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        double v = red[0][a];
        for (int w = 1; w < kBoxThreads / 64; w++)
            v = a < 3 ? fmin(v, red[w][a]) : fmax(v, red[w][a]);
        if (a < 3)
            atomicMin(&box[sc].lo_enc[a], order_enc(v));
        else
            atomicMin(&box[sc].hi_enc[a - 3], ~order_enc(v));
    }
}

// Root cube: side = largest extent (1 if all bodies coincide), centred on the
// bounding box; the quantisation scale and the squared cell side per level
// (those of levels l_first, l_first + l_step, ...).
__device__ inline void root_cube(SceneBox &b, const double lo[3], const double hi[3],
                                 int l_first = 0, int l_step = 1)
{
#pragma clang fp contract(off)
    double L = 0.0;
    for (int a = 0; a < 3; a++) {
        double e = hi[a] - lo[a];
        if (e > L) L = e;
    }
    if (L == 0.0) L = 1.0;
    for (int a = 0; a < 3; a++) {
        b.lo[a] = lo[a];
        b.hi[a] = hi[a];
        b.x0[a] = (lo[a] + hi[a]) * 0.5 - L * 0.5;
    }
    b.L = L;
    b.S = 2097152.0 / L;
    for (int l = l_first; l < kLevels; l += l_step) {
        double sd = ldexp(L, -l);
        b.s2[l] = sd * sd;
    }
}

// A header for a build about to create `roots` root nodes.
__device__ inline void reset_header(TreeHeader *__restrict__ hdr, int32_t roots)
{
    for (int l = 0; l <= kLevels; l++) hdr->level_count[l] = l == 0 ? roots : 0;
    for (int l = 0; l < kLevels; l++) hdr->cell_max[l] = 0;
    hdr->deep_count = 0;
    hdr->inner_top = 0;
}

// Root cube of a scene into `out` from the reduced box encodings of `in`
// (the same SceneBox or a copy); a scene without bodies gets the cube at 0.
__device__ inline void scene_root_cube(SceneBox &out, const SceneBox &in, bool any)
{
    double lo[3], hi[3];
    for (int a = 0; a < 3; a++) {
        lo[a] = any ? order_dec(in.lo_enc[a]) : 0.0;
        hi[a] = any ? order_dec(~in.hi_enc[a]) : 0.0;
    }
    root_cube(out, lo, hi);
    out.mild = in.mild_acc != 0u && out.L <= kMildLength ? 1u : 0u;
}

// One thread per scene: root cube from the box, and the scene's root node
// (level 0, its bodies' whole range in sorted order). Thread 0 also resets
// the per-level node counts.
__global__ __launch_bounds__(256) void k_box_final(SceneBox *__restrict__ box, int n_scenes,
                                                   const int64_t *__restrict__ offsets, int64_t n,
                                                   TreeHeader *__restrict__ hdr,
                                                   NodeInfo *__restrict__ ninfo)
{
#pragma clang fp contract(off)
    const int sc = blockIdx.x * 256 + threadIdx.x;
    if (sc == 0) {
        reset_header(hdr, n > 0 ? n_scenes : 0);
    }
    if (sc >= n_scenes) return;
    const int64_t first = offsets ? offsets[sc] : 0, end = offsets ? offsets[sc + 1] : n;
    SceneBox &b = box[sc];
    scene_root_cube(b, b, end > first);
    if (end > first)
        ninfo[sc] = NodeInfo{(int32_t)first, (int32_t)(end - first), -1, (int32_t)(sc << 16)};
}

// --------------------------------------------------------------- 2. keys

// Integer cell coordinate: clamp(floor((x - x0) * S), 0, 2^21 - 1), rounded
// exactly as written so every implementation of the cell definition agrees.
__device__ inline uint32_t quantise(double x, double x0, double S)
{
#pragma clang fp contract(off)
    double f = floor((x - x0) * S);
    if (!(f >= 0.0)) return 0u;
    if (f > (double)kQMax) return kQMax;
    return (uint32_t)f;
}

__device__ inline uint64_t morton_key(const double *x, const SceneBox &b)
{
    const uint32_t qx = quantise(x[0], b.x0[0], b.S);
    const uint32_t qy = quantise(x[1], b.x0[1], b.S);
    const uint32_t qz = quantise(x[2], b.x0[2], b.S);
    return (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
}

// pos: body i's coordinates at pos + stride * i (3: caller arrays, 4: Body)
__global__ __launch_bounds__(256) void k_keys(const double *__restrict__ pos, int stride, int64_t n,
                                              const SceneBox *__restrict__ box,
                                              const uint16_t *__restrict__ scene_of,
                                              uint64_t *__restrict__ keys,
                                              uint32_t *__restrict__ idx)
{
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    keys[i] = morton_key(pos + stride * i, box[scene_of ? scene_of[i] : 0]);
    idx[i] = (uint32_t)i;
}

// --------------------------------------------------------------- 3. sort

// Scene index of caller index v: for at most kLdsScenes scenes a binary
// search of the scene offsets staged in LDS (soff), else scene_of[v].
__device__ inline uint32_t scene_index(const int64_t *soff, int ns,
                                       const uint16_t *__restrict__ scene_of, uint32_t v)
{
    if (ns > kLdsScenes) return scene_of[v];
    int lo = 0, hi = ns;  // soff[lo] <= v < soff[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (soff[mid] <= (int64_t)v)
            lo = mid;
        else
            hi = mid;
    }
    return (uint32_t)lo;
}

// Sort digit of one element: 8 bits of its key, or for shift >= 64 8 bits of
// its scene index (shift - 64 = 0 or 8).
__device__ inline uint32_t sort_digit(uint64_t key, uint32_t val, int shift, const int64_t *soff,
                                      int ns, const uint16_t *__restrict__ scene_of)
{
    if (shift < 64) return (uint32_t)(key >> shift) & 255u;
    return (scene_index(soff, ns, scene_of, val) >> (shift - 64)) & 255u;
}

// Stages the scene offsets in LDS for the scene passes (before a barrier).
__device__ inline void stage_offsets(int64_t *soff, const int64_t *__restrict__ offsets, int ns,
                                     int shift)
{
    if (shift >= 64 && ns <= kLdsScenes)
        for (int i = threadIdx.x; i <= ns; i += blockDim.x) soff[i] = offsets[i];
}

// Per-tile digit histogram, written digit-major: counts[d * nblk + tile].
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const uint64_t *__restrict__ keys,
                                                            const uint32_t *__restrict__ vals,
                                                            const uint16_t *__restrict__ scene_of,
                                                            const int64_t *__restrict__ offsets,
                                                            int ns, int64_t n, int shift,
                                                            uint32_t *__restrict__ counts,
                                                            int nblk)
{
    __shared__ uint32_t h[256];
    __shared__ int64_t soff[kLdsScenes + 1];
    h[threadIdx.x] = 0;
    stage_offsets(soff, offsets, ns, shift);
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    for (int r = 0; r < kSortItems; r++) {
        int64_t i = base + r * kSortThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[sort_digit(keys[i], vals[i], shift, soff, ns, scene_of)], 1u);
    }
    __syncthreads();
    counts[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// k_box_final and k_keys for one scene, with the tile layout of k_sort_hist,
// and that kernel's digit counts of the first pass (bits shift..shift+7) of
// the same tile.
__global__ __launch_bounds__(kSortThreads) void k_keys_hist(const double *__restrict__ pos,
                                                            int stride, int64_t n,
                                                            SceneBox *__restrict__ box,
                                                            TreeHeader *__restrict__ hdr,
                                                            NodeInfo *__restrict__ ninfo,
                                                            uint64_t *__restrict__ keys,
                                                            uint32_t *__restrict__ idx, int shift,
                                                            uint32_t *__restrict__ counts,
                                                            int nblk)
{
#pragma clang fp contract(off)
    __shared__ uint32_t h[256];
    __shared__ SceneBox b;  // this block's copy of the root cube
    h[threadIdx.x] = 0;
    // k_box_final's work for the one scene (n > 0): every block computes the
    // root cube from the reduced box for itself, block 0 also stores it, the
    // level counts and the root node (no block reads those fields here)
    if (threadIdx.x == 0) {
        scene_root_cube(b, box[0], true);
        if (blockIdx.x == 0) {
            scene_root_cube(box[0], box[0], true);
            reset_header(hdr, 1);
            ninfo[0] = NodeInfo{0, (int32_t)n, -1, 0};
        }
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    for (int r = 0; r < kSortItems; r++) {
        const int64_t i = base + r * kSortThreads + threadIdx.x;
        if (i < n) {
            const uint64_t key = morton_key(pos + stride * i, b);
            keys[i] = key;
            idx[i] = (uint32_t)i;
            atomicAdd(&h[(uint32_t)(key >> shift) & 255u], 1u);
        }
    }
    __syncthreads();
    counts[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of one digit's row of tile counts; one block per digit.
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t *__restrict__ counts,
                                                   uint32_t *__restrict__ totals, int nblk)
{
    __shared__ uint32_t lds4[4];
    uint32_t *row = counts + (int64_t)blockIdx.x * nblk;
    uint32_t carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        int b = b0 + threadIdx.x;
        uint32_t v = b < nblk ? row[b] : 0u, tot;
        uint32_t incl = block_incl_scan_256(v, lds4, &tot);
        if (b < nblk) row[b] = carry + incl - v;
        carry += tot;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Stable scatter of one tile. Wave w holds the tile's keys w*512 .. w*512+511
// (round r, lane l: key w*512 + r*64 + l, so tile order is (wave, round,
// lane) order). Each wave ranks its keys among equal digits with ballots and
// a per-wave digit count in LDS, without block barriers; one exclusive scan
// over the waves and one over the digits then place every key in a copy of
// the tile reordered by digit, so that consecutive threads write consecutive
// addresses of each digit's output run.
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    const uint16_t *__restrict__ scene_of, const int64_t *__restrict__ offsets, int ns,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n, int shift,
    const uint32_t *__restrict__ counts, const uint32_t *__restrict__ totals, int nblk)
{
    static_assert(kSortThreads == 256 && kSortItems == 8, "four waves of eight rounds");
    constexpr int kWaveKeys = 64 * kSortItems;
    __shared__ uint32_t digit_base[256];
    __shared__ uint32_t whist[4][256];  // per-wave digit counts, then per-wave digit offsets
    __shared__ uint32_t lds4[4];
    __shared__ uint32_t lstart[256];
    __shared__ uint64_t skey[kSortTile];
    __shared__ uint32_t sval[kSortTile];
    __shared__ uint8_t sdig[kSortTile];  // digits of the reordered tile
    __shared__ int64_t soff[kLdsScenes + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    stage_offsets(soff, offsets, ns, shift);  // read after the barrier below

    uint32_t tot;
    const uint32_t t = totals[tid];
    const uint32_t incl = block_incl_scan_256(t, lds4, &tot);
    digit_base[tid] = incl - t + counts[(int64_t)tid * nblk + blockIdx.x];
    for (int w = 0; w < 4; w++) whist[w][tid] = 0;
    __syncthreads();

    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    const int64_t wbase = base + wave * kWaveKeys;
    uint64_t k[kSortItems];
    uint32_t v[kSortItems], rank[kSortItems], dig[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        const int64_t i = wbase + r * 64 + lane;
        k[r] = i < n ? kin[i] : 0ull;
        v[r] = i < n ? vin[i] : 0u;
    }
    uint32_t *const wh = whist[wave];
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        const bool valid = wbase + r * 64 + lane < n;
        const uint32_t d = valid ? sort_digit(k[r], v[r], shift, soff, ns, scene_of) : 0u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const uint64_t lower = peers & lanemask_lt(lane);
        // keys of this digit ranked by earlier rounds of this wave, read by
        // every peer before the lowest one adds this round's peers
        const uint32_t before = valid ? wh[d] : 0u;
        if (valid && lower == 0) wh[d] = before + (uint32_t)__popcll(peers);
        rank[r] = before + (uint32_t)__popcll(lower);
        dig[r] = d;
    }
    __syncthreads();
    // digit tid: exclusive offsets of the waves, and its total in the tile
    {
        uint32_t run = 0;
        for (int w = 0; w < 4; w++) {
            const uint32_t c = whist[w][tid];
            whist[w][tid] = run;
            run += c;
        }
        uint32_t ctot;
        const uint32_t ci = block_incl_scan_256(run, lds4, &ctot);
        lstart[tid] = ci - run;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        if (wbase + r * 64 + lane < n) {
            const uint32_t lp = lstart[dig[r]] + wh[dig[r]] + rank[r];
            if (lp < (uint32_t)kSortTile) {
                skey[lp] = k[r];
                sval[lp] = v[r];
                sdig[lp] = (uint8_t)dig[r];
            }
        }
    }
    __syncthreads();
    const int cnt = (int)(n - base < kSortTile ? n - base : kSortTile);
    for (int lp = tid; lp < cnt; lp += kSortThreads) {
        const uint64_t key = skey[lp];
        const uint32_t val = sval[lp];
        const uint32_t d = sdig[lp];
        const int64_t o = (int64_t)digit_base[d] + lp - lstart[d];
        if (o >= 0 && o < n) {
            kout[o] = key;
            vout[o] = val;
        }
    }
}

// ------------------------------------------------------- 3b. bucket sort

// Stable passes on the top key bits group the keys by bucket (equal top bits), in
// input order within each bucket: two on the top 16 (bits 47..62) or, where those
// leave large buckets, three on the top 24 (in place of eight on whole keys: builds
// of a Plummer sphere of 131,072 bodies take 155 us, not 217); then
// one block per tile of sorted positions takes the buckets that start in its
// tile (through the end of the last one) and sorts them by the whole key,
// stably: in LDS when they hold at most its capacity of keys, else the last
// bucket apart from the others and, where it alone is beyond the capacity, in
// place in global memory with the other key buffer as scratch. A pass whose
// digit is the same for every key of the range leaves it as it is and is
// skipped. No store changes the top bits at any position, so a block that starts
// late finds its buckets where they were. A stable sort has one result, so this is
// the order of the eight-pass sort.
__host__ __device__ inline int top_shift(int passes) { return 63 - 8 * passes; }
static_assert(63 - 8 * 2 <= 3 * (kMaxLevel - kHintLevel) &&
                  63 - 8 * 3 <= 3 * (kMaxLevel - kBucketLevel3),
              "a bucket inside a cell");
// Block shapes of the bucket sort: a block of T threads holds up to 5 rounds
// of 64 keys per wave (kCap = 5 T) and starts from tiles of kCap - 1024
// keys, so a range never exceeds kCap when no bucket holds more than 1024
// keys. Large sorts use 1024-thread blocks (4096-key tiles), smaller ones
// 256-thread blocks (256-key tiles), so that both give enough blocks.
template <int T>
struct LocalShape {
    static constexpr int kThreads = T;
    static constexpr int kWaves = T / 64;
    static constexpr int kCap = 5 * T;
    static constexpr int kWaveKeys = kCap / kWaves;  // 5 rounds of 64
    static constexpr int kTile = kCap - 1024;
};
using LocalBig = LocalShape<1024>;
using LocalSmall = LocalShape<256>;
static_assert(LocalBig::kTile > 0 && LocalSmall::kTile > 0, "tiles");
constexpr int64_t kBigSortFrom = (int64_t)256 * LocalBig::kTile;  // 256 blocks of the big shape

template <typename Sh>
struct LocalScratch {
    uint32_t whist[Sh::kWaves][256];  // per-wave digit counts, then offsets
    uint32_t base[256];               // where each digit's keys of a chunk start
    uint32_t part[4];                 // wave totals of a 256-entry scan
};

// Exclusive scan of v over threads 0..255 (the first four waves); every
// thread of the block calls it.
__device__ inline uint32_t scan256_excl(uint32_t v, uint32_t *part)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t x = tid < 256 ? v : 0u;
    const uint32_t incl = wave_incl_scan(x);
    if (lane == 63 && wave < 4) part[wave] = incl;
    __syncthreads();
    uint32_t add = 0;
    for (int w = 0; w < 4 && w < wave; w++) add += part[w];
    __syncthreads();  // part is reused by the next call
    return add + incl - x;
}

// One stable counting pass of the block over keys ksrc[0..m) with values
// vsrc into kdst / vdst, on the digit (key >> shift) & 255, in chunks of
// kCap keys taken in order. In a chunk, wave w holds keys w*kWaveKeys .. in
// rounds of 64 and ranks them among equal digits with ballots and a per-wave
// digit count; a key of digit d then goes to base[d] + (keys of d in earlier
// waves) + rank, and base[d] advances by the chunk's count of d. For
// m > kCap, base starts from a count of every digit over all keys.
template <typename Sh, typename KS, typename VS, typename KD, typename VD>
__device__ __forceinline__ void block_radix_pass(KS ksrc, VS vsrc, KD kdst, VD vdst, int64_t m,
                                                 int shift, LocalScratch<Sh> &S)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool multi = m > Sh::kCap;
    if (multi) {
        if (tid < 256) S.base[tid] = 0u;
        __syncthreads();
        for (int64_t i = tid; i < m; i += Sh::kThreads)
            atomicAdd(&S.base[(uint32_t)(ksrc[i] >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t ex = scan256_excl(tid < 256 ? S.base[tid] : 0u, S.part);
        if (tid < 256) S.base[tid] = ex;
        __syncthreads();
    }
    for (int64_t c0 = 0; c0 < m; c0 += Sh::kCap) {
        const int cm = (int)(m - c0 < Sh::kCap ? m - c0 : Sh::kCap);
        for (int i = tid; i < Sh::kWaves * 256; i += Sh::kThreads) (&S.whist[0][0])[i] = 0u;
        __syncthreads();
        uint32_t rank[Sh::kWaveKeys / 64], dig[Sh::kWaveKeys / 64];
#pragma unroll
        for (int r = 0; r < Sh::kWaveKeys / 64; r++) {
            const int i = wave * Sh::kWaveKeys + r * 64 + lane;
            const bool valid = i < cm;
            const uint32_t d = valid ? (uint32_t)(ksrc[c0 + i] >> shift) & 255u : 0u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int bt = 0; bt < 8; bt++) {
                const bool bit = (d >> bt) & 1u;
                const uint64_t bal = __ballot(bit);
                peers &= bit ? bal : ~bal;
            }
            const uint64_t lower = peers & lanemask_lt(lane);
            const uint32_t before = valid ? S.whist[wave][d] : 0u;
            if (valid && lower == 0) S.whist[wave][d] = before + (uint32_t)__popcll(peers);
            rank[r] = before + (uint32_t)__popcll(lower);
            dig[r] = d;
        }
        __syncthreads();
        // digit tid: the offsets of the waves and the chunk's total
        uint32_t run = 0;
        if (tid < 256)
            for (int w = 0; w < Sh::kWaves; w++) {
                const uint32_t c = S.whist[w][tid];
                S.whist[w][tid] = run;
                run += c;
            }
        if (!multi) {
            const uint32_t ex = scan256_excl(run, S.part);
            if (tid < 256) S.base[tid] = ex;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < Sh::kWaveKeys / 64; r++) {
            const int i = wave * Sh::kWaveKeys + r * 64 + lane;
            if (i < cm) {
                const uint32_t o = S.base[dig[r]] + S.whist[wave][dig[r]] + rank[r];
                kdst[o] = ksrc[c0 + i];
                vdst[o] = vsrc[c0 + i];
            }
        }
        __syncthreads();
        if (multi && tid < 256) S.base[tid] += run;
        __syncthreads();
    }
}

template <typename Sh>
__global__ __launch_bounds__(Sh::kThreads) void k_sort_local(uint64_t *__restrict__ keys,
                                                             uint32_t *__restrict__ idx,
                                                             uint64_t *__restrict__ ktmp,
                                                             uint32_t *__restrict__ itmp,
                                                             int64_t n, int shift,
                                                             const int64_t *__restrict__ offsets,
                                                             int ns)
{
    __shared__ LocalScratch<Sh> S;
    __shared__ uint64_t skey[2][Sh::kCap];
    __shared__ uint32_t sval[2][Sh::kCap];
    __shared__ int64_t srange[2];
    __shared__ uint32_t sdiff[2];
    __shared__ uint32_t sbig;  // a bucket of more than kRankMax keys in the range
    __shared__ int64_t soff[kLdsScenes + 1];  // scene starts in sorted order (several scenes)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * Sh::kTile;
    const int64_t t1 = t0 + Sh::kTile < n ? t0 + Sh::kTile : n;
    // Several scenes (at most kLdsScenes): each keeps its caller range of
    // positions, so a bucket also ends where a scene starts.
    if (ns > 1)
        for (int i = tid; i <= ns; i += Sh::kThreads) soff[i] = offsets[i];
    __syncthreads();
    auto next_start = [&](int64_t x) {  // the first scene start at or after x (n past the last)
        if (ns <= 1) return n;
        int lo = 0, hi = ns;  // soff[hi] = n >= x
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (soff[mid] >= x)
                hi = mid;
            else
                lo = mid + 1;
        }
        return soff[lo];
    };
    // wave 0: the first bucket that starts in [t0, t1) (past the one holding
    // key t0 - 1); wave 1: the end of the bucket holding key t1 - 1. Within a
    // scene buckets are in ascending order of their top bits, so each ends at
    // the first key whose top bits differ from the search start's, or at the
    // next scene's start.
    if (wave < 2) {
        const int64_t from = wave == 0 ? t0 : t1;
        int64_t pos = from;
        if (wave == 1 || t0 > 0) {
            const uint64_t top = keys[wave == 0 ? t0 - 1 : t1 - 1] >> shift;
            for (int64_t c = from;; c += 64) {
                const int64_t i = c + lane;
                const bool differs = i >= n || (keys[i] >> shift) != top;
                const uint64_t bal = __ballot(differs);
                if (bal) {
                    pos = c + __builtin_ctzll(bal);
                    break;
                }
            }
            pos = min(pos, next_start(from));
        }
        if (lane == 0) srange[wave] = pos;
    }
    __syncthreads();
    const int64_t ra = srange[0], rb = srange[1];
    if (ra >= t1) return;  // no bucket starts here: the block of its start sorts it
    // the range [ra, rb) one scene, and one piece of it, at a time
    auto sort_range = [&](const int64_t a, const int64_t m) {
        __syncthreads();  // the previous range is done with the LDS
        if (tid < 2) sdiff[tid] = 0u;
        __syncthreads();
        // the key bits that differ somewhere in the range (OR of key ^ first key)
        {
            const uint64_t k0 = keys[a];
            uint64_t d = 0;
            for (int64_t i = tid; i < m; i += Sh::kThreads) d |= keys[a + i] ^ k0;
            for (int o = 32; o > 0; o >>= 1) d |= __shfl_xor(d, o);
            if (lane == 0) {
                atomicOr(&sdiff[0], (uint32_t)d);
                atomicOr(&sdiff[1], (uint32_t)(d >> 32));
            }
        }
        __syncthreads();
        const uint64_t diff = (uint64_t)sdiff[1] << 32 | sdiff[0];
        if (m <= Sh::kCap) {
            for (int i = tid; i < m; i += Sh::kThreads) {
                skey[0][i] = keys[a + i];
                sval[0][i] = idx[a + i];
            }
            if (tid == 0) sbig = 0u;
            __syncthreads();
            // With buckets of at most kRankMax keys (no key has its top bits again
            // kRankMax places on) each key's place is its bucket's start plus the
            // number of keys of the bucket before it in (key, position) order, a
            // stable sort by comparison, with no radix passes. A larger bucket sends
            // the whole range to the radix passes below.
            constexpr int kR = Sh::kCap / Sh::kThreads;
            for (int i = tid; i + kRankMax < m; i += Sh::kThreads)
                if (skey[0][i] >> shift == skey[0][i + kRankMax] >> shift) sbig = 1u;
            __syncthreads();
            const bool by_rank = sbig == 0u;  // the same on every thread
            int32_t dest[kR];
#pragma unroll
            for (int r = 0; r < kR; r++) {
                const int i = tid + r * Sh::kThreads;
                dest[r] = -1;
                if (!by_rank || i >= m) continue;
                const uint64_t k = skey[0][i];
                const uint64_t top = k >> shift;
                int bs = i, be = i + 1;
                while (bs > 0 && (skey[0][bs - 1] >> shift) == top) bs--;
                while (be < m && (skey[0][be] >> shift) == top) be++;
                int32_t rank = bs;
                for (int j = bs; j < be; j++) {
                    const uint64_t kj = skey[0][j];
                    rank += kj < k || (kj == k && j < i);
                }
                dest[r] = rank;
            }
            if (by_rank) {
#pragma unroll
                for (int r = 0; r < kR; r++) {
                    const int i = tid + r * Sh::kThreads;
                    if (i < m) {
                        keys[a + dest[r]] = skey[0][i];
                        idx[a + dest[r]] = sval[0][i];
                    }
                }
                return;
            }
            int src = 0;
            for (int pass = 0; pass < 8; pass++) {
                if (((diff >> (8 * pass)) & 255u) == 0) continue;  // the same on every thread
                block_radix_pass<Sh>(skey[src], sval[src], skey[src ^ 1], sval[src ^ 1], m, 8 * pass,
                                     S);
                src ^= 1;
            }
            for (int i = tid; i < m; i += Sh::kThreads) {
                keys[a + i] = skey[src][i];
                idx[a + i] = sval[src][i];
            }
        } else {
            // buffers alternate between the keys and the scratch; an odd number
            // of passes ends with a copy back
            bool in_keys = true;
            for (int pass = 0; pass < 8; pass++) {
                if (((diff >> (8 * pass)) & 255u) == 0) continue;
                if (in_keys)
                    block_radix_pass<Sh>(keys + a, idx + a, ktmp + a, itmp + a, m, 8 * pass, S);
                else
                    block_radix_pass<Sh>(ktmp + a, itmp + a, keys + a, idx + a, m, 8 * pass, S);
                in_keys = !in_keys;
            }
            if (!in_keys) {
                for (int64_t i = tid; i < m; i += Sh::kThreads) {
                    keys[a + i] = ktmp[a + i];
                    idx[a + i] = itmp[a + i];
                }
            }
        }
    };
    // (of a range beyond the LDS only the last bucket, which alone leaves the tile,
    // goes through global memory: see piece_end)
    for (int64_t sa = ra; sa < rb;) {
        const int64_t sb = min(rb, next_start(sa + 1));
        const int64_t pe = piece_end(keys, sa, sb, Sh::kCap, shift);
        sort_range(sa, pe - sa);
        sa = pe;
    }
}

#ifdef BHX_CHECKS
// The checked build's verification of a one-scene sort: keys in order and
// every index inside the array.
__global__ __launch_bounds__(256) void k_check_order(const uint64_t *__restrict__ keys,
                                                     const uint32_t *__restrict__ idx, int64_t n,
                                                     const int64_t *__restrict__ offsets, int ns)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    BHX_CHECK(idx[i] < n, CK_INDEX);
    if (i == 0 || keys[i - 1] <= keys[i]) return;
    // a descent is in order only where a scene starts
    bool start = false;
    if (ns > 1) {
        int lo = 0, hi = ns;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (offsets[mid] >= i)
                hi = mid;
            else
                lo = mid + 1;
        }
        start = offsets[lo] == i;
    }
    BHX_CHECK(start, CK_ORDER);
}
#endif

// ------------------------------------------------------------- 4. gather

// With mark: the first sorted body of each non-empty level-kPrefixLevels
// cell, where the cell part of the key changes (one writer per cell), for
// k_prefix_levels.
__device__ inline void prefix_mark(const uint64_t *__restrict__ keys, int64_t s,
                                   int32_t *__restrict__ mark)
{
    const uint32_t c = (uint32_t)(keys[s] >> kPrefixShift);
    if (s == 0 || (uint32_t)(keys[s - 1] >> kPrefixShift) != c) mark[c] = (int32_t)s;
}

__global__ __launch_bounds__(256) void k_gather(const double *__restrict__ pos,
                                                const double *__restrict__ mass,
                                                const double *__restrict__ eps,
                                                const uint32_t *__restrict__ idx, int64_t n,
                                                Body *__restrict__ body,
                                                double *__restrict__ beps2,
                                                const uint64_t *__restrict__ keys,
                                                int32_t *__restrict__ mark)
{
    int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    if (mark) prefix_mark(keys, s, mark);
    uint32_t i = idx[s];
    if (!check_ok(i < n, CK_INDEX)) i = 0;
    body[s] = Body{pos[3 * (int64_t)i], pos[3 * (int64_t)i + 1], pos[3 * (int64_t)i + 2], mass[i]};
    if (eps) {
        double e = eps[i];
        beps2[s] = e * e;
    }
}

// The state of a multi-step call into the new order: idx holds the S index
// of each sorted body on entry and its caller index on return.
__global__ __launch_bounds__(256) void k_gather_state(const Body *__restrict__ sbody,
                                                      const double *__restrict__ svel,
                                                      const double *__restrict__ seps2,
                                                      const uint32_t *__restrict__ scidx,
                                                      int64_t n, uint32_t *__restrict__ idx,
                                                      Body *__restrict__ body,
                                                      double *__restrict__ tvel,
                                                      double *__restrict__ beps2,
                                                      const uint64_t *__restrict__ keys,
                                                      int32_t *__restrict__ mark)
{
    int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    if (mark) prefix_mark(keys, s, mark);
    int64_t p = idx[s];
    if (!check_ok(p < n, CK_INDEX)) p = 0;
    body[s] = sbody[p];
    for (int a = 0; a < 3; a++) tvel[3 * s + a] = svel[3 * p + a];
    if (seps2) beps2[s] = seps2[p];
    idx[s] = scidx[p];
}

// -------------------------------------------------------------- 5. build

// First node and node count of `level`, clamped to the node table: after an
// overflow (flagged ST_CAPACITY) a level counter can exceed what was written.
__device__ inline void level_range(const int32_t *counts, int level, int64_t node_cap,
                                   int32_t *beg, int32_t *cnt)
{
    int64_t b = 0;
    for (int l = 0; l < level; l++) {
        int64_t c = counts[l];
        b += c < node_cap - b ? c : node_cap - b;
    }
    int64_t c = counts[level];
    *beg = (int32_t)b;
    *cnt = (int32_t)(c < node_cap - b ? c : node_cap - b);
}

// Splits every node of `level` holding more than `leaf` bodies, eight lanes
// per node (one chunk: blockDim / 8 nodes): lane o finds the first body of
// octant o, and the non-empty children are written contiguously in octant
// order. A step of the block takes one chunk of nodes; or, `compact` (levels
// where most nodes are leaves), one node per thread, of which the ones that
// split are listed in LDS and split chunk by chunk, so that a leaf costs one
// load. All nodes of a chunk reserve their children with a single atomic on
// the next level's count (scans over the wave and over the block's waves give
// each node its offset): one atomic per node or per wave serialises on that
// counter. Must be called by every thread of the block (a multiple of 64
// threads, at most 1024); every thread runs the same loop iterations.
// `counts` is the per-level node count array: the tree header's, or a copy
// in LDS that a single-block kernel keeps and writes back. The block's steps
// start at nodes b_first + j stride, j = 0, 1, ... (b_first = block index x
// nodes per step; stride = that times the number of blocks).
// Nodes of at most this many bodies find their octant ranges by counting
// (each octant's count fits a byte), larger ones by binary search.
constexpr int32_t kLinearSplit = 64;

template <bool compact>
__device__ inline void build_nodes(int level, const uint64_t *__restrict__ keys, int32_t *counts,
                                   uint32_t *status, int32_t *cell_max,
                                   NodeInfo *__restrict__ ninfo, int64_t node_cap, int leaf,
                                   int64_t b_first, int64_t stride)
{
    __shared__ uint32_t s_wtot[16];
    __shared__ int32_t s_base;
    __shared__ int32_t s_cmax;
    __shared__ int32_t s_list[compact ? 1024 : 1];  // the step's nodes that split
    int32_t beg, cnt;
    level_range(counts, level, node_cap, &beg, &cnt);
    const int32_t next_beg = beg + cnt;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int o = threadIdx.x & 7, gl = lane & ~7;
    const int shift = 60 - 3 * level;  // bits of the child octant at level + 1
    // the block's largest node, merged into cell_max once
    int32_t cmax = 0;
    if (threadIdx.x == 0) s_cmax = 0;
    const uint32_t chunk = blockDim.x >> 3;
    for (int64_t b0 = b_first; b0 < cnt; b0 += stride) {
        uint32_t nlist;  // nodes of the step to give eight lanes each
        if constexpr (compact) {
            // one node per thread: list the ones that split
            const int64_t g = b0 + threadIdx.x;
            bool splits = false;
            if (g < cnt) {
                const int32_t c = ninfo[beg + (int32_t)g].count;
                splits = c > leaf && level < kMaxLevel;
                cmax = max(cmax, c);
            }
            const uint64_t sb = __ballot(splits);
            if (lane == 0) s_wtot[wave] = (uint32_t)__popcll(sb);
            __syncthreads();
            uint32_t lbefore = 0;
            nlist = 0;
            for (int w = 0; w < nwaves; w++) {
                const uint32_t t = s_wtot[w];
                if (w < wave) lbefore += t;
                nlist += t;
            }
            if (splits) s_list[lbefore + lanes_below(sb)] = beg + (int32_t)g;
            __syncthreads();  // the list is complete and s_wtot free again
        } else {
            nlist = (uint32_t)min((int64_t)chunk, cnt - b0);
        }
        for (uint32_t c0 = 0; c0 < nlist; c0 += chunk) {
            const uint32_t gi = c0 + (threadIdx.x >> 3);
            const bool live = gi < nlist;
            const uint32_t gl_node = live ? gi : c0;
            int32_t k;
            if constexpr (compact)
                k = s_list[gl_node];
            else
                k = beg + (int32_t)(b0 + gl_node);
            const NodeInfo info = ninfo[k];
            if (!compact && live) cmax = max(cmax, info.count);
            const bool split = live && info.count > leaf && level < kMaxLevel;
            int32_t start;
            if (info.count <= kLinearSplit) {
                // few bodies: the 8 lanes read them all (independent loads) and
                // count them per octant, one byte per octant, summed over the
                // group; octant o starts after the bodies of octants below it
                uint64_t hist = 0;
                if (split)
                    for (int32_t j = o; j < info.count; j += 8)
                        hist += 1ull << (8 * (int)((keys[info.first + j] >> shift) & 7ull));
                hist += __shfl_xor(hist, 1, 8);
                hist += __shfl_xor(hist, 2, 8);
                hist += __shfl_xor(hist, 4, 8);
                const uint64_t below = o == 0 ? 0ull : hist & (~0ull >> (64 - 8 * o));
                start = info.first + (split ? (int32_t)((below * 0x0101010101010101ull) >> 56) : 0);
            } else {
                int32_t a = info.first, b = split ? info.first + info.count : info.first;
                while (a < b) {
                    int32_t m = (a + b) >> 1;
                    if ((int)((keys[m] >> shift) & 7ull) < o)
                        a = m + 1;
                    else
                        b = m;
                }
                start = a;
            }
            int32_t end = __shfl_down(start, 1, 8);
            if (o == 7) end = info.first + info.count;
            BHX_CHECK(!split || (start >= info.first && start <= end &&
                                 end <= info.first + info.count),
                      CK_PARTITION);
            const bool nonempty = split && end > start;
            const uint32_t gm = (uint32_t)(__ballot(nonempty) >> gl) & 0xffu;
            const int nch = __popc(gm);
            const int rank = __popc(gm & ((1u << o) - 1u));
            const uint32_t mine = o == 0 ? (uint32_t)nch : 0u;
            const uint32_t incl = wave_incl_scan(mine);
            if (lane == 63) s_wtot[wave] = incl;
            __syncthreads();
            uint32_t before = 0, btot = 0;
            for (int w = 0; w < nwaves; w++) {
                const uint32_t t = s_wtot[w];
                if (w < wave) before += t;
                btot += t;
            }
            if (threadIdx.x == 0 && btot > 0)
                s_base = atomicAdd(&counts[level + 1], (int32_t)btot);
            __syncthreads();
            const int32_t base = btot > 0 ? s_base : 0;
            const int32_t slot =
                base + (int32_t)(before + __shfl(incl, gl) - __shfl(mine, gl));
            __syncthreads();  // s_wtot and s_base are rewritten by the next chunk
            if (!split) continue;
            const int64_t cfirst = (int64_t)next_beg + slot;
            const int32_t scene_bits = info.lvl_nch & (int32_t)0xffff0000;
            // (counted nodes are written although an overflow leaves them unlinked)
            if (nonempty && cfirst + rank < node_cap)
                ninfo[cfirst + rank] = NodeInfo{start, end - start, -1, (level + 1) | scene_bits};
            if (cfirst + nch > node_cap) {
                if (o == 0) flag_status(status, ST_CAPACITY);
                continue;
            }
            if (o == 0) {
                ninfo[k].child0 = (int32_t)cfirst;
                ninfo[k].lvl_nch = level | (nch << 8) | scene_bits;
            }
        }
        if constexpr (compact) __syncthreads();  // s_list is rewritten by the next step
    }
    for (int off = 32; off > 0; off >>= 1) cmax = max(cmax, __shfl_xor(cmax, off));
    __syncthreads();
    if (lane == 0 && cmax > 0) atomicMax(&s_cmax, cmax);
    __syncthreads();
    if (threadIdx.x == 0 && s_cmax > 0) atomicMax(cell_max, s_cmax);
}

template <bool compact>
__global__ __launch_bounds__(1024) void k_build_level(int level, const uint64_t *__restrict__ keys,
                                                      TreeHeader *__restrict__ hdr,
                                                      NodeInfo *__restrict__ ninfo,
                                                      int64_t node_cap, int leaf)
{
    const int64_t per_step = compact ? blockDim.x : blockDim.x >> 3;  // nodes per block step
    build_nodes<compact>(level, keys, hdr->level_count, hdr->status, &hdr->cell_max[level], ninfo,
                         node_cap, leaf, (int64_t)blockIdx.x * per_step,
                         (int64_t)gridDim.x * per_step);
}

// Levels from..upto-1 in one block, on a copy of the node counts in LDS
// (no other kernel runs meanwhile); stops at the first empty level.
template <bool compact>
__device__ inline void build_levels_block(int from, int upto, const uint64_t *__restrict__ keys,
                                          TreeHeader *__restrict__ hdr,
                                          NodeInfo *__restrict__ ninfo, int64_t node_cap,
                                          int leaf, int32_t *scnt)
{
    for (int level = from; level < upto; level++) {
        if (scnt[level] == 0) break;
        build_nodes<compact>(level, keys, scnt, hdr->status, &hdr->cell_max[level], ninfo, node_cap, leaf,
                             0, compact ? blockDim.x : blockDim.x >> 3);
        __syncthreads();
    }
}

// The top levels of a single scene, from the sorted keys. A level-l cell
// holds the bodies whose keys start with its 3 l bits, a contiguous run of
// the sorted keys, so the first body of every level-kPrefixLevels cell
// gives the body range of every cell on levels 1..kPrefixLevels. A cell is a
// node iff it holds a body and its parent holds more than `leaf` (then every
// ancestor does too and splits), and a node's children are its non-empty
// octants: the nodes the level-by-level split creates, numbered here in
// Morton order within each level, with no searches and no atomics.

// Exclusive prefix sums of K values at once over the 1024 threads of a block,
// with their totals; every thread calls it. s_w: LDS [16][K].
template <int K>
__device__ inline void block_excl_scan_1024(uint32_t (&v)[K], uint32_t (&tot)[K],
                                            uint32_t (*s_w)[K])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl[K];
#pragma unroll
    for (int k = 0; k < K; k++) incl[k] = wave_incl_scan(v[k]);
    if (lane == 63)
        for (int k = 0; k < K; k++) s_w[wave][k] = incl[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; k++) {
        uint32_t before = 0, t = 0;
#pragma unroll
        for (int w = 0; w < 16; w++) {  // independent LDS reads, all in flight
            const uint32_t x = s_w[w][k];
            if (w < wave) before += x;
            t += x;
        }
        v[k] = before + incl[k] - v[k];
        tot[k] = t;
    }
    __syncthreads();  // s_w may be reused
}

// Levels 1..kPrefixLevels of one scene of n > 0 sorted bodies (the root,
// node 0, written by k_box_final): one block of 1024 threads. Reads the marks
// the gather wrote (restoring them to "none"), turns them into the first
// body of every level-5 cell (held in LDS, one pad word after every 32 so
// that a thread's 32 consecutive cells fall in distinct banks), and writes
// the nodes of levels 1..5 (those of level 5 unsplit, for the level-5 split),
// the children of the root and of levels 1..4, and the node counts of levels
// 1..5. Thread t decides level-5 cells 32 t..32 t + 31, level-4 cells
// 4 t..4 t + 3 and cell t of levels 1..3; the level-4 and level-5 nodes are
// then written with consecutive lanes on consecutive cells, so that the
// stores of a wave fall on consecutive nodes.
static_assert(kPrefixLevels == 5 && kPrefixCells == 32 * 1024, "one block, 32 cells a thread");
__device__ inline int prefix_pad(int c) { return c + (c >> 5); }
__global__ __launch_bounds__(1024) void k_prefix_levels(int32_t *__restrict__ mark, int64_t n,
                                                        TreeHeader *__restrict__ hdr,
                                                        NodeInfo *__restrict__ ninfo,
                                                        int64_t node_cap, int leaf)
{
    __shared__ int32_t s_st[kPrefixCells + kPrefixCells / 32 + 1];  // first body per cell, padded
    __shared__ int32_t s_wmin[16];
    __shared__ uint32_t s_w[16][5];
    __shared__ uint32_t s_r2[64], s_r3[512];  // ranks of the level-2 and level-3 cells
    __shared__ uint32_t s_r4[1024], s_m4[1024], s_r5[1024], s_m5[1024];  // per thread
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int32_t nn = (int32_t)n;
    // 1. the marks (all loads in flight at once), restored to "none"
    {
        int32_t mv[kPrefixCells / 1024];
#pragma unroll
        for (int k = 0; k < kPrefixCells / 1024; k++) mv[k] = mark[t + 1024 * k];
#pragma unroll
        for (int k = 0; k < kPrefixCells / 1024; k++) {
            s_st[prefix_pad(t + 1024 * k)] = mv[k];
            mark[t + 1024 * k] = INT32_MAX;
        }
    }
    if (t == 0) s_st[prefix_pad(kPrefixCells)] = nn;
    __syncthreads();
    // 2. first body of every cell = the smallest mark at or after it (n past
    // the last): a suffix minimum over the thread's cells and the threads
    // after. With it, this thread's level-4 cells that hold bodies (nz4) and
    // its level-5 cells that hold bodies under a level-4 cell that splits (m5).
    const int c0 = 32 * t;
    uint32_t nz4 = 0, m5 = 0;
    {
        int32_t st[33];
#pragma unroll
        for (int j = 0; j < 32; j++) st[j] = s_st[prefix_pad(c0 + j)];
        int32_t lm = st[0];
#pragma unroll
        for (int j = 1; j < 32; j++) lm = min(lm, st[j]);
        int32_t x = lm;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_down(x, o);
            if (lane + o < 64) x = min(x, y);
        }
        int32_t carry = __shfl_down(x, 1);
        if (lane == 63) carry = INT32_MAX;
        if (lane == 0) s_wmin[wave] = x;
        __syncthreads();
        carry = min(carry, nn);
#pragma unroll
        for (int w = 0; w < 16; w++)
            if (w > wave) carry = min(carry, s_wmin[w]);
        st[32] = carry;
#pragma unroll
        for (int j = 31; j >= 0; j--) st[j] = min(st[j], st[j + 1]);
        BHX_CHECK(st[0] >= 0, CK_PARTITION);
#pragma unroll
        for (int j = 0; j < 32; j++) s_st[prefix_pad(c0 + j)] = st[j];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int32_t c4 = st[8 * q + 8] - st[8 * q];
            if (c4 > 0) nz4 |= 1u << q;
            if (c4 > leaf)
#pragma unroll
                for (int j = 8 * q; j < 8 * q + 8; j++)
                    if (st[j + 1] > st[j]) m5 |= 1u << j;
        }
    }
    __syncthreads();
    auto S = [&](int c) { return s_st[prefix_pad(c)]; };  // first body of level-5 cell c
    auto cnt = [&](int l, int c) {  // bodies of level-l cell c
        const int sh = 3 * (5 - l);
        return S((c + 1) << sh) - S(c << sh);
    };
    // 3. which cells are nodes, level by level
    const bool e1 = t < 8 && cnt(1, t) > 0 && nn > leaf;
    const bool e2 = t < 64 && cnt(2, t) > 0 && cnt(1, t >> 3) > leaf;
    const bool e3 = t < 512 && cnt(3, t) > 0 && cnt(2, t >> 3) > leaf;
    const uint32_t m4 = cnt(3, t >> 1) > leaf ? nz4 : 0u;  // under a level-3 cell that splits
    uint32_t r[5] = {e1 ? 1u : 0u, e2 ? 1u : 0u, e3 ? 1u : 0u, (uint32_t)__popc(m4),
                     (uint32_t)__popc(m5)};
    uint32_t tot[5];
    block_excl_scan_1024<5>(r, tot, s_w);
    if (t < 64) s_r2[t] = r[1];
    if (t < 512) s_r3[t] = r[2];
    s_r4[t] = r[3];
    s_m4[t] = m4;
    s_r5[t] = r[4];
    s_m5[t] = m5;
    __syncthreads();
    // 4. the nodes: level l starts after the nodes of the levels above
    const int64_t beg1 = 1, beg2 = beg1 + tot[0], beg3 = beg2 + tot[1], beg4 = beg3 + tot[2],
                  beg5 = beg4 + tot[3];
    if (beg5 + tot[4] > node_cap) {
        if (t == 0) flag_status(hdr->status, ST_CAPACITY);
        return;  // the same on every thread
    }
    auto nonempty8 = [&](int l, int c) {  // non-empty children of level-l cell c, l <= 4
        int k = 0;
        for (int o = 0; o < 8; o++) k += cnt(l + 1, 8 * c + o) > 0;
        return k;
    };
    if (t == 0) {
        for (int l = 1; l <= 5; l++) hdr->level_count[l] = (int32_t)tot[l - 1];
        if (nn > leaf) {
            ninfo[0].child0 = (int32_t)beg1;
            ninfo[0].lvl_nch = nonempty8(0, 0) << 8;
        }
    }
    // levels 1..3: cell t; its first child's rank is that of the first cell
    // of its eight on the next level
    auto upper = [&](int l, bool exists, uint32_t rank, int64_t beg, int64_t beg_next,
                     const uint32_t *rnext, int rsel) {
        if (!exists) return;
        const int32_t c = cnt(l, t);
        NodeInfo ni{S(t << (3 * (5 - l))), c, -1, l};
        if (c > leaf) {
            ni.child0 = (int32_t)(beg_next + rnext[rsel]);
            ni.lvl_nch = l | (nonempty8(l, t) << 8);
        }
        ninfo[beg + rank] = ni;
    };
    upper(1, e1, r[0], beg1, beg2, s_r2, 8 * t);
    upper(2, e2, r[1], beg2, beg3, s_r3, 8 * t);
    upper(3, e3, r[2], beg3, beg4, s_r4, 2 * t);  // level-4 cell 8 t is thread 2 t's first
    // level 4, cell c4 = 1024 k + t (owner thread c4 / 4)
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int c4 = 1024 * k + t, o = c4 >> 2, q = c4 & 3;
        const uint32_t mo = s_m4[o];
        if (!((mo >> q) & 1u)) continue;
        const int32_t first = S(c4 << 3), c = S((c4 + 1) << 3) - first;
        NodeInfo ni{first, c, -1, 4};
        if (c > leaf) {
            const uint32_t m5o = s_m5[o];  // the owner of its children too
            ni.child0 = (int32_t)(beg5 + s_r5[o] + __popc(m5o & ((1u << (8 * q)) - 1u)));
            ni.lvl_nch = 4 | (__popc((m5o >> (8 * q)) & 0xffu) << 8);
        }
        ninfo[beg4 + s_r4[o] + __popc(mo & ((1u << q) - 1u))] = ni;
    }
    // level 5, cell c = 1024 k + t (owner thread c / 32)
#pragma unroll 4
    for (int k = 0; k < 32; k++) {
        const int c = 1024 * k + t, o = c >> 5, j = c & 31;
        const uint32_t m5o = s_m5[o];
        if (!((m5o >> j) & 1u)) continue;
        const int32_t first = S(c);
        ninfo[beg5 + s_r5[o] + __popc(m5o & ((1u << j) - 1u))] =
            NodeInfo{first, S(c + 1) - first, -1, 5};
    }
}

// ------------------------------------------------------------ 6. moments

// The sums of a node's mass, centre of mass and mass-weighted softening over
// its bodies or its children, in member order, by eq. (COMinternal). Products
// and sums are rounded as written; each group's loads are all issued before its
// first addition.
struct MomentSum {
    double ms = 0.0, mx = 0.0, my = 0.0, mz = 0.0, me = 0.0;

    __device__ inline void add(double x, double y, double z, double m, double e, bool use_eps)
    {
#pragma clang fp contract(off)
        ms += m;
        mx += x * m;
        my += y * m;
        mz += z * m;
        if (use_eps) me += e * m;
    }
    __device__ inline void leaf(const Body *__restrict__ body, const double *__restrict__ beps2,
                                const NodeInfo &info, bool use_eps)
    {
        const int32_t end = info.first + info.count;
        for (int32_t s0 = info.first; s0 < end; s0 += 4) {
            Body b[4];
            double e[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int32_t s = s0 + u < end ? s0 + u : s0;
                b[u] = body[s];
                e[u] = use_eps ? beps2[s] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (s0 + u >= end) break;
                add(b[u].x, b[u].y, b[u].z, b[u].m, e[u], use_eps);
            }
        }
    }
    // G children are loaded at a time (8 from global memory, whose latency
    // counts; fewer from LDS, where registers do)
    template <int G = 8>
    __device__ inline void children(const NodeMom *nmom, const double *neps2, const NodeInfo &info,
                                    bool use_eps)
    {
        const int nch = node_nchild(info);
#pragma unroll
        for (int u0 = 0; u0 < 8; u0 += G) {
            if (u0 >= nch) break;
            NodeMom cm[G];
            double e[G];
#pragma unroll
            for (int u = 0; u < G; u++) {
                const int32_t c = info.child0 + (u0 + u < nch ? u0 + u : 0);
                cm[u] = nmom[c];
                e[u] = use_eps ? neps2[c] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < G; u++) {
                if (u0 + u >= nch) break;
                add(cm[u].x, cm[u].y, cm[u].z, cm[u].m, e[u], use_eps);
            }
        }
    }
    // The node's moments and mean eps^2; a massless cell has its centre.
    __device__ inline NodeMom moments(int level, int32_t first, const uint64_t *__restrict__ keys,
                                      const SceneBox &b, bool use_eps, double &e2) const
    {
#pragma clang fp contract(off)
        e2 = 0.0;
        if (ms > 0.0) {
            if (use_eps) e2 = me / ms;
            return NodeMom{mx / ms, my / ms, mz / ms, ms};
        }
        const uint64_t key = keys[first];
        const int sh = kMaxLevel - level;
        const double s = ldexp(b.L, -level);
        return NodeMom{b.x0[0] + ((double)(compact3(key >> 2) >> sh) + 0.5) * s,
                       b.x0[1] + ((double)(compact3(key >> 1) >> sh) + 0.5) * s,
                       b.x0[2] + ((double)(compact3(key) >> sh) + 0.5) * s, 0.0};
    }
};

// A node's moments, mean eps^2 and (QUAD) quadrupole: of an internal node
// from its children in cmom (G loaded at a time), ceps2 and cquad, of a leaf from its
// bodies.
template <bool QUAD, int G = 8>
__device__ inline NodeMom node_sums(const NodeInfo &info, int level, const Body *__restrict__ body,
                                    const double *__restrict__ beps2,
                                    const uint64_t *__restrict__ keys,
                                    const SceneBox *__restrict__ box, const NodeMom *cmom,
                                    const double *ceps2, const double *cquad, int use_eps,
                                    double &e2, double *q)
{
#pragma clang fp contract(off)
    MomentSum sum;
    if (info.child0 < 0)
        sum.leaf(body, beps2, info, use_eps);
    else
        sum.children<G>(cmom, ceps2, info, use_eps);
    const NodeMom out = sum.moments(level, info.first, keys, box[node_scene(info)], use_eps, e2);
    if constexpr (!QUAD) return out;
    // traceless quadrupole about the centre of mass: from the bodies of a leaf,
    // from the children by the parallel-axis shift
    for (int a = 0; a < 6; a++) q[a] = 0.0;
    auto add = [&](double dx, double dy, double dz, double m) {
        const double d2 = dx * dx + dy * dy + dz * dz;
        q[0] += m * (3.0 * dx * dx - d2);
        q[1] += m * (3.0 * dy * dy - d2);
        q[2] += m * (3.0 * dz * dz - d2);
        q[3] += m * 3.0 * dx * dy;
        q[4] += m * 3.0 * dx * dz;
        q[5] += m * 3.0 * dy * dz;
    };
    if (info.child0 < 0) {
        const int32_t end = info.first + info.count;
        for (int32_t s0 = info.first; s0 < end; s0 += 4) {
            Body b[4];
#pragma unroll
            for (int u = 0; u < 4; u++) b[u] = body[s0 + u < end ? s0 + u : s0];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (s0 + u >= end) break;
                add(b[u].x - out.x, b[u].y - out.y, b[u].z - out.z, b[u].m);
            }
        }
    } else {
        // (one child at a time: two or four are 1 to 3 % slower at 20,000 bodies)
        const int nch = node_nchild(info);
        for (int64_t c = info.child0; c < info.child0 + nch; c++) {
            const NodeMom cm = cmom[c];
            for (int a = 0; a < 6; a++) q[a] += cquad[6 * c + a];
            add(cm.x - out.x, cm.y - out.y, cm.z - out.z, cm.m);
        }
    }
    return out;
}

// The same for node k of the node table.
template <bool QUAD, int G = 8>
__device__ inline void node_moments(int32_t k, const NodeInfo &info, int level,
                                    const Body *__restrict__ body,
                                    const double *__restrict__ beps2,
                                    const uint64_t *__restrict__ keys,
                                    const SceneBox *__restrict__ box, NodeMom *nmom, double *neps2,
                                    double *nquad, int use_eps)
{
    double e2, q[6];
    nmom[k] = node_sums<QUAD, G>(info, level, body, beps2, keys, box, nmom, neps2, nquad, use_eps,
                                 e2, q);
    if (use_eps) neps2[k] = e2;
    if constexpr (QUAD)
        for (int a = 0; a < 6; a++) nquad[6 * (int64_t)k + a] = q[a];
}

// The moments of every node of `level`.
template <bool QUAD>
__device__ inline void moments_nodes(int level, const int32_t *counts,
                                     const NodeInfo *__restrict__ ninfo,
                                     const Body *__restrict__ body,
                                     const double *__restrict__ beps2,
                                     const uint64_t *__restrict__ keys,
                                     const SceneBox *__restrict__ box, NodeMom *__restrict__ nmom,
                                     double *__restrict__ neps2, double *__restrict__ nquad,
                                     int64_t node_cap, int use_eps, int64_t g_first,
                                     int64_t stride)
{
    int32_t beg, cnt;
    level_range(counts, level, node_cap, &beg, &cnt);
    for (int64_t g = g_first; g < cnt; g += stride) {
        const int32_t k = beg + (int32_t)g;
        node_moments<QUAD>(k, ninfo[k], level, body, beps2, keys, box, nmom, neps2, nquad, use_eps);
    }
}

// --------------------------------------------------------- 5 and 6, subtrees

// max in place; most calls find a value that is already as large.
__device__ inline void raise_max(int32_t *p, int32_t v)
{
    if (v > *(const volatile int32_t *)p) atomicMax(p, v);
}

// Everything below level `level0`, whose nodes exist: each block takes
// kSubNodes of them at a time, splits their subtrees level by level and forms
// the moments of all their nodes bottom-up, so that the levels from level0 down
// take one launch whatever their depth instead of two each. Bound by latency (a
// block's dependent loads, two barriers a step and the atomic on the node count
// that all blocks share): at 2^20 bodies and leaf 4 it takes 66 us where the
// launches of those levels and their moments took 130, at 50,000 (leaf 8) 10
// instead of 24; steps of 40,000 to 2^20 bodies are 1 to 5 % shorter. 256 threads
// a block are 1 % slower at 2^20 (more atomics), 1024 the same. The
// launches above stop at the first level whose nodes held at most kSubBodies
// bodies in the previous build, which keeps a block's work even; any node is
// handled, a larger one more slowly.
//
// A step splits 64 nodes, eight lanes each as in build_nodes, with one atomic for
// the numbers of all their children: nodes below level0 are numbered as they
// are made, level0's follow by level. A child that is a leaf gets its moments at
// once; one that splits goes on the block's list, which holds the splitting
// nodes in level order and is walked backwards for their moments. The list is in
// LDS and, beyond kSubList entries, in `inner`, of which the block then reserves
// what its subtrees can need (subtree_splits; in all at most the buffer, see
// kInnerWords).
constexpr int kSubThreads = 512;
constexpr int kSubNodes = kSubThreads / 8;
// (kSubBodies: with 1024 bodies 64 uneven scenes take 15 % longer a step, with 64 2^20 bodies 4 %)
constexpr int kSubList = 2048;
template <bool QUAD>
__global__ __launch_bounds__(kSubThreads) void k_build_subtrees(
    int level0, const uint64_t *__restrict__ keys, TreeHeader *__restrict__ hdr, NodeInfo *ninfo,
    int64_t node_cap, int leaf, const Body *__restrict__ body, const double *__restrict__ beps2,
    const SceneBox *__restrict__ box, NodeMom *nmom, double *neps2, double *nquad, int use_eps,
    int32_t *inner, int64_t inner_words)
{
    static_assert(kSubNodes <= 64, "one wave lists the subtrees' roots");
    static_assert(sizeof(hdr->inner_top) == 8 && sizeof(hdr->deep_count) == 8,
                  "totals of 2^30 bodies exceed 32 bits");
    constexpr int W = kSubThreads / 64;
    __shared__ int32_t list[kSubList];
    // first list entry per level, from level0 (entries are nodes, of which there are
    // less than 2^31)
    __shared__ int32_t lbeg[kLevels + 2];
    __shared__ int32_t made[kLevels + 1];     // nodes made per level
    __shared__ uint32_t s_wtot[2][W], s_wdeep[2][W];
    __shared__ int64_t s_base[2], s_inner, s_need;  // s_inner: kNotYet, or the reserved words' first
    __shared__ int32_t s_hint;
    constexpr int64_t kNotYet = -1, kNoRoom = -2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int o = tid & 7, gl = lane & ~7;
    int32_t beg, cnt;
    level_range(hdr->level_count, level0, node_cap, &beg, &cnt);
    const int32_t deep0 = beg + cnt;
    if (tid <= kLevels) made[tid] = 0;
    if (tid == 0) s_hint = 0;
    auto entry = [&](int i) { return i < kSubList ? list[i] : inner[s_inner + i - kSubNodes]; };
    for (int64_t g0 = (int64_t)blockIdx.x * kSubNodes; g0 < cnt;
         g0 += (int64_t)gridDim.x * kSubNodes) {
        __syncthreads();  // the previous chunk's list is read no more
        if (wave == 0) {
            const bool mine = lane < kSubNodes && g0 + lane < cnt;
            const int32_t k = beg + (int32_t)g0 + lane;
            NodeInfo info{0, 0, -1, 0};
            if (mine) info = ninfo[k];
            const bool split = info.count > leaf && level0 < kMaxLevel;
            const uint64_t sb = __ballot(split);
            if (split) list[lanes_below(sb)] = k;
            int32_t bodies = split ? info.count : 0, most = info.count;
            for (int off = 32; off > 0; off >>= 1) {
                bodies += __shfl_xor(bodies, off);
                most = max(most, __shfl_xor(most, off));
            }
            if (lane == 0) {
                lbeg[0] = 0;
                lbeg[1] = __popcll(sb);
                s_inner = kNotYet;
                s_need = subtree_splits(level0, bodies, leaf);
                raise_max(&hdr->cell_max[level0], most);
            }
            if (mine && !split)
                node_moments<QUAD, 4>(k, info, level0, body, beps2, keys, box, nmom, neps2, nquad, use_eps);
        }
        __syncthreads();
        int d = 0, hi = lbeg[1], par = 0;
        for (int lo = 0; lo < hi; d++) {  // the list entries of level level0 + d
            const int level = level0 + d, shift = 60 - 3 * level;
            int top = hi;        // end of the list
            int32_t total = 0;   // children of this level's nodes
            for (int f0 = lo; f0 < hi; f0 += kSubThreads / 8, par ^= 1) {
                const int gi = f0 + (tid >> 3);
                const bool live = gi < hi;
                const int32_t id = entry(live ? gi : f0);
                const NodeInfo info = ninfo[id];
                const int32_t count = live ? info.count : 0;
                int32_t start;
                if (info.count <= kLinearSplit) {
                    uint64_t hist = 0;  // one byte per octant
                    for (int32_t j = o; j < count; j += 8)
                        hist += 1ull << (8 * (int)((keys[info.first + j] >> shift) & 7ull));
                    hist += __shfl_xor(hist, 1, 8);
                    hist += __shfl_xor(hist, 2, 8);
                    hist += __shfl_xor(hist, 4, 8);
                    const uint64_t below = o == 0 ? 0ull : hist & (~0ull >> (64 - 8 * o));
                    start = info.first + (int32_t)((below * 0x0101010101010101ull) >> 56);
                } else {
                    int32_t a = info.first, b = info.first + count;
                    while (a < b) {
                        const int32_t mid = (a + b) >> 1;
                        if ((int)((keys[mid] >> shift) & 7ull) < o)
                            a = mid + 1;
                        else
                            b = mid;
                    }
                    start = a;
                }
                int32_t end = __shfl_down(start, 1, 8);
                if (o == 7) end = info.first + count;
                BHX_CHECK(!live || (start >= info.first && start <= end &&
                                    end <= info.first + info.count),
                          CK_PARTITION);
                const int32_t nb = end - start;
                const bool child = live && nb > 0;
                const bool deeper = child && nb > leaf && level + 1 < kMaxLevel;
                const uint64_t cb = __ballot(child), sb = __ballot(deeper);
                if (lane == 0) {
                    s_wtot[par][wave] = (uint32_t)__popcll(cb);
                    s_wdeep[par][wave] = (uint32_t)__popcll(sb);
                }
                __syncthreads();
                uint32_t before = 0, btot = 0, dbefore = 0, dtot = 0;
#pragma unroll
                for (int w = 0; w < W; w++) {
                    const uint32_t t = s_wtot[par][w], u = s_wdeep[par][w];
                    if (w < wave) before += t, dbefore += u;
                    btot += t;
                    dtot += u;
                }
                if (tid == 0) {
                    s_base[par] = (int64_t)atomicAdd(&hdr->deep_count, (unsigned long long)btot);
                    if (top + (int)dtot > kSubList && s_inner == kNotYet) {
                        s_inner =
                            (int64_t)atomicAdd(&hdr->inner_top, (unsigned long long)s_need);
                        if (s_inner + s_need > inner_words) {
                            s_inner = kNoRoom;
                            flag_status(hdr->status, ST_CAPACITY);
                        }
                    }
                }
                __syncthreads();
                const int64_t base = (int64_t)deep0 + s_base[par];
                const int64_t cid = base + (int64_t)(before + lanes_below(cb));
                const int32_t scene_bits = info.lvl_nch & (int32_t)0xffff0000;
                const bool fits = base + btot <= node_cap;  // the same on every thread
                total += (int32_t)btot;
                if (child && (fits || cid < node_cap)) {
                    const int at = top + (int)(dbefore + lanes_below(sb));
                    const NodeInfo ci{start, nb, -1, (level + 1) | scene_bits};
                    ninfo[cid] = ci;
                    if (level + 1 == kHintLevel) atomicMax(&s_hint, nb);
                    if (deeper && fits && at < kSubList)
                        list[at] = (int32_t)cid;
                    else if (deeper && fits && s_inner != kNoRoom)
                        inner[s_inner + at - kSubNodes] = (int32_t)cid;
                    else  // a leaf, or one for want of room
                        node_moments<QUAD, 4>((int32_t)cid, ci, level + 1, body, beps2, keys, box,
                                              nmom, neps2, nquad, use_eps);
                }
                if (!fits) {
                    if (tid == 0) flag_status(hdr->status, ST_CAPACITY);
                    continue;
                }
                if (live && o == 0) {
                    ninfo[id].child0 = (int32_t)cid;
                    ninfo[id].lvl_nch =
                        level | ((int)__popcll((cb >> gl) & 0xffull) << 8) | scene_bits;
                }
                top += (int)dtot;
                if (s_inner == kNoRoom && top > kSubList) top = kSubList;
            }
            if (tid == 0) {
                made[level + 1] += total;
                lbeg[d + 2] = top;
            }
            __syncthreads();
            lo = hi;
            hi = top;
        }
        for (d--; d >= 0; d--) {
            for (int i = lbeg[d] + tid; i < lbeg[d + 1]; i += kSubThreads) {
                const int32_t id = entry(i);
                node_moments<QUAD, 4>(id, ninfo[id], level0 + d, body, beps2, keys, box, nmom, neps2, nquad,
                             use_eps);
            }
            __syncthreads();
        }
    }
    __syncthreads();
    if (tid < kLevels && made[tid] > 0)
        atomicAdd(&hdr->deep[blockIdx.x % kDeepSlots].level[tid], made[tid]);
    if (tid == 0) raise_max(&hdr->cell_max[kHintLevel], s_hint);
}

// The end of a build, by one wave: the nodes that k_build_subtrees made and
// counted apart are added to their levels, and the launch hints go to pinned
// host memory (HintWord; n: the build's bodies).
__device__ inline void report_hints(TreeHeader *__restrict__ hdr, int32_t n, int32_t *out)
{
    const int l = threadIdx.x & 63;
    int32_t c = 0, most = 0;
    if (l < kLevels) {
        c = hdr->level_count[l];
        most = hdr->cell_max[l];
#pragma unroll
        for (int k = 0; k < kDeepSlots; k++) {
            c += hdr->deep[k].level[l];
            hdr->deep[k].level[l] = 0;
        }
        hdr->level_count[l] = c;
    }
    const uint64_t some = __ballot(c > 0) & ~1ull;
    if (!out) return;
    if (l == 0) {
        out[kHintDepth] = some ? 63 - __builtin_clzll(some) : 0;
        out[kHintBodies] = n;
        out[kHintScenes] = c;
    }
    if (l == kHintLevel) out[kHintMost5] = most;
    if (l < kLevels) {
        out[kHintCount + l] = c;
        out[kHintMost + l] = most;
    }
}

template <bool QUAD>
__global__ __launch_bounds__(256) void k_moments_level(
    int level, TreeHeader *__restrict__ hdr, const NodeInfo *__restrict__ ninfo,
    const Body *__restrict__ body, const double *__restrict__ beps2,
    const uint64_t *__restrict__ keys, SceneBox *box,
    NodeMom *__restrict__ nmom, double *__restrict__ neps2, double *__restrict__ nquad,
    int64_t node_cap, int use_eps, int n_bodies, int n_scenes,
    int32_t *__restrict__ depth_out)
{
    moments_nodes<QUAD>(level, hdr->level_count, ninfo, body, beps2, keys, box, nmom, neps2, nquad,
                  node_cap, use_eps, (int64_t)blockIdx.x * 256 + threadIdx.x,
                  (int64_t)gridDim.x * 256);
    // the root level reports the launch hints for the next build
    if (level == 0 && blockIdx.x == 0) {
        if (threadIdx.x < 64) report_hints(hdr, n_bodies, depth_out);
        for (int sc = threadIdx.x; sc < n_scenes; sc += 256) reset_box(box + sc);
    }
}

// Levels from-1 down to 0 of a single scene in one block (at most kHeadNodes
// nodes, one a thread), then the depth report of k_moments_level at level 0. A
// chain of latencies: the node table is read once, the leaves and level from-1 are
// summed from global memory at once, and the levels above from a copy of the
// moments in LDS: 13.5 us -> 9.5 at 50,000 bodies, 26 -> 18 with quadrupoles at
// 20,000, against a pass over global memory a level.
constexpr int kHeadLevels = 4, kHeadNodes = 1 + 8 + 64 + 512;
constexpr int kHeadThreads = 640;
static_assert(kHeadThreads >= kHeadNodes, "a node a thread");
template <bool QUAD>
__global__ __launch_bounds__(kHeadThreads) void k_moments_head(
    int from, TreeHeader *__restrict__ hdr, const NodeInfo *__restrict__ ninfo,
    const Body *__restrict__ body, const double *__restrict__ beps2,
    const uint64_t *__restrict__ keys, SceneBox *box,
    NodeMom *__restrict__ nmom, double *__restrict__ neps2, double *__restrict__ nquad,
    int64_t node_cap, int use_eps, int n_bodies, int32_t *__restrict__ depth_out)
{
    __shared__ NodeMom s_mom[kHeadNodes];
    __shared__ double s_eps2[kHeadNodes], s_quad[QUAD ? 6 * kHeadNodes : 1];
    const int t = threadIdx.x;
    int level = -1;  // of node t
    int32_t end = 0;
    for (int l = 0; l < from; l++) {
        int32_t beg, cnt;
        level_range(hdr->level_count, l, node_cap, &beg, &cnt);
        end = beg + cnt;
        if (t >= beg && t < end) level = l;
    }
    BHX_CHECK(end <= kHeadNodes, CK_PARTITION);
    NodeInfo info{0, 0, -1, 0};
    if (level >= 0) info = ninfo[t];
    auto put = [&](const NodeMom &m, double e2, const double *q) {
        nmom[t] = s_mom[t] = m;
        if (use_eps) neps2[t] = s_eps2[t] = e2;
        if constexpr (QUAD)
#pragma unroll
            for (int a = 0; a < 6; a++) nquad[6 * t + a] = s_quad[6 * t + a] = q[a];
    };
    if (level >= 0 && (level == from - 1 || info.child0 < 0)) {
        double e2, q[6];
        const NodeMom m = node_sums<QUAD>(info, level, body, beps2, keys, box, nmom, neps2, nquad,
                                    use_eps, e2, q);
        put(m, e2, q);
    }
    __syncthreads();
    for (int l = from - 2; l >= 0; l--) {
        if (level == l && info.child0 >= 0) {
            double e2, q[6];
            const NodeMom m = node_sums<QUAD>(info, level, body, beps2, keys, box, s_mom, s_eps2,
                                        s_quad, use_eps, e2, q);
            put(m, e2, q);
        }
        __syncthreads();
    }
    if (t < 64) report_hints(hdr, n_bodies, depth_out);
    if (t == 0) reset_box(box);
}

// The deep levels in one block (they hold few nodes): with `split`, first
// the split of levels to..kMaxLevel-1 (stopping at the first empty level,
// the node counts kept in LDS), then the moments of levels kMaxLevel down
// to `to`.
template <bool QUAD>
__global__ __launch_bounds__(1024) void k_moments_tail(
    int to, int split, const uint64_t *__restrict__ keys, TreeHeader *__restrict__ hdr,
    NodeInfo *__restrict__ ninfo, const Body *__restrict__ body,
    const double *__restrict__ beps2, const SceneBox *__restrict__ box,
    NodeMom *__restrict__ nmom, double *__restrict__ neps2, double *__restrict__ nquad,
    int64_t node_cap, int leaf, int use_eps)
{
    __shared__ int32_t scnt[kLevels + 1];
    if (threadIdx.x <= kLevels) scnt[threadIdx.x] = hdr->level_count[threadIdx.x];
    __syncthreads();
    if (split) {  // the same on every thread
        build_levels_block<true>(to, kMaxLevel, keys, hdr, ninfo, node_cap, leaf, scnt);
        __syncthreads();
        if (threadIdx.x <= kLevels) hdr->level_count[threadIdx.x] = scnt[threadIdx.x];
    }
    for (int level = kMaxLevel; level >= to; level--) {
        if (scnt[level] == 0) continue;  // the same on every thread
        moments_nodes<QUAD>(level, scnt, ninfo, body, beps2, keys, box, nmom, neps2, nquad, node_cap,
                      use_eps, threadIdx.x, 1024);
        __syncthreads();
    }
}

// ------------------------------------------------- whole build, small scene

// The whole build of one scene of at most kSmallBuild bodies in one block:
// box and input check, keys, a stable merge sort of (key, index), gather, every
// level of the tree and the moments. Each stage computes what the multi-launch
// path computes (the same stable order, the same node set and moments); a small
// scene is bound by latency, so the stages are chosen for few dependent steps:
//   sort     runs of 64 ranked by comparison in LDS, then runs merged in pairs,
//            each key finding its place by a binary search in the other run
//            (one barrier a round, 4 rounds at 1000 bodies, 6 at 4096, where
//            eight radix passes took 40 barriers and left most waves idle);
//   levels   only the nodes that split are carried from level to level, in an
//            LDS list; a wave reserves its children with one LDS atomic and the
//            level ends in one barrier (six, and the node table in global
//            memory, with the launches' split);
//   moments  of every leaf at once, then the internal nodes level by level from
//            a copy of the moments in LDS (up to kCacheNodes nodes).
// A ball of 1000 bodies, leaf 16: 80 -> 20 us; leaf 1 (ten levels) 119 -> 32 us;
// 4096 bodies, leaf 16: 111 -> 47 us.
constexpr int kSmallThreads = 1024;
constexpr int kCacheNodes = 3840;
// LDS: two buffers of keys and indices while sorting; the sorted keys and two
// lists of splitting nodes while splitting; node moments at the end; above all of
// these, for at most kCacheBodies bodies, the sorted bodies that the leaves sum.
constexpr int kCacheBodies = 1024;
constexpr int kSmallLds = kCacheNodes * (int)(sizeof(NodeMom) + sizeof(double));
static_assert(kSmallLds >= (int)kSmallBuild * (8 + 8), "keys and split lists");
static_assert(kCacheNodes <= 4 * kSmallThreads, "nodes a thread keeps");
constexpr int kNodeLds = (int)(sizeof(NodeMom) + sizeof(double));
constexpr int kBodyLds = kCacheBodies * (int)(sizeof(Body) + sizeof(double));
static_assert(kSmallLds - kBodyLds >= (int)kSmallBuild * (2 * (8 + 2) + 4), "bodies beside the sort");

// One round of merges: runs of LEN keys in pairs, from buffer src to dst, E keys a
// thread. A key goes to its place in its own run plus the number of keys of the
// other run before it: less, or, coming from the left run, equal (so that the
// order is stable). The searches are unrolled, three instructions and one LDS read
// at a constant offset a step, and a thread's E searches run side by side: with a
// loop over a run-time length and one search at a time the sort of 4096 bodies took
// 33 us, now 16.
template <int LEN, int E>
__device__ inline void merge_runs(const uint64_t *__restrict__ ksrc,
                                  const uint16_t *__restrict__ vsrc, uint64_t *__restrict__ kdst,
                                  uint16_t *__restrict__ vdst, int m)
{
    if (E == 1 && (int)threadIdx.x >= m) return;
    uint64_t k[E], lim[E];
    int o[E], c[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int p = threadIdx.x + e * kSmallThreads;
        k[e] = ksrc[p];
        const bool right = (p & LEN) != 0;
        o[e] = (p & ~(2 * LEN - 1)) + (right ? 0 : LEN);  // the other run
        lim[e] = k[e] + (right ? 1 : 0);                  // its keys below this come first
        c[e] = 0;
    }
#pragma unroll
    for (int s = LEN / 2; s > 0; s >>= 1)
#pragma unroll
        for (int e = 0; e < E; e++) c[e] += ksrc[o[e] + c[e] + s - 1] < lim[e] ? s : 0;
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int p = threadIdx.x + e * kSmallThreads;
        c[e] += ksrc[o[e] + c[e]] < lim[e] ? 1 : 0;
        const int to = (p & LEN ? p - LEN : p) + c[e];
        kdst[to] = k[e];
        vdst[to] = vsrc[p];
    }
}

// A stable sort of the m (1024 E, or 64 times a power of two below) keys and
// indices in buffer 0; returns the buffer that holds the order. Keys are below
// 2^64 - 1; high: their high words.
template <int E>
__device__ inline int small_sort(uint64_t (*key)[kSmallBuild], uint16_t (*val)[kSmallBuild],
                                 const uint32_t *high, int m)
{
    const int lane = threadIdx.x & 63;
    // runs of 64, one per wave: each lane counts the keys before its own, by the
    // high words (levels 1 to 10) where no two of the run are equal, else by
    // whole keys
    for (int p = threadIdx.x; p < m; p += kSmallThreads) {
        const uint64_t k = key[0][p];
        const int r0 = p - lane;
        const uint64_t *run = key[0] + r0;
        const uint4 *hrun = (const uint4 *)(high + r0);
        const uint32_t kh = (uint32_t)(k >> 32);
        int rank = 0;
#pragma unroll 4
        for (int j = 0; j < 16; j++) {
            const uint4 h = hrun[j];
            rank += (h.x < kh ? 1 : 0) + (h.y < kh ? 1 : 0) + (h.z < kh ? 1 : 0) + (h.w < kh ? 1 : 0);
        }
        // a place that two lanes claim: equal high words somewhere in the run
        val[1][r0 + rank] = (uint16_t)lane;
        __builtin_amdgcn_wave_barrier();
        if (__ballot(val[1][r0 + rank] != lane)) {
            rank = 0;
#pragma unroll 1
            for (int j = 0; j < 64; j++) {
                const uint64_t o = run[j];
                rank += (o < k || (o == k && j < lane)) ? 1 : 0;
            }
        }
        __builtin_amdgcn_wave_barrier();
        key[1][r0 + rank] = k;
        val[1][r0 + rank] = val[0][p];
    }
    __syncthreads();
    int src = 1;
    for (int len = 64; len < m; len *= 2) {
        const uint64_t *ks = key[src];
        const uint16_t *vs = val[src];
        uint64_t *kd = key[src ^ 1];
        uint16_t *vd = val[src ^ 1];
        switch (len) {
            case 64: merge_runs<64, E>(ks, vs, kd, vd, m); break;
            case 128: merge_runs<128, E>(ks, vs, kd, vd, m); break;
            case 256: merge_runs<256, E>(ks, vs, kd, vd, m); break;
            case 512: merge_runs<512, E>(ks, vs, kd, vd, m); break;
            case 1024:
                if constexpr (E > 1) merge_runs<1024, E>(ks, vs, kd, vd, m);
                break;
            default:
                if constexpr (E > 2) merge_runs<2048, E>(ks, vs, kd, vd, m);
                break;
        }
        src ^= 1;
        __syncthreads();
    }
    return src;
}

// A splitting node of a level: its number, first body and body count.
struct SplitNode {
    int32_t id;
    uint16_t first, count;
};

// One axis of launch_euler_substeps, each operation rounded as written.
__device__ inline void euler_axis(double &x, double &v, double a, double dt, int substeps)
{
#pragma clang fp contract(off)
    for (int j = 0; j < substeps; j++) {
        v = v + dt * a;
        x = x + dt * v;
    }
}

// With adv.vel the bodies are moved first (a launch of its own took 5 us of a
// 65 us substep of 1000 bodies), and pos holds the moved positions.
template <bool QUAD>
__global__ __launch_bounds__(kSmallThreads) void k_build_small(
    const double *pos, Advance adv, const double *__restrict__ mass,
    const double *__restrict__ eps, int64_t n64, int leaf, SceneBox *__restrict__ box,
    TreeHeader *__restrict__ hdr, uint64_t *__restrict__ k0, uint32_t *__restrict__ i0,
    Body *__restrict__ body,
    double *__restrict__ beps2, NodeInfo *__restrict__ ninfo, NodeMom *__restrict__ nmom,
    double *__restrict__ neps2, double *__restrict__ nquad, int64_t node_cap,
    int32_t *__restrict__ depth_out)
{
    constexpr int kPer = (int)(kSmallBuild / kSmallThreads);
    __shared__ alignas(16) char lds[kSmallLds];
    static_assert(kSmallThreads / 16 == 64, "one row of 16 lanes a lane");
    __shared__ double red[64][6];
    __shared__ SceneBox sbox;
    __shared__ bool swild[kSmallThreads / 64];
    __shared__ int32_t scnt[kLevels + 1];
    __shared__ int32_t nsplit[3];
    const int n = (int)n64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool use_eps = eps != nullptr;
    uint64_t(*skey)[kSmallBuild] = (uint64_t(*)[kSmallBuild])lds;
    uint16_t(*sval)[kSmallBuild] = (uint16_t(*)[kSmallBuild])(lds + 2 * sizeof(uint64_t) * kSmallBuild);

    // 1. box and input check
    double x[kPer][3];
    {
        double lo[3] = {kInf, kInf, kInf}, hi[3] = {-kInf, -kInf, -kInf};
        bool bad = false, wild = false;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int i = tid + j * kSmallThreads;
            if (i >= n) continue;
            for (int a = 0; a < 3; a++) x[j][a] = pos[3 * i + a];
            if (adv.vel) {
                for (int a = 0; a < 3; a++) {
                    const double acc = adv.acc[3 * i + a];
                    double v = adv.vel[3 * i + a];
                    if (adv.substeps > 0) {
                        euler_axis(x[j][a], v, acc, adv.dt, adv.substeps);
                    } else {
                        v = fma(0.5 * adv.dt, acc, v);
                        x[j][a] = fma(adv.dt, v, x[j][a]);
                    }
                    adv.vel[3 * i + a] = v;
                    adv.pos[3 * i + a] = x[j][a];
                }
            }
            const double m = mass[i];
            bad |= !(isfinite(x[j][0]) && isfinite(x[j][1]) && isfinite(x[j][2]));
            bad |= !(isfinite(m) && m >= 0.0);
            const double e = use_eps ? eps[i] : 0.0;
            bad |= !(isfinite(e) && e >= 0.0);
            wild |= wild_body(m, e * e);
            for (int a = 0; a < 3; a++) {
                lo[a] = fmin(lo[a], x[j][a]);
                hi[a] = fmax(hi[a], x[j][a]);
            }
        }
        if (__ballot(bad) && lane == 0) flag_status(hdr->status, ST_NONFINITE);
        const bool any_wild = __ballot(wild) != 0;
        if (lane == 0) swild[wave] = any_wild;
        for (int a = 0; a < 3; a++) {
            const double l = row_min(lo[a]), h = row_max(hi[a]);
            if ((lane & 15) == 0) {
                red[tid >> 4][a] = l;
                red[tid >> 4][3 + a] = h;
            }
        }
    }
    if (tid <= kLevels) scnt[tid] = tid == 0 ? 1 : 0;
    if (tid < 3) nsplit[tid] = 0;
    __syncthreads();
    if (tid < 64) {
        double v[6];
        for (int a = 0; a < 6; a++) v[a] = a < 3 ? row_min(red[lane][a]) : row_max(red[lane][a]);
#pragma unroll
        for (int o = 16; o < 64; o <<= 1)
            for (int a = 0; a < 6; a++) {
                const double u = __shfl_xor(v[a], o);
                v[a] = a < 3 ? fmin(v[a], u) : fmax(v[a], u);
            }
        const bool any_wild = __ballot(lane < kSmallThreads / 64 && swild[lane & 15]) != 0;
        if (lane == 0) reset_box(&sbox);
        root_cube(sbox, v, v + 3, lane, 64);
        if (lane == 0) sbox.mild = !any_wild && sbox.L <= kMildLength ? 1u : 0u;
    }
    __syncthreads();
    if (tid < (int)(sizeof(SceneBox) / 8)) ((uint64_t *)box)[tid] = ((const uint64_t *)&sbox)[tid];

    const bool few = n <= kCacheBodies;
    Body *const lbody = (Body *)(lds + kSmallLds - kBodyLds);
    double *const leps2 = (double *)(lds + kSmallLds - kCacheBodies * (int)sizeof(double));

    // 2. keys, in LDS; the places past n hold keys above any body's
    uint32_t *const high = (uint32_t *)(lds + 2 * (sizeof(uint64_t) + sizeof(uint16_t)) * kSmallBuild);
    int m = 64;
    while (m < n) m *= 2;
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        const int i = tid + j * kSmallThreads;
        if (i < m) {
            const uint64_t k =
                i < n ? morton_key(x[j], sbox) : (0xffffffc0ull | (uint64_t)(i & 63)) << 32;
            skey[0][i] = k;
            high[i] = (uint32_t)(k >> 32);
            sval[0][i] = (uint16_t)i;
        }
    }
    __syncthreads();

    // 3. sort, and 4. gather; the walk and the tree export read the sorted keys
    // and indices from global memory
    {
        static_assert(kSmallBuild == 4 * kSmallThreads, "keys a thread");
        const int at = m > 2 * kSmallThreads ? small_sort<4>(skey, sval, high, m)
                       : m > kSmallThreads   ? small_sort<2>(skey, sval, high, m)
                                             : small_sort<1>(skey, sval, high, m);
        uint64_t mine[kPer];
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int s = tid + j * kSmallThreads;
            if (s >= n) continue;
            const uint32_t i = sval[at][s];
            mine[j] = skey[at][s];
            k0[s] = mine[j];
            i0[s] = i;
            const Body b{pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], mass[i]};
            const double e = use_eps ? eps[i] : 0.0;
            body[s] = b;
            if (use_eps) beps2[s] = e * e;
            if (few) {
                lbody[s] = b;
                leps2[s] = e * e;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int s = tid + j * kSmallThreads;
            if (s < n) skey[0][s] = mine[j];
        }
    }
    const uint64_t *key = skey[0];
    SplitNode(*list)[kSmallBuild / 2] =
        (SplitNode(*)[kSmallBuild / 2])(lds + sizeof(uint64_t) * kSmallBuild);
    if (tid == 0) {
        if (n > leaf) {
            list[0][0] = SplitNode{0, 0, (uint16_t)n};
            nsplit[0] = 1;
        } else {
            ninfo[0] = NodeInfo{0, n, -1, 0};
        }
    }
    __syncthreads();

    // 5. tree, top-down, eight lanes a splitting node. A splitting node holds at
    // least two bodies, so a level has at most n / 2 of them. nsplit turns over
    // three counters: this level's, the next one's and the one being cleared.
    int beg = 1;  // first node of level + 1
    for (int level = 0; level < kMaxLevel; level++) {
        const int ns = nsplit[level % 3];
        if (ns == 0) break;  // the same on every thread
        const SplitNode *now = list[level & 1];
        SplitNode *next = list[(level & 1) ^ 1];
        const int o = tid & 7, gl = lane & ~7, shift = 60 - 3 * level;
        if (tid == 0) nsplit[(level + 2) % 3] = 0;
        for (int g0 = 8 * wave; g0 < ns; g0 += kSmallThreads / 8) {
            const int g = g0 + (lane >> 3);
            const SplitNode nd = now[g < ns ? g : g0];
            const int first = nd.first, count = g < ns ? nd.count : 0;
            const bool live = count > 0;  // (0: listed by an overflow)
            int start;
            if (count <= kLinearSplit) {
                uint64_t hist = 0;  // one byte per octant
                for (int j = o; j < count; j += 8)
                    hist += 1ull << (8 * (int)((key[first + j] >> shift) & 7ull));
                hist += __shfl_xor(hist, 1, 8);
                hist += __shfl_xor(hist, 2, 8);
                hist += __shfl_xor(hist, 4, 8);
                const uint64_t below = o == 0 ? 0ull : hist & (~0ull >> (64 - 8 * o));
                start = first + (int)((below * 0x0101010101010101ull) >> 56);
            } else {
                int a = first, b = first + count;
                while (a < b) {
                    const int mid = (a + b) >> 1;
                    if ((int)((key[mid] >> shift) & 7ull) < o)
                        a = mid + 1;
                    else
                        b = mid;
                }
                start = a;
            }
            int end = __shfl_down(start, 1, 8);
            if (o == 7) end = first + count;
            BHX_CHECK(start >= first && start <= end && end <= first + count, CK_PARTITION);
            const bool child = live && end > start;
            const uint64_t cb = __ballot(child);
            const bool deeper = child && end - start > leaf && level + 1 < kMaxLevel;
            const uint64_t sb = __ballot(deeper);
            int base = 0, at = 0;
            if (lane == 0) {
                base = atomicAdd(&scnt[level + 1], __popcll(cb));
                if (sb) at = atomicAdd(&nsplit[(level + 1) % 3], __popcll(sb));
            }
            base = beg + __builtin_amdgcn_readfirstlane(base);
            at = __builtin_amdgcn_readfirstlane(at);
            const int id = base + (int)lanes_below(cb);
            if (base + __popcll(cb) > node_cap) {  // the same on every lane
                // nothing is linked, but all that was counted is written
                if (lane == 0) flag_status(hdr->status, ST_CAPACITY);
                if (live && o == 0) ninfo[nd.id] = NodeInfo{first, count, -1, level};
                if (deeper) next[at + (int)lanes_below(sb)] = SplitNode{0, 0, 0};
                if (child && id < node_cap) ninfo[id] = NodeInfo{start, end - start, -1, level + 1};
                continue;
            }
            if (deeper)
                next[at + (int)lanes_below(sb)] =
                    SplitNode{id, (uint16_t)start, (uint16_t)(end - start)};
            else if (child)
                ninfo[id] = NodeInfo{start, end - start, -1, level + 1};
            if (live && o == 0)
                ninfo[nd.id] = NodeInfo{first, count, id,
                                        level | ((int)__popcll((cb >> gl) & 0xffull) << 8)};
        }
        __syncthreads();
        beg += scnt[level + 1];
    }
    int depth = 0, total = 0;
    for (int l = 0; l < kLevels; l++) {
        if (scnt[l] > 0) depth = l;
        total += scnt[l];
    }

    // 6. moments
    const int cache = few ? (kSmallLds - kBodyLds) / kNodeLds : kCacheNodes;
    if (total <= cache && total <= node_cap && !QUAD) {
        NodeMom *cm = (NodeMom *)lds;
        double *ce = (double *)(lds + cache * sizeof(NodeMom));
        int inner[4];  // an internal node's first child, children << 12 and level << 16
        __syncthreads();  // the keys and lists are read no more
        auto store = [&](int k, int level, const MomentSum &s) {
            double e2;
            const int32_t first = s.ms > 0.0 ? 0 : ninfo[k].first;  // read for a massless cell only
            const NodeMom out = s.moments(level, first, k0, sbox, use_eps, e2);
            cm[k] = out;
            nmom[k] = out;
            if (use_eps) {
                ce[k] = e2;
                neps2[k] = e2;
            }
        };
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = tid + j * kSmallThreads;
            inner[j] = -1;
            if (k >= total) continue;
            const NodeInfo info = ninfo[k];
            if (info.child0 >= 0) {
                inner[j] = info.child0 | node_nchild(info) << 12 | node_level(info) << 16;
            } else {
                MomentSum s;
                if (few)
                    s.leaf(lbody, leps2, info, use_eps);
                else
                    s.leaf(body, beps2, info, use_eps);
                store(k, node_level(info), s);
            }
        }
        __syncthreads();
        for (int level = depth - 1; level >= 0; level--) {
            // the level's nodes are consecutive, so a thread seldom has two of them
#pragma unroll 1
            for (int j = 0; j < 4; j++) {
                const int in = j == 0 ? inner[0] : j == 1 ? inner[1] : j == 2 ? inner[2] : inner[3];
                if (in < 0 || in >> 16 != level) continue;
                MomentSum s;
                s.children<4>(cm, ce, NodeInfo{0, 0, in & 0xfff, (in >> 12 & 0xf) << 8}, use_eps);
                store(tid + j * kSmallThreads, level, s);
            }
            __syncthreads();
        }
    } else {
        for (int level = depth; level >= 0; level--) {
            moments_nodes<QUAD>(level, scnt, ninfo, body, beps2, key, box, nmom, neps2, nquad, node_cap,
                          use_eps, tid, kSmallThreads);
            __syncthreads();
        }
    }
    if (tid <= kLevels) hdr->level_count[tid] = scnt[tid];
    if (depth_out && tid == 0) {
        depth_out[kHintDepth] = depth;
        depth_out[kHintMost5] = -1;  // no sort hint from a one-block build
        depth_out[kHintBodies] = n;
        depth_out[kHintScenes] = 1;
    }
    if (depth_out && tid < kLevels) {
        depth_out[kHintCount + tid] = scnt[tid];
        depth_out[kHintMost + tid] = -1;
    }
}

inline unsigned blocks_for(int64_t items, int per_block, unsigned cap)
{
    int64_t b = (items + per_block - 1) / per_block;
    if (b < 1) b = 1;
    return (unsigned)(b < (int64_t)cap ? b : cap);
}

// Upper bound on the nodes of one level: at most 8^level per scene and at
// most n in all.
inline int64_t level_bound(int level, int64_t n, int scenes)
{
    int64_t b = scenes;
    for (int l = 0; l < level && b < n; l++) b *= 8;
    return b < n ? b : n;
}

// One block per scene fills its body range.
__global__ __launch_bounds__(256) void k_scene_of(const int64_t *__restrict__ offsets,
                                                  uint16_t *__restrict__ scene_of)
{
    const int sc = blockIdx.x;
    for (int64_t i = offsets[sc] + threadIdx.x; i < offsets[sc + 1]; i += 256)
        scene_of[i] = (uint16_t)sc;
}

// One launch for a new workspace (three fills and a copy took 10 us more).
__global__ __launch_bounds__(256) void k_init(SceneBox *__restrict__ box, int scenes,
                                              uint32_t *__restrict__ hdr, uint32_t *status,
                                              int32_t *__restrict__ mark,
                                              int32_t *__restrict__ nparent, int64_t nodes)
{
    const int t = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
    for (int i = t; i < scenes; i += stride) reset_box(box + i);
    constexpr int kAt = (int)(offsetof(TreeHeader, status) / 4);
    for (int i = t; i < (int)(sizeof(TreeHeader) / 4); i += stride)
        hdr[i] = i == kAt       ? (uint32_t)(uintptr_t)status
                 : i == kAt + 1 ? (uint32_t)((uintptr_t)status >> 32)
                                : 0u;
    for (int i = t; i < kPrefixCells; i += stride) mark[i] = INT32_MAX;
    if (nparent)
        for (int64_t i = t; i < nodes; i += stride) nparent[i] = -1;
}

}  // namespace

hipError_t launch_init(const Workspace &w, int32_t *nparent)
{
    k_init<<<nparent ? 1024 : 128, 256>>>(w.box, w.max_scenes, (uint32_t *)w.hdr, w.status_dev,
                                          w.prefix_mark, nparent, w.node_cap);
    return hipGetLastError();
}

hipError_t launch_scene_of(hipStream_t s, const int64_t *offsets, int n_scenes,
                           uint16_t *scene_of)
{
    k_scene_of<<<n_scenes, 256, 0, s>>>(offsets, scene_of);
    return hipGetLastError();
}

namespace {

// Stages 2-3: keys of the bodies (coordinates at pos + stride * i) and the
// sort, leaving the sorted order in idx[0]: by buckets after top_passes passes on the
// top key bits (bucket_sort_hint), or with none by passes over the whole keys.
void enqueue_keys_sort(const Workspace &w, hipStream_t s, const Layout &lay, const double *pos,
                       int stride, int top_passes)
{
    const int64_t n = lay.n;
    const int ns = lay.n_scenes;
    const int nblk = (int)((n + kSortTile - 1) / kSortTile);
    const unsigned nb0 = blocks_for(n, 256, 1u << 30);
    if (top_passes) {
        // passes on the top key bits and, for several scenes, one on the scene
        // index (ending in buffer 0), then the buckets in place
        const int passes = ns > 1 ? top_passes + 1 : top_passes;
        const int first = passes & 1, top = top_shift(top_passes);
        if (ns == 1)  // the root cube, the keys and the first pass's digit counts
            k_keys_hist<<<nblk, kSortThreads, 0, s>>>(pos, stride, n, w.box, w.hdr, w.ninfo,
                                                      w.keys[first], w.idx[first], top,
                                                      w.sort_counts, nblk);
        else
            k_keys<<<nb0, 256, 0, s>>>(pos, stride, n, w.box, lay.scene_of, w.keys[first],
                                       w.idx[first]);
        for (int pass = 0; pass < passes; pass++) {
            const int shift = pass < top_passes ? top + 8 * pass : 64;
            const int src = (pass + first) & 1, dst = src ^ 1;
            if (ns > 1 || pass > 0)
                k_sort_hist<<<nblk, kSortThreads, 0, s>>>(w.keys[src], w.idx[src], lay.scene_of,
                                                          lay.offsets, ns, n, shift, w.sort_counts,
                                                          nblk);
            k_sort_scan<<<256, 256, 0, s>>>(w.sort_counts, w.sort_totals, nblk);
            k_sort_scatter<<<nblk, kSortThreads, 0, s>>>(w.keys[src], w.idx[src], lay.scene_of,
                                                         lay.offsets, ns, w.keys[dst], w.idx[dst],
                                                         n, shift, w.sort_counts, w.sort_totals,
                                                         nblk);
        }
        if (n >= kBigSortFrom)
            k_sort_local<LocalBig>
                <<<(unsigned)((n + LocalBig::kTile - 1) / LocalBig::kTile), LocalBig::kThreads, 0,
                   s>>>(w.keys[0], w.idx[0], w.keys[1], w.idx[1], n, top, lay.offsets, ns);
        else
            k_sort_local<LocalSmall>
                <<<(unsigned)((n + LocalSmall::kTile - 1) / LocalSmall::kTile),
                   LocalSmall::kThreads, 0, s>>>(w.keys[0], w.idx[0], w.keys[1], w.idx[1], n,
                                                 top, lay.offsets, ns);
#ifdef BHX_CHECKS
        k_check_order<<<nb0, 256, 0, s>>>(w.keys[0], w.idx[0], n, lay.offsets, ns);
#endif
        return;
    }
    // 8 passes on the Morton key, then (several scenes) one on each byte of
    // the scene index that is not always zero; the keys start in the buffer
    // that makes the last pass write buffer 0.
    const int passes = ns > 256 ? 10 : ns > 1 ? 9 : 8;
    const int first = passes & 1;
    k_keys<<<nb0, 256, 0, s>>>(pos, stride, n, w.box, lay.scene_of, w.keys[first], w.idx[first]);
    for (int pass = 0; pass < passes; pass++) {
        const int shift = pass < 8 ? 8 * pass : 64 + 8 * (pass - 8);
        const int src = (pass + first) & 1, dst = src ^ 1;
        k_sort_hist<<<nblk, kSortThreads, 0, s>>>(w.keys[src], w.idx[src], lay.scene_of,
                                                  lay.offsets, ns, n, shift, w.sort_counts, nblk);
        k_sort_scan<<<256, 256, 0, s>>>(w.sort_counts, w.sort_totals, nblk);
        k_sort_scatter<<<nblk, kSortThreads, 0, s>>>(w.keys[src], w.idx[src], lay.scene_of,
                                                     lay.offsets, ns, w.keys[dst], w.idx[dst], n,
                                                     shift, w.sort_counts, w.sort_totals, nblk);
    }
#ifdef BHX_CHECKS
    k_check_order<<<nb0, 256, 0, s>>>(w.keys[0], w.idx[0], n, lay.offsets, ns);
#endif
}

// Stages 5-6 on the sorted bodies (with the plan the gather was launched with).
// The kernels are short and start cold: code for the quadrupoles beside the plain
// sums made each of them 1 to 2 us longer, so it is instantiated apart.
template <bool QUAD>
void enqueue_levels(const Workspace &w, hipStream_t s, const Layout &lay, int leaf, bool use_eps,
                    const LevelPlan &plan)
{
    const int64_t n = lay.n;
    const int ns = lay.n_scenes;
    // Splitting: levels 0..deep-1 get a launch each, sized by the largest
    // scene; the levels from `deep` down, which the previous build on this
    // workspace left empty but for one level of growth, are handled in one
    // block. Moments: the same, and the top levels of a single scene (levels
    // 0..head-1, at most 585 nodes) in one block too. (Splitting the top
    // levels in one block was measured slower: its binary searches over all
    // bodies run four passes deep there.) The split only affects speed.
    const int deep = plan.sub >= 0 ? plan.sub : plan.deep, prev = plan.prev;
    const volatile int32_t *hint = w.depth_host;
    const int head = ns == 1 ? (deep < kHeadLevels ? deep : kHeadLevels) : 0;
    // one scene: levels 1..kPrefixLevels from the marks of the gather in one
    // block instead of one launch per level (when the previous build went deeper)
    if (plan.prefix)
        k_prefix_levels<<<1, 1024, 0, s>>>(w.prefix_mark, n, w.hdr, w.ninfo, w.node_cap, leaf);
    for (int level = plan.prefix ? kPrefixLevels : 0; level < deep; level++) {
        // a level whose next level held no more nodes in the previous build
        // holds mostly leaves: one thread per node, the splitting ones listed;
        // otherwise eight lanes per node. Levels of many nodes take 1024-thread
        // blocks (fewer reservations on the level counter), small ones 256
        // (more CUs for their searches). The choice only affects speed.
        const bool compact =
            prev >= 0 && level < kMaxLevel && hint[kHintCount + level] > 0 &&
            hint[kHintCount + level + 1] <= hint[kHintCount + level];
        const int64_t threads = level_bound(level, n, ns) * (compact ? 1 : 8);
        const int bs = threads >= 65536 ? 1024 : 256;
        const unsigned g = blocks_for(threads, bs, bs == 1024 ? 1024 : 4096);
        if (compact)
            k_build_level<true>
                <<<g, bs, 0, s>>>(level, w.keys[0], w.hdr, w.ninfo, w.node_cap, leaf);
        else
            k_build_level<false>
                <<<g, bs, 0, s>>>(level, w.keys[0], w.hdr, w.ninfo, w.node_cap, leaf);
    }
    const int ue = use_eps ? 1 : 0;
    if (plan.sub >= 0) {
        // as many blocks as the level's nodes need, by the previous build's count
        const unsigned blocks = blocks_for(plan.sub_nodes, kSubNodes, 1u << 16);
        k_build_subtrees<QUAD><<<blocks, kSubThreads, 0, s>>>(
            deep, w.keys[0], w.hdr, w.ninfo, w.node_cap, leaf, w.body, w.beps2, w.box, w.nmom,
            w.neps2, w.nquad, ue, w.inner, w.inner_words);
    } else {
        // the levels from `deep` down: their split and their moments in one block
        k_moments_tail<QUAD><<<1, 1024, 0, s>>>(deep, deep < kMaxLevel ? 1 : 0, w.keys[0], w.hdr,
                                                w.ninfo, w.body, w.beps2, w.box, w.nmom, w.neps2,
                                                w.nquad, w.node_cap, leaf, ue);
    }
    for (int level = deep - 1; level >= head; level--) {
        const unsigned g = blocks_for(level_bound(level, n, ns), 256, 4096);
        k_moments_level<QUAD><<<g, 256, 0, s>>>(level, w.hdr, w.ninfo, w.body, w.beps2, w.keys[0],
                                                w.box, w.nmom, w.neps2, w.nquad, w.node_cap, ue,
                                                (int)n, ns, w.depth_dev);
    }
    if (head > 0)
        k_moments_head<QUAD><<<1, kHeadThreads, 0, s>>>(head, w.hdr, w.ninfo, w.body, w.beps2,
                                                        w.keys[0], w.box, w.nmom, w.neps2, w.nquad,
                                                        w.node_cap, ue, (int)n, w.depth_dev);
}

}  // namespace

BHX_DEFINE_TAKE_CHECKS(tree_take_checks)

Workspace slot_view(const Workspace &w, const TreeSlots &t, int k)
{
    Workspace v = w;
    v.body = t.body + (int64_t)k * t.n;
    v.beps2 = t.beps2 + (int64_t)k * t.n;
    v.idx[0] = t.idx + (int64_t)k * t.n;
    v.keys[0] = t.keys + (int64_t)k * t.n;
    v.ninfo = t.ninfo + (int64_t)k * t.node_cap;
    v.nmom = t.nmom + (int64_t)k * t.node_cap;
    v.neps2 = t.neps2 + (int64_t)k * t.node_cap;
    v.node_cap = t.node_cap;
    v.box = t.box + k;
    v.hdr = t.hdr + k;
    v.max_scenes = 1;
    return v;
}

hipError_t launch_build(const Workspace &w, hipStream_t s, const Layout &lay, const double *pos,
                        const double *mass, const double *eps, int leaf, SortUsed *sort,
                        const Advance *adv)
{
    if (sort) *sort = SortUsed{};
    const int64_t n = lay.n;
    const int ns = lay.n_scenes;
    if (one_block_build(lay)) {
        const auto kernel = w.nquad ? k_build_small<true> : k_build_small<false>;
        kernel<<<1, kSmallThreads, 0, s>>>(pos, adv ? *adv : Advance{}, mass, eps, n, leaf, w.box,
                                           w.hdr, w.keys[0], w.idx[0], w.body, w.beps2, w.ninfo,
                                           w.nmom, w.neps2, w.nquad, w.node_cap, w.depth_dev);
        return hipGetLastError();
    }
    if (adv) return hipErrorInvalidValue;
    const unsigned sb = (unsigned)((ns + 255) / 256);
    const int per = box_chunk(n);
    const int nchunks = lay.chunks ? lay.n_chunks : (int)((n + per - 1) / per);
    if (nchunks > 0)
        k_box_chunk<<<nchunks, kBoxThreads, 0, s>>>(pos, mass, eps, n, per, lay.chunks, w.box,
                                                  w.hdr);
    // the sort is chosen once (a host read of the previous build's hint); a
    // single scene's bucket sort finishes the box in its key kernel
    bool even = false;
    const int bk = n > 0 ? bucket_sort_hint(w, lay, &even) : 0;
    if (sort) *sort = SortUsed{even, bk};
    if (!(bk && ns == 1)) k_box_final<<<sb, 256, 0, s>>>(w.box, ns, lay.offsets, n, w.hdr, w.ninfo);
    if (n == 0) return hipGetLastError();
    enqueue_keys_sort(w, s, lay, pos, 3, bk);
    const LevelPlan plan = plan_levels(w.depth_host, n, ns);
    k_gather<<<blocks_for(n, 256, 1u << 30), 256, 0, s>>>(pos, mass, eps, w.idx[0], n, w.body,
                                                          w.beps2, w.keys[0],
                                                          plan.prefix ? w.prefix_mark : nullptr);
    (w.nquad ? enqueue_levels<true> : enqueue_levels<false>)(w, s, lay, leaf, eps != nullptr, plan);
    return hipGetLastError();
}

hipError_t launch_build_state(const Workspace &w, hipStream_t s, const Layout &lay, bool use_eps,
                              int leaf, double dt, SortUsed *sort)
{
    if (sort) *sort = SortUsed{};
    const int64_t n = lay.n;
    const int ns = lay.n_scenes;
    if (n <= 0) return hipSuccess;
    const unsigned sb = (unsigned)((ns + 255) / 256);
    const int per = box_chunk(n);
    const int nchunks = lay.chunks ? lay.n_chunks : (int)((n + per - 1) / per);
    k_state_kick_drift<<<nchunks, kBoxThreads, 0, s>>>(
        w.body, w.tvel, w.tacc, w.beps2, w.idx[0], n, 0.5 * dt, dt, per, lay.chunks, w.sbody,
        w.svel, use_eps ? w.seps2 : nullptr, w.scidx, w.box, w.hdr);
    bool even;
    const int bk = bucket_sort_hint(w, lay, &even);  // read once, as in launch_build
    if (sort) *sort = SortUsed{even, bk};
    if (!(bk && ns == 1)) k_box_final<<<sb, 256, 0, s>>>(w.box, ns, lay.offsets, n, w.hdr, w.ninfo);
    enqueue_keys_sort(w, s, lay, reinterpret_cast<const double *>(w.sbody), 4, bk);
    const LevelPlan plan = plan_levels(w.depth_host, n, ns);
    k_gather_state<<<blocks_for(n, 256, 1u << 30), 256, 0, s>>>(
        w.sbody, w.svel, use_eps ? w.seps2 : nullptr, w.scidx, n, w.idx[0], w.body, w.tvel,
        w.beps2, w.keys[0], plan.prefix ? w.prefix_mark : nullptr);
    (w.nquad ? enqueue_levels<true> : enqueue_levels<false>)(w, s, lay, leaf, use_eps, plan);
    return hipGetLastError();
}

}  // namespace bhx
