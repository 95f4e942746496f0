// Internal declarations shared by the HIP translation units of libbhx.
// Device data layout, the tree header, and the kernel launchers each unit
// provides. Nothing here is part of the C ABI (include/bhx.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bhx.h"
#include "build_plan.h"
#include "capacity.h"
#include "checks.h"

namespace bhx {

constexpr uint32_t kQMax = 2097151u;    // 2^21 - 1

// Device errors, latched until bh_sync(): words of pinned host memory, one an
// error, so that a synchronisation reads them without a copy from the device (a
// 4-byte copy to pageable memory cost each synchronising call 15 us). A kernel
// that finds an error stores 1 (atomics on host memory are not needed for that).
enum : int { ST_NONFINITE = 0, ST_CAPACITY = 1, ST_WORDS = 2 };
__device__ inline void flag_status(uint32_t *status, int error)
{
    __hip_atomic_store(status + error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One body in Morton order: position and mass (32 B, one aligned load pair).
struct alignas(32) Body {
    double x, y, z, m;
};

// One node's moments: centre of mass and mass.
struct alignas(32) NodeMom {
    double x, y, z, m;
};

// One node's structure: sorted body range, first child (-1 for a leaf),
// level in bits 0..7, number of children in bits 8..15 and the scene the
// node belongs to in bits 16..31.
struct alignas(16) NodeInfo {
    int32_t first, count, child0, lvl_nch;
};

__host__ __device__ inline int node_level(const NodeInfo &i) { return i.lvl_nch & 0xff; }
__host__ __device__ inline int node_nchild(const NodeInfo &i) { return (i.lvl_nch >> 8) & 0xff; }
__host__ __device__ inline int node_scene(const NodeInfo &i)
{
    return (int)((uint32_t)i.lvl_nch >> 16);
}
constexpr int kMaxScenes = 65535;

// Root cube of one scene. lo_enc / hi_enc hold the per-axis minimum and the
// complement of the maximum as order-preserving integers while the box is being
// reduced, and all ones (no bodies yet) before and after a build; the same for
// mild_acc, zero once a mass or softening out of the ranges of kMild* was found.
struct SceneBox {
    unsigned long long lo_enc[3], hi_enc[3];
    uint32_t mild_acc;
    uint32_t mild;        // masses, softenings and side in those ranges
    double lo[3], hi[3];  // per-axis bounding box
    double L, S;          // root cube side and quantisation scale 2^21 / L
    double x0[3];         // root cube corner
    double s2[kLevels];   // squared cell side per level
};

constexpr int kDeepSlots = 16;
// Tree header, written on the device by the build and read by later kernels,
// so a whole force evaluation runs without host round trips.
struct TreeHeader {
    int32_t level_count[kLevels + 1];  // nodes created per level (all scenes)
    uint32_t *status;                  // ST_* words, set at creation
    int32_t cell_max[kLevels];         // most bodies in one node per level (0: not looked at)
    unsigned long long inner_top;      // words of Workspace::inner in use
    // nodes k_build_subtrees has created (past the node table too)
    alignas(128) unsigned long long deep_count;
    // and how many of them per level, spread over lines of their own (all blocks
    // adding to one line took longer than the rest of that kernel); added to
    // level_count, and cleared, by the kernel that reports the launch hints
    struct alignas(128) {
        int32_t level[kLevels];
    } deep[kDeepSlots];
};
constexpr int kStatusAt = 64;  // the status words follow, on a line of their own
static_assert(kHintWords <= kStatusAt, "pinned words");
constexpr int kPrefixCells = 1 << (3 * kPrefixLevels);  // 32768
constexpr int kPrefixShift = 63 - 3 * kPrefixLevels;

// Body layout of one call: n bodies in n_scenes contiguous scenes. For one
// scene every table is implicit (nullptr); otherwise scene_of gives each
// body's scene, chunks the bbox work items {scene, first, end} (none crosses
// a scene) and groups the walk groups {first, count, scene} (at most 64
// bodies, none crosses a scene), all in device memory.
struct Layout {
    int64_t n = 0;
    int n_scenes = 1;
    const int64_t *offsets = nullptr;  // device, n_scenes + 1
    const uint16_t *scene_of = nullptr;
    const int32_t *chunks = nullptr;   // [n_chunks][3]
    int n_chunks = 0;
    const int32_t *groups = nullptr;   // [n_groups][3]
    int n_groups = 0;
};
constexpr int kBoxChunk = 4096;  // bodies per bbox work item

// Morton interleave of 21-bit cell coordinates (x in the highest bit of
// each triplet) and its inverse.
// Spreads the low 21 bits of v so that bit i lands on bit 3i.
__device__ inline uint64_t spread3(uint64_t v)
{
    v &= 0x1fffffull;
    v = (v | (v << 32)) & 0x1f00000000ffffull;
    v = (v | (v << 16)) & 0x1f0000ff0000ffull;
    v = (v | (v << 8)) & 0x100f00f00f00f00full;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

// Inverse of spread3.
__device__ inline uint32_t compact3(uint64_t v)
{
    v &= 0x1249249249249249ull;
    v = (v ^ (v >> 2)) & 0x10c30c30c30c30c3ull;
    v = (v ^ (v >> 4)) & 0x100f00f00f00f00full;
    v = (v ^ (v >> 8)) & 0x1f0000ff0000ffull;
    v = (v ^ (v >> 16)) & 0x1f00000000ffffull;
    v = (v ^ (v >> 32)) & 0x1fffffull;
    return (uint32_t)v;
}

// Number of set bits of m below this lane.
__device__ inline uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive prefix sum over the 64 lanes of a wave (exact, integer), by DPP
// lane moves: four shifts within each row of 16 lanes, then the last lane of
// row 0 is added to row 1 and of row 2 to row 3, and the last lane of row 1
// to rows 2 and 3. Every lane of the wave must be active.
__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, kRowShr + 1, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kRowShr + 2, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kRowShr + 4, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kRowShr + 8, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kRowBcast15, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, kRowBcast31, 0xc, 0xf, false);
    return (uint32_t)x;
}

// 1 / sqrt(r2) in FP64 for a positive normal r2: the hardware estimate
// (relative error about 2^-24) refined by two Newton-Raphson steps on
// f(y) = y^-2 - r2, y <- y + y (1 - r2 y^2) / 2, each step squaring the
// relative error; on the whole normal range the result is within one ulp of
// the exact value. Cheaper than a correctly rounded sqrt followed by
// divisions, and well inside the FP64 parity bars.
__device__ inline double rsqrt_f64(double r2)
{
    double y = __builtin_amdgcn_rsq(r2);
    double e = fma(-(r2 * y), y, 1.0);
    y = fma(0.5 * y, e, y);
    e = fma(-(r2 * y), y, 1.0);
    return fma(0.5 * y, e, y);
}

// r2^(-3/2) for a positive normal r2 in one third-order step from the hardware
// estimate y (e = 1 - r2 y^2, at most about 2^-23): y^3 (1 - e)^(-3/2) =
// y^3 (1 + 3/2 e + 15/8 e^2) up to 35/16 e^3 < 2^-67, so only the roundings of
// the last products count (under three of them, as in cubing rsqrt_f64, at four
// instructions fewer). With RI also ri = r2^(-1/2) = y (1 + e / 2 + 3/8 e^2).
// The constants that an instruction cannot hold, kept in registers by the
// caller (the compiler would reload them for every term).
struct CubeConsts {
    double c1, c2, h2;
};
__device__ inline CubeConsts cube_consts()
{
    CubeConsts k{1.5, 1.875, 0.375};
    asm("" : "+v"(k.c1), "+v"(k.c2), "+v"(k.h2));
    return k;
}
template <bool RI>
__device__ inline double inv_cube_f64(double r2, double &ri, const CubeConsts &k)
{
    const double y = __builtin_amdgcn_rsq(r2), y2 = y * y;
    const double e = fma(-r2, y2, 1.0);
    if (RI) ri = fma(y * e, fma(e, k.h2, 0.5), y);
    const double y3 = y * y2;
    return fma(y3 * e, fma(e, k.c2, k.c1), y3);
}

// The same, with i2 = 1 / r2 = y^2 (1 + e + e^2) up to e^3.
template <bool RI = false>
__device__ inline double inv_cube_sq_f64(double r2, double &i2, double &ri, const CubeConsts &k)
{
    const double y = __builtin_amdgcn_rsq(r2), y2 = y * y;
    const double e = fma(-r2, y2, 1.0);
    i2 = fma(y2, fma(e, e, e), y2);
    if (RI) ri = fma(y * e, fma(e, k.h2, 0.5), y);
    const double y3 = y * y2;
    return fma(y3 * e, fma(e, k.c2, k.c1), y3);
}

// A pair term counts only when its squared softened distance is a positive
// normal number in the precision it is computed in: r^2 = 0 (coincident
// unsoftened bodies) and subnormal r^2 (the same coincidence below the
// number range, where 1 / r^3 overflows) contribute nothing.
// r2 is a positive normal number (not 0, subnormal, infinite or NaN).
__device__ inline bool positive_normal(double r2) { return __builtin_amdgcn_class(r2, 0x100); }
// The FP32 pair terms' form of the same test (finite r2 at or above FLT_MIN).
constexpr float kFltMin = __FLT_MIN__;
__device__ inline bool positive_normal_f(float r2) { return r2 >= kFltMin; }

// The FP64 sums form a term as (m r^-3) d, two products fewer than m d r^-3 in each
// axis. The factor m r^-3 leaves the number range in places where the term does not
// (m = 1e10 at d = 1e-100). With numbers in the ranges below it is at most 2^930 and, but
// for m = 0, at least 2^-905 wherever r^2 >= kMildEps2Min; other terms are formed by
// pair_term_f64.
constexpr double kMildLength = 0x1p200;  // largest offset
constexpr double kMildEps2 = 0x1p400;    // largest squared softening
constexpr double kMildEps2Min = 0x1p-400;
constexpr double kMildMassMin = 0x1p-300, kMildMassMax = 0x1p300;
__device__ inline bool mild_mass(double m)
{
    return m == 0.0 || (fabs(m) >= kMildMassMin && fabs(m) <= kMildMassMax);
}
// One term in the order that keeps every intermediate result in range with it: adds m d /
// r^3 to s and -m / r to ph if r2 is a positive normal number. Returns whether it is, and
// r^-5 and r^-2 for a quadrupole's term.
template <bool PHI>
__device__ inline bool pair_term_f64(double m, double dx, double dy, double dz, double r2,
                                     double &sx, double &sy, double &sz, double &ph, double &inv5,
                                     double &inv2)
{
    if (!positive_normal(r2)) return false;
    const double rinv = rsqrt_f64(r2);
    inv2 = rinv * rinv;
    const double inv3 = inv2 * rinv;
    inv5 = inv3 * inv2;
    sx += m * dx * inv3;
    sy += m * dy * inv3;
    sz += m * dz * inv3;
    if (PHI) ph -= m * rinv;
    return true;
}

// Workspace owned by a context; sized once for n_max bodies.
struct Workspace {
    int64_t n_cap = 0, node_cap = 0;
    int sort_blocks_cap = 0, max_scenes = 1;
    uint64_t *keys[2] = {nullptr, nullptr};
    uint32_t *idx[2] = {nullptr, nullptr};
    uint32_t *sort_counts = nullptr;  // [256][sort blocks], scanned per digit row
    uint32_t *sort_totals = nullptr;  // [256]
    Body *body = nullptr;             // sorted bodies
    double *beps2 = nullptr;          // sorted eps^2
    // The state of a multi-step call, kept in the Morton order of the last
    // build (body, beps2 and idx[0], the caller index of each sorted body,
    // belong to it): velocities and accelerations in sorted order, and the
    // drifted state before the next sort (same order as the sorted state).
    double *tvel = nullptr;           // [n_cap][3]
    double *tacc = nullptr;           // [n_cap][3]
    Body *sbody = nullptr;            // [n_cap]
    double *svel = nullptr;           // [n_cap][3], after sbody in one allocation
    double *seps2 = nullptr;          // [n_cap], the same
    uint32_t *scidx = nullptr;        // [n_cap]
    NodeInfo *ninfo = nullptr;
    // [inner_words] k_build_subtrees' lists beyond LDS, then the contact search's
    // table: the memory of the drifted state, which nothing reads after the gather
    int32_t *inner = nullptr;
    int64_t inner_words = 0;
    NodeMom *nmom = nullptr;
    double *neps2 = nullptr;
    double *nquad = nullptr;      // [node_cap][6] quadrupoles, only with BH_FLAG_QUAD
    SceneBox *box = nullptr;      // [max_scenes]
    TreeHeader *hdr = nullptr;
    int32_t *counts = nullptr;    // [n_cap][2] per-body walk counts, caller order
    double *scratch = nullptr;    // [n_cap] potential for diagnostics
    double *red_part = nullptr;   // [reduction blocks][8][2] compensated partial sums
    double *dpart = nullptr;      // [kDirectPart] partial direct sums of split source ranges
    // Launch hints of the last build, written by the device into pinned host
    // memory: the words of HintWord. The next build launches the levels down to
    // one below the depth one by one and the rest in one block, or whole subtrees
    // from a level of small nodes on (plan_levels), picks its sort (sort_passes)
    // and how each level is split (by the node counts).
    int32_t *depth_host = nullptr;
    int32_t *depth_dev = nullptr;  // the same memory as the device sees it
    // the ST_* words, kStatusAt words into the same allocation
    uint32_t *status_host = nullptr, *status_dev = nullptr;
    // [kPrefixCells] first sorted body of each level-kPrefixLevels cell, or
    // INT32_MAX ("none"): set at creation, written by one build and restored
    // to "none" by the same build once read.
    int32_t *prefix_mark = nullptr;
};

// The direct sum and its VJP split their sources over block rows when the
// targets alone give too few blocks; each row's partial sums (4 doubles per
// target) go to a workspace buffer of kDirectPart doubles and are added in row
// order. Up to kDirectSmall bodies the direct sum needs no rows.
constexpr int64_t kDirectSmall = 4096;
constexpr int kDirectBlocks = 1024;
constexpr int64_t kDirectPart = (int64_t)kDirectBlocks * 256 * 4;
constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kRedBlocks = 512;

// What a new workspace holds before its first build: empty boxes, a zero header with
// the status words' address, no cell marks, and no parents (an adjoint's table, or
// nullptr: a node that an overflow leaves unlinked has the entry of an earlier build, so
// that there has to be one). On the null stream.
hipError_t launch_init(const Workspace &w, int32_t *nparent);

// The sort that a build enqueued: what bucket_sort_hint gave (0 and false for a
// one-block build).
struct SortUsed {
    bool even = false;
    int passes = 0;
};

// Launchers (tree.hip). All enqueue on `s` and never synchronise; `sort` (if
// given) receives the sort that was enqueued. The build
// launches one kernel per tree level down to one below the depth the
// previous build reported (a host read of pinned memory, frozen in a
// captured graph) and handles deeper levels in one block: any depth is
// built correctly, a deeper one more slowly.
// With `adv`, only for a layout that one block builds (one_block_build): the
// bodies are moved first, in the same launch.
struct Advance {
    double *pos = nullptr, *vel = nullptr;  // caller order; pos: the build's
    const double *acc = nullptr;
    double dt = 0.0;
    int substeps = 0;  // > 0: as launch_euler_substeps; 0: as launch_kick_drift
};
hipError_t launch_build(const Workspace &w, hipStream_t s, const Layout &lay, const double *pos,
                        const double *mass, const double *eps, int leaf, SortUsed *sort = nullptr,
                        const Advance *adv = nullptr);
inline bool one_block_build(const Layout &lay)
{
    return lay.n_scenes == 1 && lay.n >= 1 && lay.n <= kSmallBuild;
}
// The same build for one step on the sorted state (multi-step calls, more
// than kSmallBuild bodies or several scenes): the step's first kick and its
// drift (v = v + dt/2 a, x = x + dt v) run in the bounding-box pass over the
// sorted state of the previous build, and the gather carries velocities,
// softening and caller indices into the new order.
hipError_t launch_build_state(const Workspace &w, hipStream_t s, const Layout &lay, bool use_eps,
                              int leaf, double dt, SortUsed *sort = nullptr);
// How the next build of `lay` sorts, and whether level kHintLevel alone allows it
// (sort_passes): a host read of the pinned hints, frozen in a captured graph. Every
// sort gives the same order; the choice only affects speed.
inline int bucket_sort_hint(const Workspace &w, const Layout &lay, bool *even = nullptr)
{
    bool e;
    return sort_passes(w.depth_host, lay.n, lay.n_scenes, even ? even : &e);
}
// The level from which the next build of `lay` builds whole subtrees in one
// launch, or -1; a host read of the pinned hints like bucket_sort_hint.
inline int subtree_hint(const Workspace &w, const Layout &lay)
{
    return plan_levels(w.depth_host, lay.n, lay.n_scenes).sub;
}
// scene_of[i] = scene of body i, from device offsets of n_scenes scenes
hipError_t launch_scene_of(hipStream_t s, const int64_t *offsets, int n_scenes,
                           uint16_t *scene_of);

struct WalkParams {
    int64_t n;
    const int32_t *groups = nullptr;  // walk groups of a multi-scene layout
    int n_groups = 0;
    double th2;     // theta^2
    double eps0sq;  // uniform softening squared (per-body eps not given)
    double G;
    double *acc;    // caller order, n x 3 (sorted order with acc_sorted)
    double *phi;    // caller order or nullptr (sorted order with acc_sorted)
    bool acc_sorted = false;
    int32_t *counts;  // caller order n x 2 or nullptr
    bool per_body_eps;
    int precision;
    int group;  // target bodies per block: 64, 32 or 16
    const double *nquad = nullptr;  // node quadrupoles: add their terms (or nullptr)
    // velocities (in the order of acc) that the walk kicks by kick_h times the
    // acceleration it writes, as launch_kick does (or nullptr)
    double *kick_vel = nullptr;
    double kick_h = 0.0;
};
constexpr int kDefaultWalkGroup = 64;
constexpr int64_t kSmallWalk = 131072;  // below this many bodies the default group is 16
// walk.hip
hipError_t launch_walk(const Workspace &w, hipStream_t s, const WalkParams &p);

// direct.hip
hipError_t launch_direct(hipStream_t s, const double *pos, const double *mass, const double *eps,
                         int64_t n, double eps0sq, double G, int precision, double *acc,
                         double *phi, double *part);

// adjoint.hip: workspace of the VJPs (BH_FLAG_ADJOINT)
// The trees a checkpointed segment's recomputation builds, one per step, kept
// for the VJPs at the same positions: slot k holds sorted bodies, eps^2,
// caller indices and keys (n each), the node tables (node_cap each), the
// scene box and the tree header of step k.
struct TreeSlots {
    int count = 0;
    int64_t n = 0, node_cap = 0;
    Body *body = nullptr;
    double *beps2 = nullptr;
    uint32_t *idx = nullptr;
    uint64_t *keys = nullptr;
    NodeInfo *ninfo = nullptr;
    NodeMom *nmom = nullptr;
    double *neps2 = nullptr;
    SceneBox *box = nullptr;
    TreeHeader *hdr = nullptr;
};
// A workspace whose tree arrays are slot k's (scratch arrays shared with w).
Workspace slot_view(const Workspace &w, const TreeSlots &t, int k);

struct AdjointWork {
    TreeSlots trees;         // allocated by the first segment VJP that fits in memory
    double *gt = nullptr;    // [n_cap][3] target-side gradients, sorted order
    double *badj = nullptr;  // [n_cap][4] source-side body adjoints, sorted order
    int64_t node_cap = 0;    // of the context's node table
    double *nadj = nullptr;  // [node_cap][4] node adjoints gX, gm, then [node_cap] g<eps^2>
    int32_t *nparent = nullptr;  // [node_cap] parent of each node (-1: the root)
    double *vwork = nullptr; // [n_cap][3] velocity while a segment is recomputed
    double *awork = nullptr; // [n_cap][3] acceleration while a segment is recomputed
};
hipError_t launch_tree_vjp(const Workspace &w, const AdjointWork &aw, hipStream_t s,
                           const WalkParams &p, const double *lambda, double *g_pos,
                           double *g_mass);
hipError_t launch_direct_vjp(hipStream_t s, const double *pos, const double *mass,
                             const double *eps, int64_t n, double eps0sq, double G,
                             const double *lambda, double *g_pos, double *g_mass, double *part);
hipError_t launch_adj_kick(hipStream_t s, double *abar, const double *vbar, int64_t n, double dt);
hipError_t launch_adj_drift_kick(hipStream_t s, double *vbar, double *abar, const double *xbar,
                                 int64_t n, double dt);
hipError_t launch_kick_drift_to(hipStream_t s, const double *x_in, double *v, const double *a,
                                double *x_out, int64_t n, double dt);
hipError_t launch_copy(hipStream_t s, double *dst, const double *src, int64_t count);

// integrate.hip
hipError_t launch_kick_drift(hipStream_t s, double *pos, double *vel, const double *acc, int64_t n,
                             double dt);
// contacts.hip: contact components of the bodies of the last build (label
// in caller order, size: n int32 scratch, counters: 3 device words).
hipError_t launch_contacts(const Workspace &w, hipStream_t s, const double *radius, int64_t n,
                           double skin, int32_t *label, int32_t *size,
                           unsigned long long *counters);
hipError_t launch_euler_substeps(hipStream_t s, double *pos, double *vel, const double *acc,
                                 int64_t n, double dt, int k);
hipError_t launch_kick(hipStream_t s, double *vel, const double *acc, int64_t n, double dt);
// The sorted state of a multi-step call from the caller's arrays (identity
// order; checks masses and softening lengths, flagging ST_NONFINITE), and
// back to them at its end.
hipError_t launch_state_pack(const Workspace &w, hipStream_t s, const double *pos,
                             const double *vel, const double *acc, const double *mass,
                             const double *eps, int64_t n, uint32_t *status);
hipError_t launch_state_unpack(const Workspace &w, hipStream_t s, double *pos, double *vel,
                               double *acc, int64_t n);
// Largest body density m / ((4/3) pi r^3) over the massive bodies and the
// gravity time-step bound 1 / (2 sqrt(G rho)) of eq. (dt_g) into out[0]
// (+inf with no massive body); work[0] is scratch; bad input sets ST_NONFINITE.
hipError_t launch_dt_bound(hipStream_t s, const double *mass, const double *radius, int64_t n,
                           double G, long long *work, double *out, uint32_t *status);
hipError_t launch_diag_reduce(hipStream_t s, const double *pos, const double *vel,
                              const double *mass, const double *phi, int64_t n, double *part,
                              double *out8_device);

}  // namespace bhx
