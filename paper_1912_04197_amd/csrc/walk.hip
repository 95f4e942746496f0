// Barnes-Hut walk (subsection "Force computation"): one block serves a group
// of GB Morton-consecutive target bodies (GB = 64, 32 or 16); one of its
// wavefronts walks the tree and three others evaluate, with 64 / GB lanes per body.
//
// The paper gives each body its own thread and its own traversal. Here the
// lanes of a wave walk the tree together, but every stack entry carries a
// GB-bit body mask: the bodies whose own traversal reaches that node. At an
// internal node each body evaluates its own opening test in FP64
// (s^2 < theta^2 D^2, eq. accuracy); the bodies that accept it take the node
// as one interaction (eq. Force_thetaTrue) and the others carry on into the
// children. A leaf contributes its bodies one by one (eq. Force_leaf) to the
// bodies that reached it, each body's own index cleared from its mask. So each
// body gets exactly the interaction set of its own walk; only the summation
// order differs from a depth-first walk. walk_traverse.h holds the traversal
// and the queue of interactions between it and the evaluating waves.
//
// Evaluation: the interaction queue holds descriptors (a leaf's body range or
// one accepted node, with a body mask). An evaluating wave takes 64 items at a
// time; lane k loads item k. An item that reaches more than GB / 6 bodies of
// the group is dense: the dense items are staged in LDS and the lanes of each
// body sweep them, each taking every (64 / GB)-th one. A sparse item becomes
// (item, body) pairs, one pair per lane, whose terms are added into per-body
// FP64 sums in LDS; most leaf bodies near the group's edge reach only a few of
// its bodies, and a sweep would leave most lanes idle on them. In FP32C mode
// each pair offset x_j - x_B is formed in FP64 and rounded once to FP32 (close
// pairs keep full FP32 precision whatever the group's extent), the rest of the
// pair term is FP32, and in the sweep FP32 partial sums over at most 16 items
// per lane are added into FP64 accumulators. The per-lane FP64 sums of a body
// and its pair sums are added at the end, wave by wave in a fixed order; the
// pair sums are LDS atomics of a single wave, applied in a fixed order, so
// results are deterministic.
#include <cstddef>
#include <type_traits>

#include "bhx_impl.h"
#include "walk_traverse.h"

namespace bhx {
namespace {

using walkx::kBatch;
using walkx::kEvals;
constexpr int kStack = 256;    // LDS traversal stack of child ranges
constexpr int kFlush = 16;     // FP32 partial sums span at most this many items per lane
constexpr int kPairCap = 448;  // body pairs evaluated one per lane in one batch
constexpr int kSweepUnroll = 4;  // items per unrolled step of an FP32C dense sweep

struct alignas(16) ItemF {  // FP32C staged source
    double x, y, z;
    float m;
    float e2h;  // half of the source's squared softening
};
struct alignas(16) ItemD {  // FP64 staged source
    double x, y, z, m;
};

// The LDS address of p as one register, so that the loads of an unrolled sweep
// are one address with immediate offsets (the compiler would compute each of
// them by an addition of its own).
template <typename T>
using LdsPtr = const __attribute__((address_space(3))) T *;
template <typename T>
__device__ inline LdsPtr<T> lds_base(const T *p)
{
    LdsPtr<T> q = (LdsPtr<T>)p;
    asm("" : "+v"(q));
    return q;
}

// What one evaluating wave works in.
template <int PREC, bool PEPS, bool PHI, bool CNT, int GB, bool QUAD>
struct EvalLds {
    // slots past kBatch are read, never used: a sweep's last step reads a slot
    // for every share of lanes
    static constexpr int kSlots = kBatch + 64 / GB - 1;
    using Item = typename std::conditional<PREC == BH_FP64, ItemD, ItemF>::type;
    using QT = typename std::conditional<PREC == BH_FP64, double, float>::type;
    Item items[kSlots];      // dense items first, then the sparse ones
    uint64_t mask[kSlots];   // bodies that take the item
    double e2h[PREC == BH_FP64 && PEPS ? kSlots : 1];  // half eps_j^2 or <eps^2>_N
    int32_t src[CNT || QUAD ? kSlots : 1];             // sorted body index, or ~node
    QT quad[QUAD ? 6 * kSlots : 1];                    // node items' quadrupoles
    uint16_t rec[kPairCap];  // pair: item slot << 6 | body
    double pacc[3 * GB];     // pair sums per body: x, y, z; at the end the wave's sums
    double pphi[PHI ? GB : 1];
    int32_t pcnt[CNT ? 2 * GB : 1];
};
// Quadrupole term of an accepted node with traceless Q (xx, yy, zz, xy, xz,
// yz), d = COM - x_B, inv5 = 1/r^5 and ri2 = 1/r^2 of the softened distance:
// a += -Q d / r^5 + 5/2 (d.Q d) d / r^7 and phi += -(d.Q d) / (2 r^5), before
// the factor G.
template <typename T>
__device__ inline void quad_term(const T *Q, T dx, T dy, T dz, T inv5, T ri2, T &ax, T &ay, T &az,
                                 T &ph)
{
    const T qx = Q[0] * dx + Q[3] * dy + Q[4] * dz;
    const T qy = Q[3] * dx + Q[1] * dy + Q[5] * dz;
    const T qz = Q[4] * dx + Q[5] * dy + Q[2] * dz;
    const T dqd = dx * qx + dy * qy + dz * qz;
    const T c = T(2.5) * dqd * inv5 * ri2;
    ax += c * dx - qx * inv5;
    ay += c * dy - qy * inv5;
    az += c * dz - qz * inv5;
    ph -= T(0.5) * dqd * inv5;
}

template <int PREC, bool PEPS, bool PHI, bool CNT, int GB, bool QUAD>
__global__ __launch_bounds__(64 * (1 + kEvals)) void k_walk(
    const Body *__restrict__ body, const double *__restrict__ beps2,
    const NodeInfo *__restrict__ ninfo, const NodeMom *__restrict__ nmom,
    const double *__restrict__ neps2, const double *__restrict__ nquad,
    const uint32_t *__restrict__ idx,
    const SceneBox *__restrict__ box, const int32_t *__restrict__ groups, int64_t n,
    int ngroups, int per_xcd, double th2, double eps0sq, double G,
    double *__restrict__ acc, double *__restrict__ phi, int32_t *__restrict__ counts,
    bool acc_sorted, double *__restrict__ kick_vel, double kick_h)
{
    static_assert(GB == 64 || GB == 32 || GB == 16, "group size");
    constexpr int LPB = 64 / GB;  // lanes per body
    constexpr uint64_t kBodyMask = GB == 64 ? ~0ull : ((1ull << GB) - 1ull);
    using EL = EvalLds<PREC, PEPS, PHI, CNT, GB, QUAD>;

    // Items that reach at most kSparse bodies of the group are evaluated as
    // (item, body) pairs, one pair per lane, into per-body FP64 sums in LDS.
    constexpr int kSparse = GB / 6;

    __shared__ walkx::Lds<kStack> L;
    __shared__ EL eval_lds[kEvals];

    // Blocks are dealt to the 8 XCDs round-robin. One scene: give each XCD a
    // contiguous (so spatially compact) range of groups to share its L2. A
    // group table (several scenes) is already in dealing order, costliest
    // first (per_xcd = 0): block b takes group b.
    const int grp = per_xcd ? (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3)
                            : (int)blockIdx.x;
    if (grp >= ngroups) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int bq = GB == 64 ? lane : lane % GB;  // body of this lane within the group
    const int sub = GB == 64 ? 0 : lane / GB;    // which share of the items it sweeps
    // the group: up to GB consecutive sorted bodies of one scene
    int64_t g0 = (int64_t)grp * GB;
    int gcount = (int)min((int64_t)GB, n - g0);
    int scene = 0;
    if (groups) {
        g0 = groups[3 * grp];
        gcount = groups[3 * grp + 1];
        scene = groups[3 * grp + 2];
    }
    const int64_t s = g0 + bq;
    const bool valid = bq < gcount;
    const Body me = body[valid ? s : g0];

    if (threadIdx.x == 0) L.published = 0;
    if (threadIdx.x < kEvals) L.head[threadIdx.x] = 0;
    __syncthreads();

    if (wave == 0) {
        // the group's bounding box (exact: min and max of its bodies' coordinates)
        double glo[3], ghi[3];
        walkx::group_box<GB>(valid, me.x, me.y, me.z, glo, ghi);
        const uint64_t active = __ballot(valid) & kBodyMask;
        // the scene's root is node `scene`
        walkx::traverse<GB>(L, scene, active, ninfo, nmom, walkx::SideSq(box[scene]), glo, ghi,
                            me.x, me.y, me.z, th2);
    } else {
        EL &sh = eval_lds[wave - 1];
        double *const pacc = sh.pacc;
        double *const pphi = sh.pphi;
        int32_t *const pcnt = sh.pcnt;
        const double eb2 = PEPS ? beps2[valid ? s : g0] : 0.0;
        const double ebh = 0.5 * eb2;  // (eps_B^2 + e_j^2) / 2 = ebh + e_j^2 / 2 exactly
        const float e2hB = (float)ebh;
        const float eps0f = (float)eps0sq;
        // every body of the wave has a positive FP32 softening (the sweep's r^2 > 0 test is moot)
        const bool soft_all =
            __ballot(!valid || positive_normal_f(PEPS ? e2hB : eps0f)) == ~0ull;
        const int woff = bq >= 32 ? 1 : 0;
        const CubeConsts cc = cube_consts();
        // FP64: no factor m r^-3 is out of range while r^2 >= kMildEps2Min, and every
        // pair is softened that far. Such waves test no term; the others, whose rare
        // loops cost the batch registers, have code of their own.
        // (softened, 100,000 bodies of a rubble pile at leaf 8: 398 us with a test
        // of every term for a positive normal r^2, 384 without; unsoftened, 50,000 of
        // a ball: 158 before, 160 with the terms outside the range kept.)
        const bool mild = PREC == BH_FP64 && box[scene].mild != 0 &&
                          (PEPS || eps0sq <= kMildEps2);
        const bool mild_soft = mild && (PEPS ? __ballot(!(ebh >= kMildEps2Min)) == 0
                                             : eps0sq >= kMildEps2Min);

        double ax = 0.0, ay = 0.0, az = 0.0, ph = 0.0;
        int32_t cnode = 0, cpair = 0;
        // finite numbers in slots that a sweep reads before any item was staged there
        for (int i = lane; i < EL::kSlots; i += 64) {
            sh.items[i] = typename EL::Item{};
            if (PREC == BH_FP64 && PEPS) sh.e2h[PREC == BH_FP64 && PEPS ? i : 0] = 0.0;
            if (CNT || QUAD) sh.src[CNT || QUAD ? i : 0] = 0;
        }
        for (int i = lane; i < 3 * GB; i += 64) pacc[i] = 0.0;
        if (PHI && lane < GB) pphi[lane] = 0.0;
        if (CNT)
            for (int i = lane; i < 2 * GB; i += 64) pcnt[i] = 0;

        // Stages the batch and evaluates it: the dense items by a sweep of the
        // lanes of each body, the sparse ones as pairs. `plain`: mild_soft.
        auto evaluate = [&](auto plain, walkx::Batch &bt) {
            constexpr bool kPlain = decltype(plain)::value;
            const int c = bt.count;
            // Load item `lane` and its body mask; the split below decides where
            // in LDS it goes.
            uint64_t mk;
            int32_t src;
            walkx::take_batch(L, wave - 1, bt, src, mk);
            double x = 0.0, y = 0.0, z = 0.0, m = 0.0, e2 = 0.0;
            double qn[QUAD ? 6 : 1] = {};
            if (lane < c) {
                if (src >= 0) {
                    if (!check_ok(src < n, CK_INDEX)) src = 0;
                    const int64_t rel = (int64_t)src - g0;
                    if (rel >= 0 && rel < GB) mk &= ~(1ull << rel);  // not itself
                    const Body b = body[src];
                    x = b.x, y = b.y, z = b.z, m = b.m;
                    e2 = PEPS ? beps2[src] : 0.0;
                } else {
                    const NodeMom nm = nmom[~src];
                    x = nm.x, y = nm.y, z = nm.z, m = nm.m;
                    e2 = PEPS ? neps2[~src] : 0.0;
                    if constexpr (QUAD)
                        for (int t = 0; t < 6; t++) qn[t] = nquad[6 * (int64_t)(~src) + t];
                }
            }
            // Split the batch: an item reaching at most kSparse bodies becomes
            // that many (item, body) pairs while they fit in the pair list; the
            // others are dense and go to slots 0..nd-1, the sparse ones after.
            const int pk = __popcll(mk);
            const bool sparse = lane < c && pk <= kSparse;
            const uint32_t pv = sparse ? (uint32_t)pk : 0u;
            const uint32_t pend = wave_incl_scan(pv);
            const bool fits = sparse && pend <= (uint32_t)kPairCap;
            const bool dense = lane < c && !fits;
            const uint64_t db = __ballot(dense);
            const uint64_t fb = __ballot(fits && pk > 0);
            const int nd = __popcll(db);
            const int np = fb ? __builtin_amdgcn_readlane((int)pend, 63 - __builtin_clzll(fb)) : 0;
            BHX_CHECK(np <= kPairCap, CK_PAIRS);
            if (dense || (fits && pk > 0)) {
                const int slot = dense ? (int)lanes_below(db) : nd + (int)lanes_below(fb);
                if constexpr (PREC == BH_FP64) {
                    sh.items[slot] = ItemD{x, y, z, m};
                    if (PEPS) sh.e2h[slot] = 0.5 * e2;
                } else {
                    sh.items[slot] = ItemF{x, y, z, (float)m, (float)(0.5 * e2)};
                }
                sh.mask[slot] = mk;
                if (CNT || QUAD) sh.src[slot] = src;
                if constexpr (QUAD)
                    if (src < 0)
                        for (int t = 0; t < 6; t++)
                            sh.quad[6 * slot + t] = (typename EL::QT)qn[t];
                if (fits) {
                    uint64_t bits = mk;
                    uint32_t at = pend - pv;
                    while (bits) {
                        sh.rec[at++] = (uint16_t)(slot << 6 | __builtin_ctzll(bits));
                        bits &= bits - 1;
                    }
                }
            }
            walkx::wave_sync();
            // One FP64 term of a source on a target, nothing unless `on` and (not
            // kPlain) r^2 is large enough for its factor; otherwise `lost` is set.
            // (nothing is tried where !mild: offsets may be infinite)
            bool lost = !kPlain && !mild;
            const int nd_try = kPlain || PREC != BH_FP64 || mild ? nd : 0;
            const int np_try = kPlain || PREC != BH_FP64 || mild ? np : 0;
            constexpr double near = kMildEps2Min;
            auto term64 = [&](const ItemD &it, double bx, double by, double bz, double e2, bool on,
                              bool node, int j, double &sx, double &sy, double &sz, double &sp) {
                const double dx = it.x - bx, dy = it.y - by, dz = it.z - bz;
                const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, e2)));
                bool live = on;
                if constexpr (!kPlain) {
                    live = on && r2 >= near;
                    lost = lost || (on && !live);
                }
                double ri = 0.0, i2 = 0.0, i3;
                if constexpr (QUAD)
                    i3 = inv_cube_sq_f64<PHI>(r2, i2, ri, cc);
                else
                    i3 = inv_cube_f64<PHI>(r2, ri, cc);
                const double c3 = live ? it.m * i3 : 0.0;
                sx = fma(c3, dx, sx);
                sy = fma(c3, dy, sy);
                sz = fma(c3, dz, sz);
                if (PHI) sp = fma(-it.m, live ? ri : 0.0, sp);
                if constexpr (QUAD && PREC == BH_FP64)
                    if (node && live) {
                        const double *Q = sh.quad + 6 * j;
                        quad_term(Q, dx, dy, dz, i3 * i2, i2, sx, sy, sz, sp);
                    }
            };
            if constexpr (PREC == BH_FP64) {
                // jj is the same on every lane; lane share `sub` takes item jj + sub
                LdsPtr<ItemD> ip = lds_base(sh.items + sub);
                LdsPtr<uint64_t> mp = lds_base(sh.mask + sub);
#pragma unroll 2
                for (int jj = 0; jj < nd_try; jj += LPB) {
                    const int j = jj + sub;  // past nd: a slot that is not taken
                    const ItemD it = ItemD{ip[jj].x, ip[jj].y, ip[jj].z, ip[jj].m};
                    const bool on = j < nd && ((mp[jj] >> bq) & 1ull);
                    const bool node = (CNT || QUAD) && sh.src[CNT || QUAD ? j : 0] < 0;
                    const double es = PEPS ? ebh + sh.e2h[PEPS ? j : 0] : eps0sq;
                    term64(it, me.x, me.y, me.z, es, on, node, j, ax, ay, az, ph);
                    if (CNT && on) {
                        if (node)
                            cnode++;
                        else
                            cpair++;
                    }
                }
            } else {
              // With every body of the wave softened (its FP32 half eps^2 a normal
              // number), r^2 >= that softening for every pair, so r^2 is a
              // positive normal number and the test is dropped.
              auto sweep = [&](auto all_soft) {
#pragma unroll 1
                for (int j0 = 0; j0 < nd; j0 += kFlush * LPB) {
                    const int jn = min(nd, j0 + kFlush * LPB);
                    float fx = 0.f, fy = 0.f, fz = 0.f, fp = 0.f;
                    // jj is the same on every lane; lane share `sub` takes item jj + sub
                    LdsPtr<ItemF> ip = lds_base(sh.items + sub);
                    // lanes 32..63 of a 64-body group read the high words of the masks
                    LdsPtr<uint32_t> mp = lds_base((const uint32_t *)(sh.mask + sub) + woff);
#pragma unroll kSweepUnroll
                    for (int jj = j0; jj < jn; jj += LPB) {
                        const int j = jj + sub;  // past jn: a slot that is not taken
                        const float qm = ip[jj].m, qe = ip[jj].e2h;
                        const float dx = (float)(ip[jj].x - me.x), dy = (float)(ip[jj].y - me.y),
                                    dz = (float)(ip[jj].z - me.z);
                        const float e2 = PEPS ? qe + e2hB : eps0f;
                        const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, e2)));
                        // all ones where the body takes the item, else 0
                        int32_t on = __builtin_amdgcn_sbfe((int)mp[2 * jj], bq & 31, 1);
                        if (GB != 64) on = j < jn ? on : 0;
                        float rinv = __int_as_float(
                            __float_as_int(__builtin_amdgcn_rsqf(r2)) & on);
                        if (!decltype(all_soft)::value) rinv = positive_normal_f(r2) ? rinv : 0.f;
                        const float mr = qm * rinv;
                        const float mr3 = mr * rinv * rinv;
                        fx = fmaf(mr3, dx, fx);
                        fy = fmaf(mr3, dy, fy);
                        fz = fmaf(mr3, dz, fz);
                        if (PHI) fp -= mr;
                        const bool node = (CNT || QUAD) && sh.src[CNT || QUAD ? j : 0] < 0;
                        if constexpr (QUAD)
                            if (node) {
                                const float ri2 = rinv * rinv;
                                quad_term(sh.quad + 6 * j, dx, dy, dz, ri2 * ri2 * rinv, ri2, fx,
                                          fy, fz, fp);
                            }
                        if (CNT && on) {
                            if (node)
                                cnode++;
                            else
                                cpair++;
                        }
                    }
                    ax += (double)fx;
                    ay += (double)fy;
                    az += (double)fz;
                    if (PHI) ph += (double)fp;
                }
              };
              if (soft_all)
                  sweep(std::true_type{});
              else
                  sweep(std::false_type{});
            }
            // Pairs: lane i takes pair i of the list; its body's coordinates come
            // from that body's lane. Each pair term goes into the body's FP64 sums.
            auto add_pair = [&](int b, double fx, double fy, double fz, double fp) {
                __hip_atomic_fetch_add(&pacc[3 * b], fx, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(&pacc[3 * b + 1], fy, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(&pacc[3 * b + 2], fz, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                if (PHI)
                    __hip_atomic_fetch_add(&pphi[b], fp, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            };
#pragma unroll 1
            for (int i0 = 0; i0 < np_try; i0 += 64) {
                const int i = i0 + lane;
                const bool on = i < np;
                const uint32_t r = sh.rec[on ? i : i0];
                const int k = (int)(r >> 6), b = (int)(r & 63u);
                const double tx = __shfl(me.x, b), ty = __shfl(me.y, b), tz = __shfl(me.z, b);
                const bool node = (CNT || QUAD) && sh.src[CNT || QUAD ? k : 0] < 0;
                double fx = 0.0, fy = 0.0, fz = 0.0, fp = 0.0;
                if constexpr (PREC == BH_FP64) {
                    const double te = PEPS ? __shfl(ebh, b) : 0.0;
                    const double es = PEPS ? te + sh.e2h[PEPS ? k : 0] : eps0sq;
                    term64(sh.items[k], tx, ty, tz, es, on, node, k, fx, fy, fz, fp);
                } else {
                    const float te = PEPS ? __shfl(e2hB, b) : 0.f;
                    const ItemF it = sh.items[k];
                    const float dx = (float)(it.x - tx), dy = (float)(it.y - ty),
                                dz = (float)(it.z - tz);
                    const float e2 = PEPS ? it.e2h + te : eps0f;
                    const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, e2)));
                    const float rinv =
                        (on && positive_normal_f(r2)) ? __builtin_amdgcn_rsqf(r2) : 0.f;
                    const float mr = it.m * rinv;
                    const float mr3 = mr * rinv * rinv;
                    float gxf = mr3 * dx, gyf = mr3 * dy, gzf = mr3 * dz, gpf = -mr;
                    if constexpr (QUAD)
                        if (node) {
                            const float ri2 = rinv * rinv;
                            quad_term(sh.quad + 6 * k, dx, dy, dz, ri2 * ri2 * rinv, ri2, gxf, gyf,
                                      gzf, gpf);
                        }
                    fx = (double)gxf;
                    fy = (double)gyf;
                    fz = (double)gzf;
                    if (PHI) fp = (double)gpf;
                }
                if (on) {
                    add_pair(b, fx, fy, fz, fp);
                    if (CNT)
                        __hip_atomic_fetch_add(&pcnt[2 * b + (node ? 0 : 1)], 1, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            // the terms that are not in the sums yet, one by one
            if constexpr (PREC == BH_FP64 && !kPlain) {
                if (__ballot(lost) != 0) {
                    auto left = [&](const auto &it, int k, const Body &t, double th, double &sx,
                                    double &sy, double &sz, double &sp) {
                        const double dx = it.x - t.x, dy = it.y - t.y, dz = it.z - t.z;
                        const double r2 = fma(
                            dx, dx, fma(dy, dy, fma(dz, dz, PEPS ? th + sh.e2h[PEPS ? k : 0] : eps0sq)));
                        if (mild && r2 >= near) return;
                        double i5, i2;
                        const bool live =
                            pair_term_f64<PHI>(it.m, dx, dy, dz, r2, sx, sy, sz, sp, i5, i2);
                        if constexpr (QUAD && PREC == BH_FP64)
                            if (live && sh.src[k] < 0)
                                quad_term(sh.quad + 6 * k, dx, dy, dz, i5, i2, sx, sy, sz, sp);
                    };
#pragma unroll 1
                    for (int j = sub; j < nd; j += LPB) {
                        if (!((sh.mask[j] >> bq) & 1ull)) continue;
                        left(sh.items[j], j, me, ebh, ax, ay, az, ph);
                        if (CNT && !mild) {
                            if (sh.src[CNT ? j : 0] < 0)
                                cnode++;
                            else
                                cpair++;
                        }
                    }
#pragma unroll 1
                    for (int i = lane; i < np; i += 64) {
                        const int k = sh.rec[i] >> 6, b = sh.rec[i] & 63;
                        double fx = 0.0, fy = 0.0, fz = 0.0, fp = 0.0;
                        left(sh.items[k], k, body[g0 + b], PEPS ? 0.5 * beps2[g0 + b] : 0.0, fx, fy, fz, fp);
                        add_pair(b, fx, fy, fz, fp);
                        if (CNT && !mild)
                            __hip_atomic_fetch_add(&pcnt[2 * b + (sh.src[CNT ? k : 0] < 0 ? 0 : 1)],
                                                   1, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
            walkx::wave_sync();
        };

        walkx::Batch bt;
        bt.start = (uint32_t)(kBatch * (wave - 1));
        if (PREC == BH_FP64 && mild_soft)
            while (walkx::next_batch(L, wave - 1, bt)) evaluate(std::true_type{}, bt);
        else
            while (walkx::next_batch(L, wave - 1, bt)) evaluate(std::false_type{}, bt);

        // add the lanes' partial sums of each body in a fixed order
#pragma unroll
        for (int o = GB; o < 64; o <<= 1) {
            ax += __shfl_xor(ax, o);
            ay += __shfl_xor(ay, o);
            az += __shfl_xor(az, o);
            if (PHI) ph += __shfl_xor(ph, o);
            if (CNT) {
                cnode += __shfl_xor(cnode, o);
                cpair += __shfl_xor(cpair, o);
            }
        }
        if (sub == 0) {  // then the pair sums
            pacc[3 * bq] += ax;
            pacc[3 * bq + 1] += ay;
            pacc[3 * bq + 2] += az;
            if (PHI) pphi[bq] += ph;
            if (CNT) {
                pcnt[2 * bq] += cnode;
                pcnt[2 * bq + 1] += cpair;
            }
        }
    }
    __syncthreads();
    // the waves' sums in wave order
    if (wave != 1 || !valid || sub != 0) return;
    double ax = 0.0, ay = 0.0, az = 0.0, ph = 0.0;
    int32_t cnode = 0, cpair = 0;
    for (int e = 0; e < kEvals; e++) {
        const EL &sh = eval_lds[e];
        ax += sh.pacc[3 * bq];
        ay += sh.pacc[3 * bq + 1];
        az += sh.pacc[3 * bq + 2];
        if (PHI) ph += sh.pphi[PHI ? bq : 0];
        if (CNT) {
            cnode += sh.pcnt[CNT ? 2 * bq : 0];
            cpair += sh.pcnt[CNT ? 2 * bq + 1 : 0];
        }
    }
    const int64_t o = idx[s];
    const int64_t oa = acc_sorted ? s : o;  // where acc and phi go
    const double a[3] = {G * ax, G * ay, G * az};
    for (int k = 0; k < 3; k++) acc[3 * oa + k] = a[k];
    if (kick_vel)
        for (int k = 0; k < 3; k++) kick_vel[3 * oa + k] = fma(kick_h, a[k], kick_vel[3 * oa + k]);
    if (PHI) phi[oa] = G * ph;
    if (CNT) {
        counts[2 * o] = cnode;
        counts[2 * o + 1] = cpair;
    }
}

template <int PREC, bool PEPS, bool PHI, bool CNT, int GB, bool QUAD>
hipError_t launch_t(const Workspace &w, hipStream_t s, const WalkParams &p)
{
    const int ngroups = p.groups ? p.n_groups : (int)((p.n + GB - 1) / GB);
    const int per_xcd = p.groups ? 0 : (ngroups + 7) / 8;
    if (ngroups == 0) return hipSuccess;
    k_walk<PREC, PEPS, PHI, CNT, GB, QUAD>
        <<<p.groups ? ngroups : 8 * per_xcd, 64 * (1 + kEvals), 0, s>>>(
            w.body, w.beps2, w.ninfo, w.nmom, w.neps2, p.nquad, w.idx[0], w.box, p.groups, p.n,
            ngroups, per_xcd, p.th2, p.eps0sq, p.G, p.acc, p.phi, p.counts, p.acc_sorted,
            p.kick_vel, p.kick_h);
    return hipGetLastError();
}

template <int PREC, bool PEPS, bool PHI, bool CNT>
hipError_t launch_g(const Workspace &w, hipStream_t s, const WalkParams &p)
{
    switch (p.group) {
        case 64:
            return p.nquad ? launch_t<PREC, PEPS, PHI, CNT, 64, true>(w, s, p)
                           : launch_t<PREC, PEPS, PHI, CNT, 64, false>(w, s, p);
        case 32:
            return p.nquad ? launch_t<PREC, PEPS, PHI, CNT, 32, true>(w, s, p)
                           : launch_t<PREC, PEPS, PHI, CNT, 32, false>(w, s, p);
        default:
            return p.nquad ? launch_t<PREC, PEPS, PHI, CNT, 16, true>(w, s, p)
                           : launch_t<PREC, PEPS, PHI, CNT, 16, false>(w, s, p);
    }
}

template <int PREC, bool PEPS>
hipError_t launch_p(const Workspace &w, hipStream_t s, const WalkParams &p)
{
    const bool phi = p.phi != nullptr, cnt = p.counts != nullptr;
    if (phi && cnt) return launch_g<PREC, PEPS, true, true>(w, s, p);
    if (phi) return launch_g<PREC, PEPS, true, false>(w, s, p);
    if (cnt) return launch_g<PREC, PEPS, false, true>(w, s, p);
    return launch_g<PREC, PEPS, false, false>(w, s, p);
}

}  // namespace

BHX_DEFINE_TAKE_CHECKS(walk_take_checks)

hipError_t launch_walk(const Workspace &w, hipStream_t s, const WalkParams &p)
{
    if (p.n <= 0) return hipSuccess;
    if (p.precision == BH_FP64)
        return p.per_body_eps ? launch_p<BH_FP64, true>(w, s, p)
                              : launch_p<BH_FP64, false>(w, s, p);
    return p.per_body_eps ? launch_p<BH_FP32C, true>(w, s, p) : launch_p<BH_FP32C, false>(w, s, p);
}

}  // namespace bhx
