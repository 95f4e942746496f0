// Vector-Jacobian products of the force map (the gradient of
// sum_i lambda_i . a_i with respect to positions and masses), with the tree
// and every opening decision held fixed, and the elementwise parts of the
// kick-drift-kick adjoint.
//
// For one softened term t = G m_s d / r^3 (d = X_s - x_i, r^2 = |d|^2 + e2)
// and the target's upstream lambda:
//   dt/dd = G m_s K, K = I / r^3 - 3 d d^T / r^5   (x_i gets -K lambda, X_s +K lambda)
//   dt/dm_s = G d / r^3,   dt/de2 = -3/2 G m_s d / r^5.
// A node source passes its adjoints to its members through its centre of mass
// X_N = sum m_j x_j / m_N, its mass m_N = sum m_j and its mass-weighted
// softening <eps^2>_N = sum m_j eps_j^2 / m_N.
//
// Tree VJP, on the GPU:
//   1. the same build as the forward evaluation (deterministic, so the same
//      tree and decisions);
//   2. a walk with the forward walk's traversal and decisions (one block per
//      group of Morton-consecutive targets, one wave traversing and the others
//      evaluating, staged items split into dense items and pairs); each target's terms are
//      summed in registers and LDS, each source's terms are summed over the
//      group and added with FP64 atomics into the body or node adjoints;
//   3. node adjoints become per-node coefficients (A = gX / m_N,
//      E = ge2 / m_N, C = gm - X.A - <eps^2> E), summed from the root down
//      over each leaf's ancestors (found through a parent table);
//   4. per body: g_x += m_j sum A, g_m += sum C + x_j . sum A + eps_j^2 sum E,
//      plus its own target and source terms, added into the caller's arrays.
// Source-side atomics make the last bits of the gradients order-dependent.
#include <type_traits>

#include "bhx_impl.h"
#include "walk_traverse.h"

namespace bhx {
namespace {

using walkx::kBatch;
using walkx::kEvals;
constexpr int kStack = 320;

struct alignas(16) ItemV {  // staged source
    double x, y, z, m;
    double e2;      // source's squared softening (eps_j^2 or <eps^2>_N)
    uint64_t mask;
    int32_t src;    // sorted body index, or ~node
    float gm;       // G m rounded to FP32 (FP32C terms)
    float e2h;      // half the squared softening rounded to FP32 (FP32C terms)
    int32_t pad;
};
// Lane exchanges inside a row of 16 lanes (DPP): quad_perm [1,0,3,2] is
// lane ^ 1, quad_perm [2,3,0,1] is lane ^ 2, row_ror:4 and row_ror:8 rotate
// the row by 4 and 8 lanes.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128;
template <int CTRL>
__device__ inline double dpp(double v)
{
    const uint64_t u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
template <int CTRL>
__device__ inline float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

constexpr int kPairCap = 448;  // pairs per batch

// What one evaluating wave works in.
template <int GB>
struct EvalLds {
    ItemV items[kBatch];        // dense items first, then the sparse ones
    double sacc[5 * kBatch];    // pair source-side sums per staged item
    double tacc[3 * GB];        // pair target-side sums per body; at the end the wave's sums
    uint16_t rec[kPairCap];     // pair: item slot << 6 | body
};

// badj: per sorted body {gX x, y, z, gm}; nadj: per node the same; nadj_e: per
// node ge2.
//
// The traversal and the opening decisions are those of the forward walk. A
// staged batch is split like the forward walk's: a dense item (reaching
// more than kSparse of the group's bodies) is swept by the lanes of its
// bodies, eight items at a time; each lane takes the eight in an order set by
// its lane bits so that three halving exchanges (lane ^ 1, ^ 2, ^ 32) leave
// lane L with one item's source-side terms summed over eight lanes, and three
// more (rotations by 4 and 8 inside a row, lane ^ 16) complete the sum over
// the group. Then one lane permute puts the four components of each item on
// four neighbouring lanes, and one FP64 atomic per lane adds them to the item's
// adjoints, which lie together: a request for each item instead of one for each
// component (the atomics bound this kernel: with a component per instruction and
// eight lanes active, 40,000 bodies took 458 us, now 215). A sparse item
// becomes (item, body) pairs, one per lane, whose target-side terms go to
// per-body and whose source-side terms go to per-item FP64 sums in LDS, flushed
// to the adjoints once per batch, four lanes an item.
template <bool PEPS, int GB, bool F32>
__global__ __launch_bounds__(64 * (1 + kEvals)) void k_vjp_walk(
    const Body *__restrict__ body, const double *__restrict__ beps2,
    const NodeInfo *__restrict__ ninfo, const NodeMom *__restrict__ nmom,
    const double *__restrict__ neps2, const uint32_t *__restrict__ idx,
    const SceneBox *__restrict__ box, int64_t n, int ngroups, int per_xcd, double th2,
    double eps0sq, double G, const double *__restrict__ lambda, double *__restrict__ gt,
    double *__restrict__ badj, double *__restrict__ nadj, double *__restrict__ nadj_e)
{
    static_assert(GB == 64 || GB == 32 || GB == 16, "group size");
    constexpr int NC = PEPS ? 5 : 4;  // source-side components: gX (3), gm, g<eps^2>
    constexpr int LPB = 64 / GB;      // lanes per body
    constexpr uint64_t kBodyMask = GB == 64 ? ~0ull : ((1ull << GB) - 1ull);
    constexpr int kSparse = GB / 4;   // items reaching at most this many bodies go to pair mode
    // FP32C: every term in FP32 from the FP64 offset rounded once, the terms
    // of a step summed in FP32 and added into FP64 sums and adjoints
    using VT = typename std::conditional<F32, float, double>::type;
    __shared__ walkx::Lds<kStack> L;
    __shared__ EvalLds<GB> eval_lds[kEvals];

    const int grp = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
    if (grp >= ngroups) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int bq = GB == 64 ? lane : lane % GB;  // body of this lane within the group
    const int sub = GB == 64 ? 0 : lane / GB;    // which share of the items it takes
    const int64_t g0 = (int64_t)grp * GB;
    const int64_t s = g0 + bq;
    const bool valid = s < n;
    const Body me = body[valid ? s : g0];

    if (threadIdx.x == 0) L.published = 0;
    if (threadIdx.x < kEvals) L.head[threadIdx.x] = 0;
    __syncthreads();

    if (wave == 0) {
        double glo[3], ghi[3];  // the group's bounding box
        walkx::group_box<GB>(valid, me.x, me.y, me.z, glo, ghi);
        const uint64_t active = __ballot(valid) & kBodyMask;
        walkx::traverse<GB>(L, 0, active, ninfo, nmom, walkx::SideSq(box[0]), glo, ghi, me.x, me.y,
                            me.z, th2);
    } else {
        EvalLds<GB> &sh = eval_lds[wave - 1];
        ItemV *const items = sh.items;
        uint16_t *const rec = sh.rec;
        double *const tacc = sh.tacc;
        double *const sacc = sh.sacc;
        const double eb2 = PEPS ? beps2[valid ? s : g0] : 0.0;
        const float ebhf = (float)(0.5 * eb2);  // FP32C: half the target's squared softening
        const CubeConsts cc = cube_consts();
        double lx = 0.0, ly = 0.0, lz = 0.0;
        if (valid) {
            const int64_t o = idx[s];
            lx = lambda[3 * o];
            ly = lambda[3 * o + 1];
            lz = lambda[3 * o + 2];
        }
        // This lane's order of its share's eight items of a dense step: slot bits
        // 2 and 1 follow lane bits 0 and 1, slot bit 0 lane bit 5 (GB = 64) or 3.
        const int perm = ((lane & 1) << 2) | (lane & 2) | (GB == 64 ? lane >> 5 : (lane >> 3) & 1);

        // every upstream value of the wave's bodies, and every offset, is finite; other
        // waves have code of their own (a test a term made FP64 VJPs of 200,000 bodies 5 %
        // longer)
        const bool finite = __ballot(!(isfinite(lx) && isfinite(ly) && isfinite(lz))) == 0 &&
                            box[0].L <= 0x1p1000;

        double gx = 0.0, gy = 0.0, gz = 0.0;  // target-side gradient of this lane's body
        const VT lxv = (VT)lx, lyv = (VT)ly, lzv = (VT)lz;
        for (int i = lane; i < 3 * GB; i += 64) tacc[i] = 0.0;

        // One softened term of source (x, y, z, m, e2) on a target at (bx, by, bz)
        // with softening eb and upstream (ux, uy, uz): the target-side gradient is
        // minus the first three source-side components. In FP32C the offset is the
        // FP64 difference rounded once and the rest of the term is FP32; the term
        // counts when its r^2 is a positive normal number of the precision used.
        // In FP32C the pair softening is the sum of the two halves rounded to
        // FP32 (ebh: the target's), as in the forward FP32C walk.
        auto term = [&](auto all_finite, const ItemV &it, double bx, double by, double bz, double eb, float ebh, VT ux,
                        VT uy, VT uz, bool on, VT out[5]) {
            out[0] = out[1] = out[2] = out[3] = out[4] = VT(0);
            if constexpr (F32) {
                const float dx = (float)(it.x - bx), dy = (float)(it.y - by), dz = (float)(it.z - bz);
                const float e2 = PEPS ? it.e2h + ebh : (float)eps0sq;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, e2)));
                if (on && positive_normal_f(r2)) {
                    const float rinv = __builtin_amdgcn_rsqf(r2), inv2 = rinv * rinv;
                    const float inv3 = inv2 * rinv;
                    const float inv5 = inv3 * inv2;
                    const float ld = ux * dx + uy * dy + uz * dz;
                    const float gms = it.gm;
                    const float c = 3.0f * ld * inv5;
                    out[0] = gms * (ux * inv3 - dx * c);
                    out[1] = gms * (uy * inv3 - dy * c);
                    out[2] = gms * (uz * inv3 - dz * c);
                    out[3] = (float)G * ld * inv3;
                    out[4] = -1.5f * gms * ld * inv5;
                }
            } else {
                const double dx = it.x - bx, dy = it.y - by, dz = it.z - bz;
                const double e2 = PEPS ? 0.5 * (eb + it.e2) : eps0sq;
                const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, e2)));
                const bool live = on && positive_normal(r2);
                const double ld = ux * dx + uy * dy + uz * dz;
                double i2, ri;
                double i3 = inv_cube_sq_f64(r2, i2, ri, cc);
                i3 = live ? i3 : 0.0;
                const double li = live ? ld * i2 : 0.0;
                const double g3 = G * it.m * i3, k3 = 3.0 * li;
                out[0] = g3 * fma(-k3, dx, ux);
                out[1] = g3 * fma(-k3, dy, uy);
                out[2] = g3 * fma(-k3, dz, uz);
                out[3] = G * ld * i3;
                out[4] = -1.5 * g3 * li;
                // zero, where a factor of zero does not make it so
                if (!decltype(all_finite)::value && !live)
                    out[0] = out[1] = out[2] = out[3] = out[4] = 0.0;
            }
        };
        // where component q (0..3) of an item's source-side sum is added, and its
        // fifth, of a node (e2 = (eps_B^2 + <eps^2>_N) / 2)
        auto adj = [&](int32_t src, int q) {
            return src >= 0 ? badj + 4 * (int64_t)src + q : nadj + 4 * (int64_t)(~src) + q;
        };
        auto add_e2 = [&](int32_t src, double v) {
            if (src < 0) unsafeAtomicAdd(nadj_e + ~src, 0.5 * v);
        };
        // After the exchanges of a dense step the lanes that agree in the bits of
        // `perm` and `sub` hold the same item's sums. Lane t of the flush adds
        // component t & 3 of the step's item t / 4 (16 items a flush for GB = 16 and
        // 32, all 8 for GB = 64): it reads them from the lane that holds that item
        // and has the component in the remaining lane bits.
        constexpr int kFlushes = GB == 16 ? 2 : 1, kFlushItems = GB == 64 ? 8 : 16;
        const int fq = lane & 3, fi = lane >> 2;
        int from = ((fi >> 2) & 1) | (fi & 2);  // the lane bits of the item's place in its share
        from |= GB == 64 ? (fi & 1) << 5 : (fi & 1) << 3;
        if (GB == 64) from |= fq << 2;                                    // component: bits 2, 3
        if (GB == 32) from |= (fq & 1) << 2 | (fq >> 1) << 4 | (fi >> 3) << 5;  // bits 2, 4
        if (GB == 16) from |= (fq & 1) << 2 | (fi >> 3) << 4;             // bit 2 (and two values)

        auto evaluate = [&](auto all_finite, walkx::Batch &bt) {
            const int c = bt.count;
            uint64_t mk;
            int32_t src;
            walkx::take_batch(L, wave - 1, bt, src, mk);
            ItemV ld_it{0.0, 0.0, 0.0, 0.0, 0.0, 0ull, 0, 0.f, 0.f, 0};
            if (lane < c) {
                if (src >= 0) {
                    if (!check_ok(src < n, CK_INDEX)) src = 0;
                    const int64_t rel = (int64_t)src - g0;
                    if (rel >= 0 && rel < GB) mk &= ~(1ull << rel);
                    const Body b = body[src];
                    const double e2 = PEPS ? beps2[src] : 0.0;
                    ld_it = ItemV{b.x,  b.y, b.z, b.m, e2, mk, src, (float)(G * b.m),
                                  (float)(0.5 * e2), 0};
                } else {
                    const NodeMom nm = nmom[~src];
                    const double e2 = PEPS ? neps2[~src] : 0.0;
                    ld_it = ItemV{nm.x, nm.y, nm.z, nm.m, e2, mk, src, (float)(G * nm.m),
                                  (float)(0.5 * e2), 0};
                }
            }
            const int pk = __popcll(mk);
            const bool sparse = lane < c && pk <= kSparse;
            const uint32_t pv = sparse ? (uint32_t)pk : 0u;
            const uint32_t pend = wave_incl_scan(pv);
            const bool fits = sparse && pend <= (uint32_t)kPairCap;
            const bool dense = lane < c && !fits;
            const uint64_t db = __ballot(dense);
            const uint64_t fb = __ballot(fits && pk > 0);
            const int nd = __popcll(db);
            const int ns = __popcll(fb);
            const int np = fb ? __builtin_amdgcn_readlane((int)pend, 63 - __builtin_clzll(fb)) : 0;
            BHX_CHECK(np <= kPairCap, CK_PAIRS);
            if (dense || (fits && pk > 0)) {
                const int slot = dense ? (int)lanes_below(db) : nd + (int)lanes_below(fb);
                items[slot] = ld_it;
                if (fits) {
#pragma unroll
                    for (int q = 0; q < 5; q++) sacc[5 * slot + q] = 0.0;
                    uint64_t bits = mk;
                    uint32_t at = pend - pv;
                    while (bits) {
                        rec[at++] = (uint16_t)(slot << 6 | __builtin_ctzll(bits));
                        bits &= bits - 1;
                    }
                }
            }
            walkx::wave_sync();

            // dense items, eight per share of lanes per step
#pragma unroll 1
            for (int j0 = 0; j0 < nd; j0 += 8 * LPB) {
                VT v[8][NC];
                VT sx = VT(0), sy = VT(0), sz = VT(0);  // FP32C: this step's target-side terms
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    const int j = j0 + 8 * sub + (t ^ perm);
                    const ItemV it = items[j < nd ? j : j0];
                    const bool on = j < nd && ((it.mask >> bq) & 1ull);
                    VT o[5];
                    term(all_finite, it, me.x, me.y, me.z, eb2, ebhf, lxv, lyv, lzv, on, o);
                    if constexpr (F32) {
                        sx -= o[0];
                        sy -= o[1];
                        sz -= o[2];
                    } else {
                        gx -= o[0];
                        gy -= o[1];
                        gz -= o[2];
                    }
#pragma unroll
                    for (int q = 0; q < NC; q++) v[t][q] = o[q];
                }
                if constexpr (F32) {
                    gx += (double)sx;
                    gy += (double)sy;
                    gz += (double)sz;
                }
#pragma unroll
                for (int t = 0; t < 4; t++)
#pragma unroll
                    for (int q = 0; q < NC; q++) v[t][q] += dpp<kDppXor1>(v[t + 4][q]);
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int q = 0; q < NC; q++) v[t][q] += dpp<kDppXor2>(v[t + 2][q]);
#pragma unroll
                for (int q = 0; q < NC; q++) {
                    VT w;
                    if constexpr (GB == 64) {
                        w = v[0][q] + __shfl_xor(v[1][q], 32);
                        w += dpp<kDppRor4>(w);
                        w += dpp<kDppRor8>(w);
                        w += __shfl_xor(w, 16);
                    } else {
                        w = v[0][q] + dpp<kDppRor8>(v[1][q]);  // lane ^ 8 inside the row
                        w += __shfl_xor(w, 4);
                        if (GB == 32) w += __shfl_xor(w, 16);
                    }
                    v[0][q] = w;
                }
                if constexpr (GB == 16) {
                    // two of the four components per source lane, picked by the reader
                    const VT va = (lane & 4) ? v[0][1] : v[0][0], vb = (lane & 4) ? v[0][3] : v[0][2];
#pragma unroll
                    for (int f = 0; f < kFlushes; f++) {
                        const VT wa = __shfl(va, from | f << 5), wb = __shfl(vb, from | f << 5);
                        const int j = j0 + kFlushItems * f + fi;
                        if (j < nd) unsafeAtomicAdd(adj(items[j].src, fq), (double)(fq >> 1 ? wb : wa));
                    }
                } else {
                    const int c = GB == 64 ? (lane >> 2) & 3 : ((lane >> 2) & 1) | ((lane >> 4) & 1) << 1;
                    const VT lo = c & 1 ? v[0][1] : v[0][0], hi = c & 1 ? v[0][3] : v[0][2];
                    const VT w = __shfl(c >> 1 ? hi : lo, from);
                    const int j = j0 + fi;
                    if (fi < kFlushItems && j < nd) unsafeAtomicAdd(adj(items[j].src, fq), (double)w);
                }
                if constexpr (PEPS) {
                    // each share's sums of items j0 + 8 sub + perm sit in its lanes with
                    // lane bits 2 and 3, 4 (GB = 64) or 2 (and 4 for GB = 32) clear
                    const int j = j0 + 8 * sub + perm;
                    const bool lead =
                        GB == 64 ? (lane & 28) == 0 : GB == 32 ? (lane & 20) == 0 : (lane & 4) == 0;
                    if (lead && j < nd) add_e2(items[j].src, (double)v[0][4]);
                }
            }

            // sparse items as pairs
#pragma unroll 1
            for (int i0 = 0; i0 < np; i0 += 64) {
                const int i = i0 + lane;
                const bool on = i < np;
                const uint32_t r = rec[on ? i : i0];
                const int k = (int)(r >> 6), b = (int)(r & 63u);
                const double bx = __shfl(me.x, b), by = __shfl(me.y, b), bz = __shfl(me.z, b);
                const double eb = PEPS && !F32 ? __shfl(eb2, b) : 0.0;
                const float ebh = PEPS && F32 ? __shfl(ebhf, b) : 0.f;
                const VT ux = __shfl(lxv, b), uy = __shfl(lyv, b), uz = __shfl(lzv, b);
                const ItemV it = items[k];
                VT o[5];
                term(all_finite, it, bx, by, bz, eb, ebh, ux, uy, uz, on, o);
                if (on) {
#pragma unroll
                    for (int q = 0; q < 3; q++)
                        __hip_atomic_fetch_add(&tacc[3 * b + q], -(double)o[q], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                    for (int q = 0; q < NC; q++)
                        __hip_atomic_fetch_add(&sacc[5 * k + q], (double)o[q], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            walkx::wave_sync();
            for (int i = lane; i < 4 * ns; i += 64) {
                const int k = nd + (i >> 2);
                unsafeAtomicAdd(adj(items[k].src, i & 3), sacc[5 * k + (i & 3)]);
            }
            if (PEPS && lane < ns) add_e2(items[nd + lane].src, sacc[5 * (nd + lane) + 4]);
            walkx::wave_sync();
        };

        walkx::Batch bt;
        bt.start = (uint32_t)(kBatch * (wave - 1));
        if (F32 || finite)
            while (walkx::next_batch(L, wave - 1, bt)) evaluate(std::true_type{}, bt);
        else if constexpr (!F32)
            while (walkx::next_batch(L, wave - 1, bt)) evaluate(std::false_type{}, bt);

        // the lanes' shares of each body, in a fixed order, then its pair sums
#pragma unroll
        for (int o = GB; o < 64; o <<= 1) {
            gx += __shfl_xor(gx, o);
            gy += __shfl_xor(gy, o);
            gz += __shfl_xor(gz, o);
        }
        if (sub == 0) {
            tacc[3 * bq] += gx;
            tacc[3 * bq + 1] += gy;
            tacc[3 * bq + 2] += gz;
        }
    }
    __syncthreads();
    // the waves' sums in wave order
    if (wave != 1 || !valid || sub != 0) return;
    for (int a = 0; a < 3; a++) {
        double v = 0.0;
        for (int e = 0; e < kEvals; e++) v += eval_lds[e].tacc[3 * bq + a];
        gt[3 * s + a] = v;
    }
}

// Zeroes body adjoints (4 per body) and node adjoints (4 and 1 per node that
// exists), and writes each node's parent (-1 for the root).
__global__ __launch_bounds__(256) void k_vjp_clear(double *__restrict__ badj, int64_t n,
                                                   double *__restrict__ nadj,
                                                   double *__restrict__ nadj_e,
                                                   int32_t *__restrict__ nparent,
                                                   const NodeInfo *__restrict__ ninfo,
                                                   const TreeHeader *__restrict__ hdr,
                                                   int64_t node_cap)
{
    int64_t nn = 0;
    for (int l = 0; l < kLevels; l++) nn += hdr->level_count[l];
    if (nn > node_cap) nn = node_cap;
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t i = t; i < 4 * n; i += stride) badj[i] = 0.0;
    for (int64_t i = t; i < 4 * nn; i += stride) nadj[i] = 0.0;
    for (int64_t i = t; i < nn; i += stride) nadj_e[i] = 0.0;
    if (t == 0 && nn > 0) nparent[0] = -1;
    for (int64_t k = t; k < nn; k += stride) {
        const NodeInfo info = ninfo[k];
        if (info.child0 < 0) continue;
        const int nch = node_nchild(info);
        for (int o = 0; o < nch; o++)
            if (check_ok((int64_t)info.child0 + o < nn, CK_INDEX)) nparent[info.child0 + o] = (int32_t)k;
    }
}

// Per-node coefficients of the member update, from the node's adjoints.
__device__ inline void node_coeffs(const double *__restrict__ nadj,
                                   const double *__restrict__ nadj_e, const NodeMom &nm, double e2,
                                   int64_t k, double out[5])
{
    const double *a = nadj + 4 * k;
    if (nm.m > 0.0) {
        const double inv = 1.0 / nm.m;
        out[0] = a[0] * inv;
        out[1] = a[1] * inv;
        out[2] = a[2] * inv;
        out[4] = nadj_e[k] * inv;
        out[3] = a[3] - (nm.x * out[0] + nm.y * out[1] + nm.z * out[2]) - e2 * out[4];
    } else {
        out[0] = out[1] = out[2] = out[4] = 0.0;
        out[3] = a[3];
    }
}

// Every leaf hands the ancestor sums of the node coefficients to its
// members and adds the members' own terms into the caller's gradient arrays
// (caller order, +=). A leaf collects its chain of ancestors through the
// parent table (at most kLevels nodes) and sums their coefficients from the
// root down.
__global__ __launch_bounds__(256) void k_vjp_finish(
    const TreeHeader *__restrict__ hdr, const NodeInfo *__restrict__ ninfo,
    const NodeMom *__restrict__ nmom, const double *__restrict__ neps2,
    const int32_t *__restrict__ nparent, const double *__restrict__ nadj,
    const double *__restrict__ nadj_e,
    const Body *__restrict__ body, const double *__restrict__ beps2, int use_eps,
    const uint32_t *__restrict__ idx, const double *__restrict__ gt,
    const double *__restrict__ badj, double *__restrict__ g_pos, double *__restrict__ g_mass,
    int64_t node_cap)
{
    int64_t nn = 0;
    for (int l = 0; l < kLevels; l++) nn += hdr->level_count[l];
    if (nn > node_cap) nn = node_cap;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < nn;
         k += (int64_t)gridDim.x * 256) {
        const NodeInfo info = ninfo[k];
        if (info.child0 >= 0) continue;
        int32_t chain[kLevels];  // chain[d]: the leaf's ancestor d levels up, or -1
        int32_t cur = (int32_t)k;
#pragma unroll
        for (int d = 0; d < kLevels; d++) {
            chain[d] = cur;
            cur = cur >= 0 ? nparent[cur] : -1;
        }
        double p[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int d = kLevels - 1; d >= 0; d--) {
            const int32_t c = chain[d];
            if (c < 0) continue;
            double cf[5];
            node_coeffs(nadj, nadj_e, nmom[c], use_eps ? neps2[c] : 0.0, c, cf);
            for (int q = 0; q < 5; q++) p[q] = p[q] + cf[q];
        }
        for (int32_t s = info.first; s < info.first + info.count; s++) {
            const Body b = body[s];
            const double e2 = use_eps ? beps2[s] : 0.0;
            const int64_t o = idx[s];
            const double *ba = badj + 4 * (int64_t)s;
            g_pos[3 * o] += gt[3 * s] + ba[0] + b.m * p[0];
            g_pos[3 * o + 1] += gt[3 * s + 1] + ba[1] + b.m * p[1];
            g_pos[3 * o + 2] += gt[3 * s + 2] + ba[2] + b.m * p[2];
            g_mass[o] += ba[3] + p[3] + b.x * p[0] + b.y * p[1] + b.z * p[2] + e2 * p[4];
        }
    }
}

// Direct-sum VJP, gathered per body p (no atomics):
//   g_x_p += G sum_{q != p} K(d_pq) (m_p lambda_q - m_q lambda_p)
//   g_m_p += G sum_{q != p} lambda_q . (x_p - x_q) / r^3
// A block's four waves share 64 bodies p (one per lane) and take the groups of
// 32 sources of a 256-source tile in turn; block row y sums the y-th range of
// tiles (one row unless the targets alone give too few blocks; the rows'
// partial sums are then added in row order by k_direct_vjp_reduce). Bound by
// VALU issue, as the direct sum, and like there the pairs of a group are tested
// together: a group with a dead pair (or body p itself) takes them singly.
// K w = w / r^3 - 3 d (d.w) / r^5 with r^-3 in one third-order step and
// r^-5 = r^-3 r^-2 from the same estimate: 38 instructions a pair, 58 with two
// Newton steps. 8192 bodies: 137 -> 104 us, 50000: 4.9 -> 3.4 ms;
// 2048: 60 -> 18 us (256 blocks instead of 64).
struct alignas(16) SrcV {
    double x, y, z, m, lx, ly, lz, eh;  // eh: half the squared softening
};
constexpr int kVjpGroup = 32, kVjpTile = 256;

template <bool PEPS>
__global__ __launch_bounds__(256) void k_direct_vjp(const double *__restrict__ pos,
                                                    const double *__restrict__ mass,
                                                    const double *__restrict__ eps, int64_t n,
                                                    double eps0sq, double G,
                                                    const double *__restrict__ lambda,
                                                    double *__restrict__ g_pos,
                                                    double *__restrict__ g_mass, int64_t chunk,
                                                    double *__restrict__ part)
{
    __shared__ SrcV src[kVjpTile];
    __shared__ double red[3][4][64];  // the other waves' sums
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * 64, p = b0 + lane;
    const bool valid = p < n;
    // lanes past the end repeat the last body; nothing of theirs is stored
    const int64_t pc = valid ? p : n - 1;
    const double xp = pos[3 * pc], yp = pos[3 * pc + 1], zp = pos[3 * pc + 2], mp = mass[pc];
    const double lpx = lambda[3 * pc], lpy = lambda[3 * pc + 1], lpz = lambda[3 * pc + 2];
    const double ehp = PEPS ? 0.5 * (eps[pc] * eps[pc]) : 0.0;
    const CubeConsts k = cube_consts();
    double gx = 0.0, gy = 0.0, gz = 0.0, gm = 0.0;
    // adds the pair with source s to (ax, ay, az, am)
    auto pair = [&](const SrcV &s, double dx, double dy, double dz, double r2, double &ax,
                    double &ay, double &az, double &am) {
        double i2, ri;
        const double i3 = inv_cube_sq_f64(r2, i2, ri, k), i5 = i3 * i2;
        // w = m_p lambda_q - m_q lambda_p
        const double wx = fma(mp, s.lx, -(s.m * lpx)), wy = fma(mp, s.ly, -(s.m * lpy)),
                     wz = fma(mp, s.lz, -(s.m * lpz));
        const double c = 3.0 * (dx * wx + dy * wy + dz * wz) * i5;
        ax = fma(-c, dx, fma(wx, i3, ax));
        ay = fma(-c, dy, fma(wy, i3, ay));
        az = fma(-c, dz, fma(wz, i3, az));
        am = fma(-(s.lx * dx + s.ly * dy + s.lz * dz), i3, am);
    };
    auto dist2 = [&](const SrcV &s, double &dx, double &dy, double &dz) {
        dx = s.x - xp, dy = s.y - yp, dz = s.z - zp;
        return fma(dx, dx, fma(dy, dy, fma(dz, dz, PEPS ? ehp + s.eh : eps0sq)));
    };
    const int64_t s_lo = (int64_t)blockIdx.y * chunk;
    const int64_t s_hi = s_lo + chunk < n ? s_lo + chunk : n;
    for (int64_t base = s_lo; base < s_hi; base += kVjpTile) {
        const int64_t q = base + tid;
        if (q < s_hi) {
            const double e = PEPS ? eps[q] : 0.0;
            src[tid] = SrcV{pos[3 * q], pos[3 * q + 1], pos[3 * q + 2], mass[q],
                            lambda[3 * q], lambda[3 * q + 1], lambda[3 * q + 2], 0.5 * (e * e)};
        }
        __syncthreads();
        const int cnt = (int)((s_hi - base) < kVjpTile ? (s_hi - base) : kVjpTile);
#pragma unroll 1
        for (int g = wave * kVjpGroup; g < cnt; g += 4 * kVjpGroup) {
            const SrcV *sg = src + g;
            const int gc = cnt - g < kVjpGroup ? cnt - g : kVjpGroup;
            const bool own = base + g < b0 + 64 && base + g + gc > b0;
            if (gc == kVjpGroup && !own) {
                double ax = 0.0, ay = 0.0, az = 0.0, am = 0.0;
                bool live = true;
#pragma unroll 2
                for (int j = 0; j < kVjpGroup; j++) {
                    const SrcV s = sg[j];
                    double dx, dy, dz;
                    const double r2 = dist2(s, dx, dy, dz);
                    live = live && positive_normal(r2);
                    pair(s, dx, dy, dz, r2, ax, ay, az, am);
                }
                if (__ballot(!live) == 0) {
                    gx += ax;
                    gy += ay;
                    gz += az;
                    gm += am;
                    continue;
                }
            }
#pragma unroll 1
            for (int j = 0; j < gc; j++) {
                const SrcV s = sg[j];
                double dx, dy, dz;
                const double r2 = dist2(s, dx, dy, dz);
                if (base + g + j != p && positive_normal(r2)) pair(s, dx, dy, dz, r2, gx, gy, gz, gm);
            }
        }
        __syncthreads();
    }
    if (wave > 0) {
        double(*r)[64] = red[wave - 1];
        r[0][lane] = gx;
        r[1][lane] = gy;
        r[2][lane] = gz;
        r[3][lane] = gm;
    }
    __syncthreads();
    if (wave > 0 || !valid) return;
#pragma unroll
    for (int w = 0; w < 3; w++) {  // in wave order
        gx += red[w][0][lane];
        gy += red[w][1][lane];
        gz += red[w][2][lane];
        gm += red[w][3][lane];
    }
    if (gridDim.y == 1) {
        g_pos[3 * p] += G * gx;
        g_pos[3 * p + 1] += G * gy;
        g_pos[3 * p + 2] += G * gz;
        g_mass[p] += G * gm;
    } else {
        double *o = part + 4 * ((int64_t)blockIdx.y * n + p);
        o[0] = gx;
        o[1] = gy;
        o[2] = gz;
        o[3] = gm;
    }
}

// Adds G times the rows' partial sums, in row order, into the gradients; one
// thread per body and component, so that a wave reads whole lines.
__global__ __launch_bounds__(256) void k_direct_vjp_reduce(const double *__restrict__ part,
                                                           int64_t n, int rows, double G,
                                                           double *__restrict__ g_pos,
                                                           double *__restrict__ g_mass)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t p = t >> 2;
    if (p >= n) return;
    double s = 0.0;
#pragma unroll 8
    for (int r = 0; r < rows; r++) s += part[4 * (int64_t)r * n + t];
    double *o = (t & 3) == 3 ? g_mass + p : g_pos + 3 * p + (t & 3);
    *o += G * s;
}

// Adjoint of the second kick: abar += dt/2 vbar.
__global__ __launch_bounds__(256) void k_adj_kick(double *__restrict__ abar,
                                                  const double *__restrict__ vbar, int64_t n3,
                                                  double h)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n3) abar[i] += h * vbar[i];
}

// Adjoint of the drift and the first kick: vbar += dt xbar; abar = dt/2 vbar.
__global__ __launch_bounds__(256) void k_adj_drift_kick(double *__restrict__ vbar,
                                                        double *__restrict__ abar,
                                                        const double *__restrict__ xbar,
                                                        int64_t n3, double dt, double h)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n3) return;
    const double v = vbar[i] + dt * xbar[i];
    vbar[i] = v;
    abar[i] = h * v;
}

// x_out = x_in + dt (v + dt/2 a); v += dt/2 a (kick and drift into a new buffer)
__global__ __launch_bounds__(256) void k_kick_drift_to(const double *__restrict__ x_in,
                                                       double *__restrict__ v,
                                                       const double *__restrict__ a,
                                                       double *__restrict__ x_out, int64_t n3,
                                                       double h, double dt)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n3) return;
    const double u = v[i] + h * a[i];
    v[i] = u;
    x_out[i] = x_in[i] + dt * u;
}

__global__ __launch_bounds__(256) void k_copy(double *__restrict__ dst,
                                              const double *__restrict__ src, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

inline unsigned blocks(int64_t items, unsigned cap = 1u << 30)
{
    int64_t b = (items + 255) / 256;
    if (b < 1) b = 1;
    return (unsigned)(b < (int64_t)cap ? b : cap);
}

}  // namespace

BHX_DEFINE_TAKE_CHECKS(adjoint_take_checks)

hipError_t launch_tree_vjp(const Workspace &w, const AdjointWork &aw, hipStream_t s,
                           const WalkParams &p, const double *lambda, double *g_pos,
                           double *g_mass)
{
    if (p.n <= 0) return hipSuccess;
    // the fifth component of every node follows the four of all
    double *const nadj_e = aw.nadj + 4 * aw.node_cap;
    k_vjp_clear<<<1024, 256, 0, s>>>(aw.badj, p.n, aw.nadj, nadj_e, aw.nparent, w.ninfo, w.hdr,
                                     w.node_cap);
    const int gb = p.group == 16 || p.group == 32 ? p.group : 64;
    const int ngroups = (int)((p.n + gb - 1) / gb);
    const int per_xcd = (ngroups + 7) / 8;
    auto walk = [&](auto peps, auto gbc) {
        if (p.precision == BH_FP32C)
            k_vjp_walk<decltype(peps)::value, decltype(gbc)::value, true>
                <<<8 * per_xcd, 64 * (1 + kEvals), 0, s>>>(w.body, w.beps2, w.ninfo, w.nmom, w.neps2, w.idx[0],
                                            w.box, p.n, ngroups, per_xcd, p.th2, p.eps0sq, p.G,
                                            lambda, aw.gt, aw.badj, aw.nadj, nadj_e);
        else
            k_vjp_walk<decltype(peps)::value, decltype(gbc)::value, false>
                <<<8 * per_xcd, 64 * (1 + kEvals), 0, s>>>(w.body, w.beps2, w.ninfo, w.nmom, w.neps2, w.idx[0],
                                            w.box, p.n, ngroups, per_xcd, p.th2, p.eps0sq, p.G,
                                            lambda, aw.gt, aw.badj, aw.nadj, nadj_e);
    };
    using T = std::true_type;
    using F = std::false_type;
    using I16 = std::integral_constant<int, 16>;
    using I32 = std::integral_constant<int, 32>;
    using I64 = std::integral_constant<int, 64>;
    if (p.per_body_eps) {
        if (gb == 16) walk(T{}, I16{});
        else if (gb == 32) walk(T{}, I32{});
        else walk(T{}, I64{});
    } else {
        if (gb == 16) walk(F{}, I16{});
        else if (gb == 32) walk(F{}, I32{});
        else walk(F{}, I64{});
    }
    const int use_eps = p.per_body_eps ? 1 : 0;
    k_vjp_finish<<<blocks(p.n, 4096), 256, 0, s>>>(w.hdr, w.ninfo, w.nmom, w.neps2, aw.nparent,
                                                   aw.nadj, nadj_e, w.body, w.beps2, use_eps, w.idx[0],
                                                   aw.gt, aw.badj, g_pos, g_mass, w.node_cap);
    return hipGetLastError();
}

hipError_t launch_direct_vjp(hipStream_t s, const double *pos, const double *mass,
                             const double *eps, int64_t n, double eps0sq, double G,
                             const double *lambda, double *g_pos, double *g_mass, double *part)
{
    if (n <= 0) return hipSuccess;
    // rows of source ranges (whole tiles): as many as the partial buffer holds
    // and at most kDirectBlocks * 4 blocks
    const int64_t tb = (n + 63) / 64;
    const int64_t all = (n + kVjpTile - 1) / kVjpTile;
    int64_t rows = part ? kDirectPart / (4 * n) : 1;
    if (rows > 4 * kDirectBlocks / tb) rows = 4 * kDirectBlocks / tb;
    if (rows < 1) rows = 1;
    if (rows > all) rows = all;
    const int64_t tiles = (all + rows - 1) / rows;
    rows = (all + tiles - 1) / tiles;
    const int64_t chunk = rows == 1 ? n : tiles * kVjpTile;
    const dim3 grid((unsigned)tb, (unsigned)rows);
    if (eps)
        k_direct_vjp<true><<<grid, 256, 0, s>>>(pos, mass, eps, n, eps0sq, G, lambda, g_pos,
                                                g_mass, chunk, part);
    else
        k_direct_vjp<false><<<grid, 256, 0, s>>>(pos, mass, eps, n, eps0sq, G, lambda, g_pos,
                                                 g_mass, chunk, part);
    if (rows > 1)
        k_direct_vjp_reduce<<<(unsigned)((4 * n + 255) / 256), 256, 0, s>>>(part, n, (int)rows, G,
                                                                            g_pos, g_mass);
    return hipGetLastError();
}

hipError_t launch_adj_kick(hipStream_t s, double *abar, const double *vbar, int64_t n, double dt)
{
    if (n <= 0) return hipSuccess;
    k_adj_kick<<<blocks(3 * n), 256, 0, s>>>(abar, vbar, 3 * n, 0.5 * dt);
    return hipGetLastError();
}

hipError_t launch_adj_drift_kick(hipStream_t s, double *vbar, double *abar, const double *xbar,
                                 int64_t n, double dt)
{
    if (n <= 0) return hipSuccess;
    k_adj_drift_kick<<<blocks(3 * n), 256, 0, s>>>(vbar, abar, xbar, 3 * n, dt, 0.5 * dt);
    return hipGetLastError();
}

hipError_t launch_kick_drift_to(hipStream_t s, const double *x_in, double *v, const double *a,
                                double *x_out, int64_t n, double dt)
{
    if (n <= 0) return hipSuccess;
    k_kick_drift_to<<<blocks(3 * n), 256, 0, s>>>(x_in, v, a, x_out, 3 * n, 0.5 * dt, dt);
    return hipGetLastError();
}

hipError_t launch_copy(hipStream_t s, double *dst, const double *src, int64_t count)
{
    if (count <= 0) return hipSuccess;
    k_copy<<<blocks(count), 256, 0, s>>>(dst, src, count);
    return hipGetLastError();
}

}  // namespace bhx
