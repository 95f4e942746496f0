// The traversal shared by the forward walk (walk.hip) and the VJP walk
// (adjoint.hip): one wavefront walks the tree for a group of target bodies,
// every stack entry carrying the mask of the bodies whose own walk reaches it,
// and each body taking its own opening decisions (eq. accuracy), so both
// kernels see exactly the interaction lists of the per-body walk.
//
// A block is one traversing wave and kEvals evaluating waves. The traversal
// queues interaction descriptors in an LDS ring; evaluating wave e takes the
// batches of 64 items number e, e + kEvals, e + 2 kEvals, ... A batch is the same
// 64 items in the same order as one wave doing both would take, and the waves'
// sums are added in a fixed order. One wave doing both was bound by the latency
// of its own chain (LDS and L2 round trips of the traversal, then of staging):
// with 64-body groups at 2^20 bodies the VALU was 64 % busy and at 40,000 bodies
// with 16-body groups 38 %, the traversal's rounds and the batches taking turns.
// Walk, one wave -> 1 + 3 waves: 2^20 bodies (leaf 4, FP32C) 2.37 -> 1.80 ms,
// 131072 (Plummer, leaf 16) 1.20 -> 0.75 ms, 50,000 (FP64, leaf 8) 308 -> 163 us,
// 1000 (leaf 16) 51 -> 16 us. Two evaluating waves: 4 % slower at 2^20, 15 %
// at 131072 and 8 % at 50,000; four: 25 % slower at 2^20 (fewer blocks fit a
// CU's LDS), 5 % faster at 1000.
#pragma once

#include "bhx_impl.h"

namespace bhx {
namespace walkx {

// Relative margin of the group-box opening test. The per-body test's D^2
// and theta^2 D^2 carry a relative rounding error below 1e-15, so a box
// bound that clears the threshold by this margin decides every body alike.
constexpr double kMacMargin = 1e-12;
constexpr int kRanges = 8;      // ranges popped per round (<= 8 nodes each)
constexpr int kReserve = 150;   // a depth-first descent adds <= 7 ranges per level
constexpr int kBatch = 64;      // items evaluated together
constexpr int kEvals = 3;       // evaluating waves of a block
constexpr int kRing = 256;      // descriptors in flight
constexpr int kPollSleep = 8;   // a waiting wave looks again after this many 64 cycles

struct alignas(16) PopCom {  // popped node as the per-body opening test needs it
    double x, y, z, s2;
};
struct DqRange {  // a descriptor's items: running number of the first, count
    uint32_t at;
    int32_t n;
};

// The opening test, rounded exactly as written: accept iff s^2 < theta^2 D^2.
__device__ inline bool accept_node(double cx, double cy, double cz, double bx, double by,
                                   double bz, double s2, double th2)
{
#pragma clang fp contract(off)
    double dx = cx - bx, dy = cy - by, dz = cz - bz;
    double D2 = dx * dx + dy * dy + dz * dz;
    return s2 < th2 * D2;
}

// Orders a wave's own LDS accesses around this point. The LDS unit serves a
// wave's instructions in order, so a later read by any lane sees an earlier
// write by any other without a wait; only the compiler has to keep them so.
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The LDS a traversal works in: the stack of child ranges, the ring of
// interaction descriptors (a leaf's body range or one accepted node, with
// the mask of the bodies that take it), the mixed nodes of a round, and what
// the waves tell each other: items queued and descriptors written (bit 31 of
// the latter: no more will come), and each evaluating wave's first descriptor
// still in use.
template <int kStack>
struct Lds {
    static_assert((kRing & (kRing - 1)) == 0, "ring indices wrap by masking");
    // When all evaluating waves wait, fewer than 64 items are left for the one
    // whose batch comes first, and the heads of the others are past them; a
    // round adds at most 64 descriptors.
    static_assert(kRing >= 64 + 64, "the traversal never waits for waves that wait for it");
    int32_t st_c0[kStack];
    uint8_t st_n[kStack];
    uint64_t st_mask[kStack];
    int32_t dq_a[kRing];    // leaf: first body; node: ~node
    DqRange dq_r[kRing];
    uint64_t dq_mask[kRing];
    PopCom mix[64];
    uint64_t published;     // items queued | descriptors written << 32
    uint32_t head[kEvals];
};
constexpr uint32_t kDone = 0x80000000u;

// The squared cell side per level, (L 2^-l)^2: the root's times 4^-l, which is
// the same number while it is normal from the first level to the last; a root cube
// so small or large that it is not (side below about 1e-139 or above 1e154) reads its
// table.
struct SideSq {
    const double *tab;
    double root;
    bool scaled;
    __device__ explicit SideSq(const SceneBox &b)
        : tab(b.s2), root(b.s2[0]), scaled(b.s2[kMaxLevel] > 0x1p-1000 && b.s2[0] < __builtin_huge_val())
    {
    }
    __device__ double at(int level) const
    {
        return scaled ? ldexp(root, -2 * level) : tab[level];
    }
};

// The group's bounding box: exact min and max of its bodies' coordinates
// (lanes of invalid bodies do not count).
template <int GB>
__device__ inline void group_box(bool valid, double x, double y, double z, double lo[3],
                                 double hi[3])
{
    lo[0] = valid ? x : __builtin_huge_val(), hi[0] = valid ? x : -__builtin_huge_val();
    lo[1] = valid ? y : __builtin_huge_val(), hi[1] = valid ? y : -__builtin_huge_val();
    lo[2] = valid ? z : __builtin_huge_val(), hi[2] = valid ? z : -__builtin_huge_val();
#pragma unroll
    for (int o = 1; o < GB; o <<= 1)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fmin(lo[a], __shfl_xor(lo[a], o));
            hi[a] = fmax(hi[a], __shfl_xor(hi[a], o));
        }
}

// The whole traversal of one group by one wave, from the root node `root` (a
// range of one) with the group's body mask `active`.
//
// A round pops up to kRanges child ranges (at most 64 nodes, lane 8 r + o
// taking child o of range r) so that after expanding them at least kReserve
// stack entries stay free for a depth-first descent, and each lane loads its
// node and keeps it in registers. Opening tests: the lane first bounds its
// node's distance to the group's bounding box; when the test comes out the same
// for every point of the box, with a margin far above the rounding of the
// per-body test, that is every body's decision. The other ("mixed") internal
// nodes go through LDS and are tested by every body, 64 / GB nodes per step (one
// per share of lanes), each step's result going to the node's lane. Then all
// lanes at once: a node opened by the bodies in O pushes its child range with
// mask O; a leaf, or a node accepted by the bodies in A, queues a descriptor
// (mask: the bodies that reached the leaf, or A) and the round is published.
template <int GB, int kStack>
__device__ __forceinline__ void traverse(Lds<kStack> &L, int32_t root, uint64_t active,
                                         const NodeInfo *__restrict__ ninfo,
                                         const NodeMom *__restrict__ nmom,
                                         const SideSq &side, const double glo[3],
                                         const double ghi[3], double bx, double by, double bz,
                                         double th2)
{
    constexpr int LPB = 64 / GB;  // lanes per body
    constexpr uint64_t kBodyMask = GB == 64 ? ~0ull : ((1ull << GB) - 1ull);
    const int lane = threadIdx.x & 63;
    const int sub = GB == 64 ? 0 : lane / GB;

    // the other waves of the block wait for this one (2^20 bodies: 3 % faster)
    __builtin_amdgcn_s_setprio(3);
    int sp = 1;              // stack entries
    uint32_t dq_tail = 0;    // descriptors written
    uint32_t queued = 0;     // items queued
    uint32_t freed = 0;      // descriptors no evaluating wave needs any more
    if (lane == 0) {
        L.st_c0[0] = root;
        L.st_n[0] = 1;
        L.st_mask[0] = active;
    }
    wave_sync();
    while (sp > 0) {
        int cr = min(kRanges, sp);
        const int room = (kStack - kReserve - sp) / 7;
        if (cr > room) cr = room > 1 ? room : 1;
        const int base = sp - cr;
        int32_t k = -1;
        uint64_t M = 0;
        {
            const int r = lane >> 3, o = lane & 7;
            if (r < cr) {
                const int e = base + r;
                if (o < L.st_n[e]) {
                    k = L.st_c0[e] + o;
                    M = L.st_mask[e];
                }
            }
        }
        sp = base;
        const bool mine = k >= 0;
        NodeInfo info{0, 0, -1, 0};
        NodeMom nm{0.0, 0.0, 0.0, 0.0};
        double s2 = 0.0;
        uint64_t accepted = 0;
        bool mixed = false;
        if (mine) {
            info = ninfo[k];
            nm = nmom[k];
            if (info.child0 >= 0) {
                s2 = side.at(node_level(info));
                const double ex = fmax(0.0, fmax(glo[0] - nm.x, nm.x - ghi[0]));
                const double ey = fmax(0.0, fmax(glo[1] - nm.y, nm.y - ghi[1]));
                const double ez = fmax(0.0, fmax(glo[2] - nm.z, nm.z - ghi[2]));
                const double fx = fmax(fabs(nm.x - glo[0]), fabs(nm.x - ghi[0]));
                const double fy = fmax(fabs(nm.y - glo[1]), fabs(nm.y - ghi[1]));
                const double fz = fmax(fabs(nm.z - glo[2]), fabs(nm.z - ghi[2]));
                const double dmin2 = ex * ex + ey * ey + ez * ez;
                const double dmax2 = fx * fx + fy * fy + fz * fz;
                if (s2 < th2 * dmin2 * (1.0 - kMacMargin))
                    accepted = kBodyMask;
                else
                    mixed = !(s2 > th2 * dmax2 * (1.0 + kMacMargin));
            }
        }
        const uint64_t mb = __ballot(mixed);
        const int rank = (int)lanes_below(mb);
        if (mixed) L.mix[rank] = PopCom{nm.x, nm.y, nm.z, s2};
        wave_sync();
        const int nmix = __popcll(mb);
#pragma unroll 1
        for (int p0 = 0; p0 < nmix; p0 += LPB) {
            const int p = p0 + sub;
            const PopCom q = L.mix[p < nmix ? p : p0];
            const bool ok = accept_node(q.x, q.y, q.z, bx, by, bz, q.s2, th2);
            const uint64_t bal = __ballot(ok);
            if constexpr (LPB == 1) {
                if (mixed && rank == p0) accepted = bal;
            } else {
                if (mixed && rank / LPB == p0 / LPB)
                    accepted = (bal >> (rank % LPB * GB)) & kBodyMask;
            }
        }

        const bool leaf = mine && info.child0 < 0;
        const uint64_t A = (mine && !leaf) ? (accepted & M) : 0ull;
        const uint64_t O = (mine && !leaf) ? (M & ~accepted) : 0ull;
        const uint64_t pushb = __ballot(O != 0);
        if (O != 0) {
            const int e = sp + (int)lanes_below(pushb);
            if (check_ok(e < kStack, CK_STACK)) {
                L.st_c0[e] = info.child0;
                L.st_n[e] = (uint8_t)node_nchild(info);
                L.st_mask[e] = O;
            }
        }
        sp += __popcll(pushb);
        const bool hasq = leaf || A != 0;
        const uint64_t qb = __ballot(hasq);
        if (qb) {
            // room in the ring for the round: wait for the evaluating waves
            const uint32_t need = dq_tail + (uint32_t)__popcll(qb);
            while ((int32_t)(need - freed) > kRing) {
                // the smallest head: lane e reads wave e's
                uint32_t h = 0;
                if (lane < kEvals)
                    h = __hip_atomic_load(&L.head[lane], __ATOMIC_ACQUIRE,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
                freed = (uint32_t)__builtin_amdgcn_readlane((int)h, 0);
                for (int e = 1; e < kEvals; e++) {
                    const uint32_t he = (uint32_t)__builtin_amdgcn_readlane((int)h, e);
                    if ((int32_t)(he - freed) < 0) freed = he;
                }
                if ((int32_t)(need - freed) > kRing) __builtin_amdgcn_s_sleep(kPollSleep);
            }
            const uint32_t nitems = leaf ? (uint32_t)info.count : (A != 0 ? 1u : 0u);
            const uint32_t incl = wave_incl_scan(nitems);
            if (hasq) {
                const uint32_t d = (dq_tail + lanes_below(qb)) & (kRing - 1);
                L.dq_a[d] = leaf ? info.first : ~k;
                L.dq_r[d] = DqRange{queued + incl - nitems, (int32_t)nitems};
                L.dq_mask[d] = leaf ? M : A;
            }
            dq_tail = need;
            queued += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            BHX_CHECK((int32_t)(dq_tail - freed) <= kRing, CK_RING);
        }
        const uint64_t pub = (uint64_t)(dq_tail | (sp == 0 ? kDone : 0u)) << 32 | queued;
        if (lane == 0)
            __hip_atomic_store(&L.published, pub, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// An evaluating wave's view of the queue: its next batch.
struct Batch {
    uint32_t start = 0;  // running number of its first item
    uint32_t head = 0;   // first descriptor not used up before it
    uint32_t tail = 0;   // descriptors written
    int count = 0;       // its items, at most 64
};

// Moves head past the descriptors used up before start (they form a prefix).
template <int kStack>
__device__ inline void skip_used(const Lds<kStack> &L, Batch &b)
{
    const int lane = threadIdx.x & 63;
    for (;;) {
        const uint32_t d = b.head + lane;
        bool used = false;
        if ((int32_t)(b.tail - d) > 0) {
            const DqRange r = L.dq_r[d & (kRing - 1)];
            used = (int32_t)(r.at + (uint32_t)r.n - b.start) <= 0;
        }
        const int k = __popcll(__ballot(used));
        b.head += (uint32_t)k;
        if (k < 64) break;
    }
}

template <int kStack>
__device__ inline void publish_head(Lds<kStack> &L, int e, const Batch &b)
{
    wave_sync();
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(&L.head[e], b.head, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Wave e waits for items start .. start + 63, or for the end of the traversal;
// false when no item is left. The traversal ends after finitely many rounds and
// waits only for ring space, which a wave waiting here gives back as it learns
// of descriptors that are not its own (see Lds).
template <int kStack>
__device__ inline bool next_batch(Lds<kStack> &L, int e, Batch &b)
{
    uint32_t queued, seen = ~0u;  // no tail has this value
    for (;;) {
        const uint64_t pub =
            __hip_atomic_load(&L.published, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        queued = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)pub);
        const uint32_t tail = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(pub >> 32));
        b.tail = tail & ~kDone;
        if ((int32_t)(queued - b.start) >= kBatch || (tail & kDone)) break;
        if (b.tail != seen) {  // new descriptors: give back those before start
            seen = b.tail;
            const uint32_t was = b.head;
            skip_used(L, b);
            if (b.head != was) publish_head(L, e, b);
        }
        __builtin_amdgcn_s_sleep(kPollSleep);
    }
    b.count = min((int32_t)(queued - b.start), kBatch);
    if (b.count <= 0) return false;
    skip_used(L, b);  // the batches in between
    return true;
}

// Lane L < count of the wave gets item start + L of the batch: its descriptor's
// source (a body, or ~node) and body mask. A batch needs at most 64
// descriptors; each that starts inside it flags the lane of its first item
// (one forward lane permute; the head's item 0 needs no flag, and lanes
// without one write there), and a ballot of the flags gives every lane its
// descriptor. Moves head past the descriptors that the batch uses up, tells
// the traversal (`e`: this wave's number) and moves start on.
template <int kStack>
__device__ __forceinline__ void take_batch(Lds<kStack> &L, int e, Batch &b, int32_t &src,
                                           uint64_t &mask)
{
    const int lane = threadIdx.x & 63;
    const uint32_t d = b.head + lane;
    const bool in = (int32_t)(b.tail - d) > 0;
    DqRange r{0u, 0};
    if (in) r = L.dq_r[d & (kRing - 1)];
    const uint32_t rel = r.at - b.start;
    const bool flag = lane > 0 && in && rel < (uint32_t)b.count;
    const uint64_t starts =
        __ballot(__builtin_amdgcn_ds_permute(flag ? (int)rel << 2 : 0, flag ? 1 : 0) != 0) & ~1ull;
    const uint32_t dsel = lanes_below(starts) + (uint32_t)((starts >> lane) & 1ull);
    mask = 0;
    src = 0;
    if (lane < b.count) {
        const uint32_t at = (b.head + dsel) & (kRing - 1);
        const int32_t a = L.dq_a[at];
        mask = L.dq_mask[at];
        src = a < 0 ? a : a + (int32_t)(b.start + (uint32_t)lane - L.dq_r[at].at);
    }
    const bool used = in && (int32_t)(r.at + (uint32_t)r.n - (b.start + (uint32_t)b.count)) <= 0;
    b.head += (uint32_t)__popcll(__ballot(used));
    publish_head(L, e, b);
    b.start += (uint32_t)(kBatch * kEvals);
}

}  // namespace walkx
}  // namespace bhx
