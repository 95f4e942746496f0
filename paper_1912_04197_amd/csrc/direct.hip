// Direct N^2 sum, eq. (Newton) with every term softened as in
// eq. (Force_rComp): a_i = G sum_{j != i} m_j d_ij / (|d_ij|^2 + eps_ij^2)^(3/2).
//
// Sources are summed in groups of 32, staged in LDS; positions stay FP64, so
// that d_ij is formed in FP64 even in FP32C mode, where only the pair
// arithmetic after the difference is FP32 and the FP32 partial sums of one
// group are added into FP64 accumulators. Two kernels sweep the groups:
//   k_direct        a block's four waves share 128 targets (two per lane) and
//                   take the groups of a 256-source tile in turn; where the
//                   targets give too few blocks to fill the GPU, block row y
//                   sums the y-th range of tiles into a partial buffer, and a
//                   second kernel adds the rows in order;
//   k_direct_small  up to kDirectSmall bodies: a block serves 8 or 16
//                   targets and all sources, its lanes sharing the groups, so
//                   that one launch fills the GPU and nothing is added later.
// Every sum has a fixed order, so results do not depend on scheduling.
#include <cmath>
#include <mutex>
#include <type_traits>

#include "bhx_impl.h"

namespace bhx {
namespace {

constexpr int kGroup = 32;  // sources of one FP32C partial sum
constexpr int kTile = 256;  // sources staged at a time by k_direct
constexpr int kTargets = 2;              // targets per lane of k_direct
constexpr int kBlockTargets = 64 * kTargets;

// One source as LDS holds it, read from one address with immediate offsets.
template <bool PEPS>
struct alignas(16) SrcD {  // FP64: position, mass
    double x, y, z, m;
};
template <>
struct alignas(16) SrcD<true> {  // and half the squared softening
    double x, y, z, m, eh, pad;
};
struct alignas(16) SrcF {  // FP32C: FP64 position; FP32 mass and half squared softening
    double x, y, z;
    float m, eh;
};
template <int PREC, bool PEPS>
using Src = typename std::conditional<PREC == BH_FP64, SrcD<PEPS>, SrcF>::type;

template <int PREC, bool PEPS>
__device__ inline Src<PREC, PEPS> load_source(const double *__restrict__ pos,
                                              const double *__restrict__ mass,
                                              const double *__restrict__ eps, int64_t j)
{
    double eh = 0.0;
    if (PEPS) {
        const double e = eps[j];
        eh = 0.5 * (e * e);
    }
    Src<PREC, PEPS> q;
    q.x = pos[3 * j];
    q.y = pos[3 * j + 1];
    q.z = pos[3 * j + 2];
    if constexpr (PREC == BH_FP64) {
        q.m = mass[j];
        if constexpr (PEPS) q.eh = eh;
    } else {  // the FP32 operands, rounded once per source
        q.m = (float)mass[j];
        q.eh = (float)eh;
    }
    return q;
}

struct Target {
    double x, y, z;
    double eh;  // half the squared softening: (eps_i^2 + eps_j^2) / 2 = eh_i + eh_j exactly
    float ehf;
    double ax, ay, az, ph;  // sums
};

// Whether a pair has to be looked at before it is added. A group in which no
// target meets itself needs no index test. In FP32C, where every pair's FP32
// softening is a positive normal number, so is its r^2, and the r^2 test is
// dropped too; other FP32C pairs are tested one by one. In FP64 the pairs of a
// group are tested together, by their factors m r^-3: a pair counts if that is a
// normal number, which it is only of a positive normal r^2 and in the number range, or
// zero with the mass. Where no factor can underflow (kPlain) the rest is seen in the
// sums: a factor that is infinite or not a number leaves none of them finite. Only a
// group with a dead or extreme pair takes them singly.
enum { kPlain = 0, kTest = 1, kSkip = 2 };

// Adds the terms of `cnt` sources at q to the T targets of this lane. skip[t]
// (kSkip only): target t's own place in the group, or outside 0..cnt-1.
//
// Bound by VALU issue (a wave64 FP32 or FP64 operation takes about four cycles
// of its SIMD). An FP32C pair takes 16 instructions softened and 18 unsoftened,
// where testing every pair's index and r^2 took 19; an FP64 pair 17 (18 with a test
// of every pair), where two Newton steps, the cube and m d r^-3 per axis took 27. Two
// targets per lane halve the LDS reads (two ds_read_b128 per source), which kept the
// LDS pipe 62 % busy with one. 65536 bodies, one sum, before and after: FP32C 2.19 ->
// 1.76 ms (per-body softening), 2.14 -> 1.65 ms (one softening), FP64 4.43 ->
// 2.61 ms (2.73 with the test).
template <int PREC, bool PEPS, bool PHI, int T, int MODE, bool FULL>
__device__ __forceinline__ void sum_group(const Src<PREC, PEPS> *q, int cnt, Target (&tg)[T],
                                          double eps0sq, float eps0f, const int (&skip)[T])
{
    if (FULL) cnt = kGroup;
    if constexpr (PREC == BH_FP64) {
        const CubeConsts k = cube_consts();
        auto one = [&](const Src<PREC, PEPS> &s, Target &g, int jj, int own) {
            const double dx = s.x - g.x, dy = s.y - g.y, dz = s.z - g.z;
            double e2 = eps0sq;
            if constexpr (PEPS) e2 = g.eh + s.eh;
            const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, e2)));
            double i5, i2;
            if (MODE != kSkip || jj != own)
                pair_term_f64<PHI>(s.m, dx, dy, dz, r2, g.ax, g.ay, g.az, g.ph, i5, i2);
        };
        if constexpr (FULL) {
            // every pair live but a target's own: the group's sums, kept if so
            double sx[T], sy[T], sz[T], sp[T];
#pragma unroll
            for (int t = 0; t < T; t++) sx[t] = sy[t] = sz[t] = sp[t] = 0.0;
            bool live = true;
#pragma unroll 2
            for (int jj = 0; jj < kGroup; jj++) {
                const Src<PREC, PEPS> s = q[jj];
                // classes of a good factor: normal numbers, and with a massless source zeros
                const int numbers = s.m == 0.0 ? 0x168 : 0x108;
#pragma unroll
                for (int t = 0; t < T; t++) {
                    const bool own = MODE == kSkip && jj == skip[t];  // d = 0 there
                    const double dx = s.x - tg[t].x, dy = s.y - tg[t].y, dz = s.z - tg[t].z;
                    double e2 = eps0sq;
                    if constexpr (PEPS) e2 = tg[t].eh + s.eh;
                    const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, e2)));
                    double ri;
                    double c = s.m * inv_cube_f64<PHI>(r2, ri, k);
                    if (MODE != kPlain)
                        live = live && (own || __builtin_amdgcn_class(c, numbers));
                    if (own) c = ri = 0.0;
                    sx[t] = fma(c, dx, sx[t]);
                    sy[t] = fma(c, dy, sy[t]);
                    sz[t] = fma(c, dz, sz[t]);
                    if (PHI) sp[t] -= s.m * ri;
                }
            }
            if (MODE == kPlain)
#pragma unroll
                for (int t = 0; t < T; t++) live = live && isfinite(sx[t] + sy[t] + sz[t]);
            if (__ballot(!live) == 0) {
#pragma unroll
                for (int t = 0; t < T; t++) {
                    tg[t].ax += sx[t];
                    tg[t].ay += sy[t];
                    tg[t].az += sz[t];
                    if (PHI) tg[t].ph += sp[t];
                }
                return;
            }
        }
#pragma unroll 1
        for (int jj = 0; jj < cnt; jj++) {
            const Src<PREC, PEPS> s = q[jj];
#pragma unroll
            for (int t = 0; t < T; t++) one(s, tg[t], jj, MODE == kSkip ? skip[t] : -1);
        }
    } else {
        float fx[T], fy[T], fz[T], fp[T];
#pragma unroll
        for (int t = 0; t < T; t++) fx[t] = fy[t] = fz[t] = fp[t] = 0.f;
#pragma unroll(FULL ? 4 : 1)
        for (int jj = 0; jj < cnt; jj++) {
            const SrcF s = q[jj];
#pragma unroll
            for (int t = 0; t < T; t++) {
                const float dx = (float)(s.x - tg[t].x), dy = (float)(s.y - tg[t].y),
                            dz = (float)(s.z - tg[t].z);
                const float e2 = PEPS ? s.eh + tg[t].ehf : eps0f;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, e2)));
                float rinv = __builtin_amdgcn_rsqf(r2);
                if (MODE != kPlain)
                    rinv = positive_normal_f(r2) && (MODE != kSkip || jj != skip[t]) ? rinv : 0.f;
                const float mr = s.m * rinv;
                const float mr3 = mr * rinv * rinv;
                fx[t] = fmaf(mr3, dx, fx[t]);
                fy[t] = fmaf(mr3, dy, fy[t]);
                fz[t] = fmaf(mr3, dz, fz[t]);
                if (PHI) fp[t] -= mr;
            }
        }
#pragma unroll
        for (int t = 0; t < T; t++) {
            tg[t].ax += (double)fx[t];
            tg[t].ay += (double)fy[t];
            tg[t].az += (double)fz[t];
            if (PHI) tg[t].ph += (double)fp[t];
        }
    }
}

// The same, choosing the form: `own` (the same on every active lane) where a
// target may be among the sources, `plain` (the same on every active lane) where
// every pair of the group is as kPlain asks.
template <int PREC, bool PEPS, bool PHI, int T>
__device__ __forceinline__ void add_group(const Src<PREC, PEPS> *q, int cnt, bool full,
                                          Target (&tg)[T], double eps0sq, float eps0f,
                                          const int (&skip)[T], bool own, bool plain)
{
    if (!full)
        sum_group<PREC, PEPS, PHI, T, kSkip, false>(q, cnt, tg, eps0sq, eps0f, skip);
    else if (own)
        sum_group<PREC, PEPS, PHI, T, kSkip, true>(q, cnt, tg, eps0sq, eps0f, skip);
    else if (plain)
        sum_group<PREC, PEPS, PHI, T, kPlain, true>(q, cnt, tg, eps0sq, eps0f, skip);
    else
        sum_group<PREC, PEPS, PHI, T, kTest, true>(q, cnt, tg, eps0sq, eps0f, skip);
}

template <bool PEPS>
__device__ inline Target load_target(const double *__restrict__ pos,
                                     const double *__restrict__ eps, int64_t i)
{
    Target g;
    g.x = pos[3 * i];
    g.y = pos[3 * i + 1];
    g.z = pos[3 * i + 2];
    g.eh = 0.0;
    if (PEPS) {
        const double e = eps[i];
        g.eh = 0.5 * (e * e);
    }
    g.ehf = (float)g.eh;
    g.ax = g.ay = g.az = g.ph = 0.0;
    return g;
}

// Targets and sources whose groups may be plain. FP32C: the target's softening makes
// every r^2 a positive normal FP32 number if the source's half is a number (not NaN).
// FP64: lengths and masses keep every factor but that of a massless source above 2^-910.
template <int PREC, bool PEPS>
__device__ inline bool plain_target(const Target &g, double eps0sq, float eps0f)
{
    if (PREC == BH_FP64)
        return fabs(g.x) + fabs(g.y) + fabs(g.z) <= 0.5 * kMildLength &&
               (PEPS ? g.eh : eps0sq) <= kMildEps2;
    return positive_normal_f(PEPS ? g.ehf : eps0f);
}
template <int PREC, bool PEPS>
__device__ inline bool plain_source(const Src<PREC, PEPS> &s)
{
    if constexpr (PREC == BH_FP64) {
        bool ok = fabs(s.x) + fabs(s.y) + fabs(s.z) <= 0.5 * kMildLength &&
                  (s.m == 0.0 || fabs(s.m) >= kMildMassMin);
        if constexpr (PEPS) ok = ok && s.eh <= kMildEps2;
        return ok;
    } else {
        return !PEPS || s.eh >= 0.f;
    }
}

template <int PREC, bool PEPS, bool PHI>
__global__ __launch_bounds__(256) void k_direct(const double *__restrict__ pos,
                                                const double *__restrict__ mass,
                                                const double *__restrict__ eps, int64_t n,
                                                double eps0sq, double G,
                                                double *__restrict__ acc,
                                                double *__restrict__ phi, int64_t chunk,
                                                double *__restrict__ part)
{
    using S = Src<PREC, PEPS>;
    __shared__ S src[kTile];
    __shared__ bool group_ok[kTile / kGroup];  // the group's sources are plain
    __shared__ double red[3][4][kBlockTargets];  // the other waves' sums
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * kBlockTargets;
    Target tg[kTargets];
    int64_t ti[kTargets];
    const float eps0f = (float)eps0sq;
    bool plain = true;
#pragma unroll
    for (int t = 0; t < kTargets; t++) {
        ti[t] = b0 + 64 * t + lane;
        // lanes past the end repeat the last target; nothing of theirs is stored
        tg[t] = load_target<PEPS>(pos, eps, ti[t] < n ? ti[t] : n - 1);
        plain = plain && plain_target<PREC, PEPS>(tg[t], eps0sq, eps0f);
    }
    plain = __ballot(!plain) == 0;
    // this block row's sources: [s_lo, s_hi)
    const int64_t s_lo = (int64_t)blockIdx.y * chunk;
    const int64_t s_hi = s_lo + chunk < n ? s_lo + chunk : n;
    for (int64_t base = s_lo; base < s_hi; base += kTile) {
        const int64_t j = base + tid;
        if (j < s_hi) {
            const S s = load_source<PREC, PEPS>(pos, mass, eps, j);
            src[tid] = s;
            // half a wave loads a group
            const uint64_t odd = __ballot(!plain_source<PREC, PEPS>(s));
            if (tid % kGroup == 0) group_ok[tid / kGroup] = (uint32_t)(odd >> (lane & 32)) == 0;
        }
        __syncthreads();
        const int cnt = (int)((s_hi - base) < kTile ? (s_hi - base) : kTile);
        const bool own = base < b0 + kBlockTargets && base + cnt > b0;
#pragma unroll 1
        for (int g = wave; g * kGroup < cnt; g += 4) {
            const int gc = cnt - g * kGroup < kGroup ? cnt - g * kGroup : kGroup;
            int skip[kTargets];
#pragma unroll
            for (int t = 0; t < kTargets; t++) {
                const int64_t at = ti[t] - base - g * kGroup;
                skip[t] = own && at >= 0 && at < gc ? (int)at : -1;
            }
            add_group<PREC, PEPS, PHI, kTargets>(src + g * kGroup, gc, gc == kGroup, tg, eps0sq,
                                                 eps0f, skip, own, plain && group_ok[g]);
        }
        __syncthreads();
    }
    // the waves' sums in wave order
    if (wave > 0)
#pragma unroll
        for (int t = 0; t < kTargets; t++) {
            double(*r)[kBlockTargets] = red[wave - 1];
            r[0][64 * t + lane] = tg[t].ax;
            r[1][64 * t + lane] = tg[t].ay;
            r[2][64 * t + lane] = tg[t].az;
            if (PHI) r[3][64 * t + lane] = tg[t].ph;
        }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int t = 0; t < kTargets; t++) {
        const int64_t i = ti[t];
        if (i >= n) continue;
        double ax = tg[t].ax, ay = tg[t].ay, az = tg[t].az, ph = tg[t].ph;
#pragma unroll
        for (int w = 0; w < 3; w++) {
            ax += red[w][0][64 * t + lane];
            ay += red[w][1][64 * t + lane];
            az += red[w][2][64 * t + lane];
            if (PHI) ph += red[w][3][64 * t + lane];
        }
        if (gridDim.y == 1) {
            acc[3 * i] = G * ax;
            acc[3 * i + 1] = G * ay;
            acc[3 * i + 2] = G * az;
            if (PHI) phi[i] = G * ph;
        } else {
            double *q = part + 4 * ((int64_t)blockIdx.y * n + i);
            q[0] = ax;
            q[1] = ay;
            q[2] = az;
            q[3] = ph;
        }
    }
}

// acc_i = G * sum over the block rows of their partial sums, in row order;
// one thread per target and component, so that a wave reads whole lines.
__global__ __launch_bounds__(256) void k_direct_reduce(const double *__restrict__ part,
                                                       int64_t n, int rows, double G,
                                                       double *__restrict__ acc,
                                                       double *__restrict__ phi)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t i = t >> 2;
    const int c = (int)(t & 3);
    if (i >= n || (c == 3 && !phi)) return;
    double s = 0.0;
#pragma unroll 8
    for (int r = 0; r < rows; r++) s += part[4 * (int64_t)r * n + t];
    if (c == 3)
        phi[i] = G * s;
    else
        acc[3 * i + c] = G * s;
}

// Up to kDirectSmall bodies: 512 threads serve TG targets; lane l of wave w is
// share w (64 / TG) + l / TG of target l % TG and sums every S-th group of
// sources, S = 512 / TG shares, the S groups of a step staged in LDS (each
// group 16 bytes past a multiple of 256, so that the shares of a wave read
// from distinct banks).
constexpr int kSmallThreads = 512;
template <int PREC, bool PEPS, bool PHI, int TG>
__global__ __launch_bounds__(kSmallThreads) void k_direct_small(
    const double *__restrict__ pos, const double *__restrict__ mass,
    const double *__restrict__ eps, int n, double eps0sq, double G, double *__restrict__ acc,
    double *__restrict__ phi)
{
    using S = Src<PREC, PEPS>;
    constexpr int kShares = kSmallThreads / TG, kWaveShares = 64 / TG, W = kSmallThreads / 64;
    constexpr int kStride = kGroup * (int)sizeof(S) + 16;
    static_assert((kGroup * sizeof(S)) % 256 == 0, "group stride");
    __shared__ alignas(16) char tile[kShares * kStride];
    __shared__ double red[W][4][TG];
    __shared__ bool group_ok[kShares];  // the group's sources are plain
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tl = lane % TG, share = wave * kWaveShares + lane / TG;
    const int b0 = (int)blockIdx.x * TG, i = b0 + tl;
    const float eps0f = (float)eps0sq;
    Target tg[1] = {load_target<PEPS>(pos, eps, i < n ? i : n - 1)};
    const bool plain = __ballot(!plain_target<PREC, PEPS>(tg[0], eps0sq, eps0f)) == 0;
    for (int base = 0; base < n; base += kShares * kGroup) {
        const int in = n - base < kShares * kGroup ? n - base : kShares * kGroup;
        for (int k = tid; k < in; k += kSmallThreads) {
            const S s = load_source<PREC, PEPS>(pos, mass, eps, base + k);
            *(S *)(tile + (k / kGroup) * kStride + (k % kGroup) * (int)sizeof(S)) = s;
            // half a wave loads a group
            const uint64_t odd = __ballot(!plain_source<PREC, PEPS>(s));
            if (k % kGroup == 0) group_ok[k / kGroup] = (uint32_t)(odd >> (lane & 32)) == 0;
        }
        __syncthreads();
        const int left = in - share * kGroup;
        const int cnt = left < 0 ? 0 : left < kGroup ? left : kGroup;
        const int at = i - base - share * kGroup;
        const int skip[1] = {at >= 0 && at < cnt ? at : -1};
        // uniform over the wave: whether any of its shares holds one of the
        // block's targets, and whether all its groups are whole
        const int g0 = base + share * kGroup;
        const bool own = __ballot(g0 < b0 + TG && g0 + cnt > b0) != 0;
        const bool full = __ballot(cnt != kGroup) == 0;
        const bool tile_ok = __ballot(cnt > 0 && !group_ok[share]) == 0;
        if (__ballot(cnt > 0) != 0)
            add_group<PREC, PEPS, PHI, 1>((const S *)(tile + share * kStride), cnt, full, tg,
                                          eps0sq, eps0f, skip, own, plain && tile_ok);
        __syncthreads();
    }
    // the shares in a fixed order: over the wave, then over the waves
    double v[4] = {tg[0].ax, tg[0].ay, tg[0].az, tg[0].ph};
#pragma unroll
    for (int o = TG; o < 64; o <<= 1)
#pragma unroll
        for (int c = 0; c < (PHI ? 4 : 3); c++) v[c] += __shfl_xor(v[c], o);
    if (lane < TG)
#pragma unroll
        for (int c = 0; c < (PHI ? 4 : 3); c++) red[wave][c][lane] = v[c];
    __syncthreads();
    const int c = tid / TG;  // one thread per target and component
    if (c >= (PHI ? 4 : 3) || b0 + tid % TG >= n) return;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; w++) s += red[w][c][tid % TG];
    const int64_t o = b0 + tid % TG;
    if (c == 3)
        phi[o] = G * s;
    else
        acc[3 * o + c] = G * s;
}

template <int PREC, bool PEPS, bool PHI>
hipError_t launch_t(hipStream_t s, const double *pos, const double *mass, const double *eps,
                    int64_t n, double eps0sq, double G, double *acc, double *phi, double *part)
{
    if (n <= kDirectSmall) {
        // the fewest targets per block that keep the blocks near one per CU:
        // one sum of 2048 bodies 41 -> 12 us in FP64 (64 blocks of 256 targets
        // and the row sums' launch before), 21 -> 11 us in FP32C; 4096 bodies
        // 43 -> 21 and 23 -> 16 us. Above, k_direct's rows fill the GPU and its
        // two targets per lane win (6000 bodies in FP64: 36 us against 50 here
        // with 32 targets per block)
        if (n <= 2048)
            k_direct_small<PREC, PEPS, PHI, 8><<<(unsigned)((n + 7) / 8), kSmallThreads, 0, s>>>(
                pos, mass, eps, (int)n, eps0sq, G, acc, phi);
        else
            k_direct_small<PREC, PEPS, PHI, 16>
                <<<(unsigned)((n + 15) / 16), kSmallThreads, 0, s>>>(pos, mass, eps, (int)n,
                                                                     eps0sq, G, acc, phi);
        return hipGetLastError();
    }
    // rows of source ranges (whole tiles): as many as the partial buffer holds and at
    // least a tile each, which makes at most about 2048 blocks (eight a CU): 561 at 4097
    // bodies, 2048 at 8192, 1564 at 100,000 (two whole rows), 1025 (one) above 131,072
    const int64_t tb = (n + kBlockTargets - 1) / kBlockTargets;
    const int64_t all = (n + kTile - 1) / kTile;
    int64_t rows = part ? kDirectPart / (4 * n) : 1;
    if (rows < 1) rows = 1;
    if (rows > all) rows = all;  // at least one source tile per row
    const int64_t tiles = (all + rows - 1) / rows;
    rows = (all + tiles - 1) / tiles;
    const dim3 grid((unsigned)tb, (unsigned)rows);
    k_direct<PREC, PEPS, PHI><<<grid, 256, 0, s>>>(pos, mass, eps, n, eps0sq, G, acc, phi,
                                                   rows == 1 ? n : tiles * kTile, part);
    if (rows > 1)
        k_direct_reduce<<<(unsigned)((4 * n + 255) / 256), 256, 0, s>>>(part, n, (int)rows, G, acc,
                                                                        phi);
    return hipGetLastError();
}

template <int PREC, bool PEPS>
hipError_t launch_p(hipStream_t s, const double *pos, const double *mass, const double *eps,
                    int64_t n, double eps0sq, double G, double *acc, double *phi, double *part)
{
    return phi ? launch_t<PREC, PEPS, true>(s, pos, mass, eps, n, eps0sq, G, acc, phi, part)
               : launch_t<PREC, PEPS, false>(s, pos, mass, eps, n, eps0sq, G, acc, phi, part);
}

}  // namespace

hipError_t launch_direct(hipStream_t s, const double *pos, const double *mass, const double *eps,
                         int64_t n, double eps0sq, double G, int precision, double *acc,
                         double *phi, double *part)
{
    if (n <= 0) return hipSuccess;
    if (precision == BH_FP64)
        return eps ? launch_p<BH_FP64, true>(s, pos, mass, eps, n, eps0sq, G, acc, phi, part)
                   : launch_p<BH_FP64, false>(s, pos, mass, eps, n, eps0sq, G, acc, phi, part);
    return eps ? launch_p<BH_FP32C, true>(s, pos, mass, eps, n, eps0sq, G, acc, phi, part)
               : launch_p<BH_FP32C, false>(s, pos, mass, eps, n, eps0sq, G, acc, phi, part);
}

}  // namespace bhx

// ------------------------------------------------- no-allocation entry point

namespace {

// The split-row partial sums of bh_compute_accel_direct_noalloc: one array
// per device, held by the library until the process ends and shared by every
// call on that device (calls that overlap on one device race on it).
__device__ __align__(256) double scratch[bhx::kDirectPart];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch[kMaxDevices] = {};

// The device address of this device's scratch array (the array's name is
// only a host-side stand-in), looked up once per device with it current.
bh_status scratch_ptr(double **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BH_E_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return BH_E_HIP;
        g_scratch[dev] = static_cast<double *>(ptr);
    }
    *out = g_scratch[dev];
    return BH_OK;
}

}  // namespace

extern "C" bh_status bh_compute_accel_direct_noalloc(void *hip_stream, int32_t precision,
                                                     double G, const double *pos,
                                                     const double *mass, double softening,
                                                     const double *eps, double *acc, double *phi,
                                                     int64_t n)
{
    if (n < 0 || n > BH_NOALLOC_MAX_N) return BH_E_CAPACITY;
    if (precision != BH_FP64 && precision != BH_FP32C) return BH_E_INVALID;
    if (!std::isfinite(G)) return BH_E_INVALID;
    if (!(std::isfinite(softening) && softening >= 0.0)) return BH_E_INVALID;
    if (n > 0 && (!pos || !mass || !acc)) return BH_E_INVALID;
    if (n == 0) return BH_OK;
    double *part = nullptr;
    const bh_status st = scratch_ptr(&part);
    if (st != BH_OK) return st;
    // every partial sum is written before it is read (no clearing needed):
    // row r of the split writes 4 doubles for each of the n targets
    const hipError_t e = bhx::launch_direct((hipStream_t)hip_stream, pos, mass, eps, n,
                                            softening * softening, G, precision, acc, phi, part);
    return e == hipSuccess ? BH_OK : BH_E_HIP;
}
