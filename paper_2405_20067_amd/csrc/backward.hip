// Analytic backward pass (Sec. 4.1): gradients of every Gaussian's mean,
// factor, weight and colour given g = dl/df.
//
// With y = L^-1 d (d = x - m), G = exp(-|y|^2/2), s = g . c, w = alpha G s,
// z = L^-T y:
//   dl/dalpha = c . H,  dl/dc = alpha H,        H  = sum_x G g
//   dl/dm     = L^-T B1 = S^T B1,               B1 = sum_x w y
//   dl/dL     = tril(S^T B2),                   B2 = sum_x w y y^T
// (dl/dm = sum w z and dl/dL = tril(sum w z y^T) with z = S^T y.)
//
// Atomics-free and Gaussian-major.  Culled: the forward pass records, for
// every candidate entry (tile, Gaussian) and every 64-query group of the
// tile, whether it kept the pair group (one byte); the backward visits only
// the kept groups, so it sums over exactly the pairs the forward summed,
// recomputing y, G and the exp rather than storing them.  In large mixtures
// (backward_light) a Gaussian to which a handful of queries add anything takes
// those alone (k_light_moments, k_light_gradients); the others go to work items,
// as all do elsewhere.  A work item is one
// Gaussian and at most kItemTiles of its candidate entries (the transposed
// lists); one wave evaluates the item's kept groups 64 queries at a time,
// keeps per-lane partial moments in registers (B1: n, B2: n(n+1)/2, H: 3),
// reduces them across lanes once and writes them to the item's slot.
// k_backward_finalize then adds each Gaussian's items in item order and
// applies S^T.  Dense: one to sixteen waves per Gaussian over all queries.
#include <algorithm>
#include <type_traits>

#include "eval_common.hpp"
#include "ngd_internal.hpp"
#include "wave.hpp"

namespace ngd {
namespace {

constexpr int kBwdThreads = 256;
constexpr int kMaxGroups = 16;   // 64-query groups of the largest tile (1024)
constexpr int64_t kBwdItemBlocks = 4096;
constexpr int kWavesPerBlock = kBwdThreads / kWave;
static_assert(kItemTiles <= kWave, "an item's tile list must fit one wave");

// ---- dense: every Gaussian over all queries --------------------------------
// W waves per Gaussian, PER Gaussians per workgroup; a Gaussian's waves take
// the 64-query blocks in turn (lane = query), keep per-lane moments and reduce
// them over the lanes, then over the waves in order through LDS, and its first
// threads form the outputs.  With W waves per Gaussian a mixture of a few
// hundred Gaussians fills the chip: with one wave per Gaussian the loads of each
// block waited in a single chain (K = 256, Q = 65,536, n = 4: 327 us, now 28,
// against 17 us of vector operations).  No workspace, so calls
// on several streams stay independent.
template <int N, int W, int PER>
__global__ __launch_bounds__(PER *W *kWave) void k_backward_dense(
    int64_t first, int64_t k, int64_t q, const float *__restrict__ rec,
    const float *__restrict__ xq, const float *__restrict__ gq, float *__restrict__ g_mean,
    float *__restrict__ g_factor, float *__restrict__ g_weight, float *__restrict__ g_colour)
{
    constexpr int T = N * (N + 1) / 2;
    constexpr int R = (N + T + 7 + 3) / 4 * 4;
    constexpr int NM = N + T + 3;   // B1 | B2 | H
    constexpr int VP = (NM + 3) & ~3, Q4 = VP / 4;
    constexpr int AL = N + T + 3, CO = N + T + 4;
    __shared__ float s_part[PER][W][VP];
    const int lane = lane_id(), w = int(threadIdx.x) / kWave % W;
    const int own = uniform(int(threadIdx.x) / (W * kWave));
    const int64_t gi = (first + blockIdx.x) * PER + own;
    const int64_t g = gi < k ? gi : k - 1;   // past the end the last one, not stored
    auto &part = s_part[own];
    const float *__restrict__ r = rec + g * R;
    const float alpha = r[AL], c0 = r[CO], c1 = r[CO + 1], c2 = r[CO + 2];

    float mv[VP];
#pragma unroll
    for (int e = 0; e < VP; ++e) mv[e] = 0.0f;
    // 64 queries from b; FULL: all of them there, otherwise a lane past the end
    // repeats the last with nothing upstream
    auto block = [&]<bool FULL>(int64_t b) {
        const bool valid = FULL || b + lane < q;
        // (loaded from 64-bit addresses and without a condition, the three values
        // by one load: three took twice the time in few dimensions)
        const int64_t p = valid ? b + lane : q - 1;
        const float *__restrict__ xp = xq + p * N, *__restrict__ gp = gq + p * 3;
        float d[N], y[N];
#pragma unroll
        for (int a = 0; a < N; ++a) d[a] = xp[a];
        const float u0 = gp[0], u1 = gp[1], u2 = gp[2];
        const float g0 = valid ? u0 : 0.0f, g1 = valid ? u1 : 0.0f, g2 = valid ? u2 : 0.0f;
        float msq = 0.0f;
#pragma unroll
        for (int row = 0; row < N; ++row) {
            d[row] -= r[row];
            const float *srow = r + N + row * (row + 1) / 2;
            float acc = srow[0] * d[0];
#pragma unroll
            for (int j = 1; j <= row; ++j) acc = fmaf(srow[j], d[j], acc);
            y[row] = acc;
            msq = fmaf(acc, acc, msq);
        }
        const float G = valid ? __builtin_amdgcn_exp2f(-msq) : 0.0f;
        const float sdot = fmaf(g2, c2, fmaf(g1, c1, g0 * c0));
        const float wt = alpha * G * sdot;
        mv[N + T + 0] = fmaf(G, g0, mv[N + T + 0]);
        mv[N + T + 1] = fmaf(G, g1, mv[N + T + 1]);
        mv[N + T + 2] = fmaf(G, g2, mv[N + T + 2]);
#pragma unroll
        for (int a = 0; a < N; ++a) {
            const float wy = wt * y[a];
            mv[a] += wy;
#pragma unroll
            for (int c = 0; c <= a; ++c)
                mv[N + a * (a + 1) / 2 + c] = fmaf(wy, y[c], mv[N + a * (a + 1) / 2 + c]);
        }
    };
    int64_t b = int64_t(uniform(w)) * kWave;
    for (; b + kWave <= q; b += W * kWave) block.template operator()<true>(b);
    if (b < q) block.template operator()<false>(b);
    // lane 16 i + 15 holds the totals of the i-th quarter
    wave_reduce_scatter<VP>(mv);
    if ((lane & 15) == 15) {
        const int r0 = (lane >> 4) * Q4;
#pragma unroll
        for (int i = 0; i < Q4; ++i) part[w][r0 + i] = mv[i];
    }
    __syncthreads();
    const int t = int(threadIdx.x) % (W * kWave);
    for (int e = t; W > 1 && e < NM; e += W * kWave) {
        float acc = part[0][e];
#pragma unroll
        for (int i = 1; i < W; ++i) acc += part[i][e];
        part[0][e] = acc;   // this thread's own column
    }
    __syncthreads();
    // S = S' / sqrt(c), y = y' / sqrt(c), c = log2(e)/2:
    //   S^T B1 = S'^T B1' / c,  S^T B2 = S'^T B2' / c^1.5
    const float inv_c = float(1.0 / kHalfLog2e);
    const float inv_c15 = float(1.0 / (kHalfLog2e * kSqrtHalfLog2e));
    const float *tot = part[0];
    for (int e = t; e < NM + 1 && gi < k; e += W * kWave) {
        if (e < N) {
            float acc = 0.0f;
            for (int kk = e; kk < N; ++kk) acc = fmaf(r[N + kk * (kk + 1) / 2 + e], tot[kk], acc);
            g_mean[g * N + e] = acc * inv_c;
        } else if (e < N + T) {
            const int f = e - N;   // entry (a, c) of the packed factor
            int a = 0;
            while ((a + 1) * (a + 2) / 2 <= f) ++a;
            const int c = f - a * (a + 1) / 2;
            float acc = 0.0f;
            for (int kk = a; kk < N; ++kk)
                acc = fmaf(r[N + kk * (kk + 1) / 2 + a], tot[N + kk * (kk + 1) / 2 + c], acc);
            g_factor[g * T + f] = acc * inv_c15;
        } else if (e < NM) {
            g_colour[g * 3 + e - N - T] = alpha * tot[e];
        } else {
            g_weight[g] = fmaf(c2, tot[N + T + 2], fmaf(c1, tot[N + T + 1], c0 * tot[N + T]));
        }
    }
}

// ---- culled: work items (Gaussian, up to kItemTiles of its tiles) ---------
template <int N> struct BwdLayout {
    static constexpr int T = N * (N + 1) / 2;
    static constexpr int R = (N + T + 7 + 3) / 4 * 4;
    static constexpr int NM = N + T + 3;             // B1 | B2 | H
};

// y and msq for one lane; d[a] = x[a] - m[a].
template <int N>
__device__ __forceinline__ void brows(const float *__restrict__ r, const float (&x)[N],
                                      float (&d)[N], float (&y)[N], float &msq)
{
#pragma unroll
    for (int row = 0; row < N; ++row) {
        d[row] = x[row] - r[row];
        const float *srow = r + N + row * (row + 1) / 2;
        float acc = srow[0] * d[0];
#pragma unroll
        for (int j = 1; j <= row; ++j) acc = fmaf(srow[j], d[j], acc);
        y[row] = acc;
        msq = fmaf(acc, acc, msq);
    }
}

// One work item (wave-uniform `it`).
template <int N>
__device__ __forceinline__ void backward_item(
    int64_t it, int64_t g, int64_t q, int tile, const float *__restrict__ grec,
    const float *__restrict__ qs, const float *__restrict__ gs,
    const int64_t *__restrict__ a_off, const int32_t *__restrict__ a_ent,
    const int32_t *__restrict__ ent_tile, const uint8_t *__restrict__ act,
    const int64_t *__restrict__ gitem_off, float *__restrict__ gpart,
    int32_t *__restrict__ gflag)
{
    using Lay = BwdLayout<N>;
    constexpr int T = Lay::T;
    const int lane = lane_id();
    const int64_t j0 = uniform64(gitem_off[g]);
    const int64_t t0 = uniform64(a_off[g]), t1 = uniform64(a_off[g + 1]);
    const int64_t e0 = t0 + (it - j0) * kItemTiles;
    const int64_t e1 = (e0 + kItemTiles < t1) ? e0 + kItemTiles : t1;
    const float *__restrict__ r = grec + g * Lay::R;
    constexpr int AL = N + T + 3, CO = N + T + 4;
    const float alpha = r[AL], c0 = r[CO], c1 = r[CO + 1], c2 = r[CO + 2];

    float b1[N], b2[T], h0 = 0.0f, h1 = 0.0f, h2 = 0.0f;
#pragma unroll
    for (int a = 0; a < N; ++a) b1[a] = 0.0f;
#pragma unroll
    for (int e = 0; e < T; ++e) b2[e] = 0.0f;

    // The item's entries, lane = entry (at most kItemTiles <= 64): the
    // entry's tile and the flags of its query groups, loaded together once
    // the entry is known; then the kept (entry, group) pairs in ascending
    // entry order, groups ascending within an entry.
    const int ngroups = (tile + kWave - 1) / kWave;
    const int nent = int(e1 - e0);
    int tl = 0;
    uint32_t fl = 0;   // bit g: group g kept
    if (lane < nent) {
        const int64_t ent = a_ent[e0 + lane];
        tl = ent_tile[ent];
        const uint8_t *af = act + ent * ngroups;
        if (ngroups == 4) {
            // one aligned 4-byte load: tiles of 193..256 queries
            const uint32_t v = *reinterpret_cast<const uint32_t *>(af);
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) fl |= uint32_t(((v >> (8 * gq)) & 0xffu) != 0) << gq;
        } else {
            // tiles of at most 1024 queries: at most 16 groups, loaded
            // together
#pragma unroll
            for (int gq = 0; gq < kMaxGroups; ++gq)
                if (gq < ngroups) fl |= uint32_t(af[gq] != 0) << gq;
        }
    }
    bool any = false;
    for (uint64_t m = ballot(fl != 0); m != 0; m = ballot(fl != 0)) {
        const int l = __ffsll(static_cast<unsigned long long>(m)) - 1;
        const uint32_t fb = __builtin_amdgcn_readlane(fl, l);
        const int gq = __builtin_ctz(fb);
        if (lane == l) fl = fb & (fb - 1);
        {
            const int64_t p0 = int64_t(__builtin_amdgcn_readlane(tl, l)) * tile + gq * kWave;
            const int64_t p = p0 + lane;
            const bool valid = (gq * kWave + lane < tile) && (p < q);
            // every lane loads (a lane past the end from the group's first
            // query, which a kept group has) and the invalid ones are zeroed:
            // no branches
            const int64_t pc = valid ? p : p0;
            float x[N], d[N], y[N];
#pragma unroll
            for (int a = 0; a < N; ++a) x[a] = qs[a * q + pc];
            float msq = 0.0f;
            brows<N>(r, x, d, y, msq);
            any = true;
            const float G = valid ? __builtin_amdgcn_exp2f(-msq) : 0.0f;
            const float g0v = valid ? gs[pc] : 0.0f;
            const float g1v = valid ? gs[q + pc] : 0.0f;
            const float g2v = valid ? gs[2 * q + pc] : 0.0f;
            const float sdot = fmaf(g2v, c2, fmaf(g1v, c1, g0v * c0));
            const float w = alpha * G * sdot;
            h0 = fmaf(G, g0v, h0);
            h1 = fmaf(G, g1v, h1);
            h2 = fmaf(G, g2v, h2);
#pragma unroll
            for (int a = 0; a < N; ++a) {
                const float wy = w * y[a];
                b1[a] += wy;
#pragma unroll
                for (int b = 0; b <= a; ++b)
                    b2[a * (a + 1) / 2 + b] = fmaf(wy, y[b], b2[a * (a + 1) / 2 + b]);
            }
        }
    }
    if (!any) {
        if (lane == 0) gflag[it] = 0;
        return;
    }
    // the moments (B1 | B2 | H, padded to a multiple of 4) summed over the
    // wave; lane 16 r + 15 writes the totals of the r-th quarter
    constexpr int VP = (Lay::NM + 3) & ~3, Q = VP / 4;
    float mv[VP];
#pragma unroll
    for (int a = 0; a < N; ++a) mv[a] = b1[a];
#pragma unroll
    for (int e = 0; e < T; ++e) mv[N + e] = b2[e];
    mv[N + T + 0] = h0;
    mv[N + T + 1] = h1;
    mv[N + T + 2] = h2;
#pragma unroll
    for (int e = Lay::NM; e < VP; ++e) mv[e] = 0.0f;
    wave_reduce_scatter<VP>(mv);
    if ((lane & 15) != 15) return;
    float *out = gpart + it * Lay::NM;
    const int r0 = (lane >> 4) * Q;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        if (r0 + i < Lay::NM) out[r0 + i] = mv[i];
    if (lane == kWave - 1) gflag[it] = 1;
}

// The items (their number on the device) taken by the launched waves in
// turn: a wave's items lie a grid apart.
template <int N>
__global__ __launch_bounds__(kBwdThreads) void k_backward_items(
    int64_t k, int64_t q, int tile, const float *__restrict__ grec,
    const float *__restrict__ qs, const float *__restrict__ gs,
    const int64_t *__restrict__ a_off, const int32_t *__restrict__ a_ent,
    const int32_t *__restrict__ ent_tile, const uint8_t *__restrict__ act,
    const int64_t *__restrict__ gitem_off, const int32_t *__restrict__ gitem_g,
    float *__restrict__ gpart, int32_t *__restrict__ gflag)
{
    const int64_t nit = uniform64(gitem_off[k]);
    const int64_t stride = int64_t(gridDim.x) * kWavesPerBlock;
    // a lane looks up each of the next 64, so that those left out cost nothing
    for (int64_t base = int64_t(blockIdx.x) * kWavesPerBlock + uniform(int(threadIdx.x) / kWave);
         base < nit; base += stride * kWave) {
        const int64_t mine = base + lane_id() * stride;
        const int g = mine < nit ? gitem_g[mine] : -1;
        for (uint64_t m = ballot(g >= 0); m != 0; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            backward_item<N>(base + l * stride, __builtin_amdgcn_readlane(g, l), q, tile, grec, qs,
                             gs, a_off, a_ent, ent_tile, act, gitem_off, gpart, gflag);
        }
    }
}

// ---- culled: Gaussians with a handful of queries --------------------------
// Where a Gaussian is small against the queries' spacing (10-D, 2^20 queries:
// 1.4 kept groups a Gaussian, 1.5 queries of each above the skip threshold),
// an item's wave adds moments that are zero in nearly all lanes, and its sum
// over the lanes takes longer than its pairs.  Here a lane is a query for the
// distances only; the few that count leave their factors in LDS, and the lanes
// then take a moment each.
//
// A query counts unless every term it would add is zero, its value having
// underflowed (below 2^-126: some 3.7 times the threshold's distance) or nothing
// coming from upstream, so that the sums are those of the items over every query
// of the kept groups.  (Counting those above tau 2^-24 only, the step of 2^20
// queries took 16 us less of 2,271, that of 2^22 as long, but an upstream
// gradient large enough makes any of the others matter.)
constexpr int kLightGaussians = 8;    // of a wave (4 and 16: 5 % slower at 2^20 and at 2^22 queries)
constexpr int kLightRows = 32;        // queries of a pair that can count
constexpr int kLightQueries = 64;     // queries of a Gaussian
constexpr int kLightEntries = 8;      // kept entries of a Gaussian (4: 1,527 us at 2^22 queries,
                                      // 8: 1,431, 16: 1,436, 32: 1,439)

// Whether the pass leaves every Gaussian to the items: where they have more
// entries on average than one of its own may have, or at most one in four has any
// (a_off: their entries' offsets).  K = 262,144, n = 10: uniform queries, Q =
// 2^20, 223 us without the pass, 277 with it, 242 so; an image's (66 kept groups a
// Gaussian) 6.93, 7.11 and 6.93 ms.
__device__ __forceinline__ bool light_none(int64_t k, const int64_t *__restrict__ a_off)
{
    const int64_t all = uniform64(a_off[k]);
    return all > kLightEntries * k || 4 * all < k;
}

// ncount: the Gaussian's queries, its moments then in row g of mom (if any), or
// -1 where there are more than the above: it goes to items.  Bound by the loads of the pairs' queries, 13 separate rows of 256
// bytes at n = 10: 165 us at 10-D, 2^20 queries (351 at 2^22), with an L2 miss
// for 43% of the lines.  Loading a pair ahead, or the records' lines beforehand,
// changed nothing, and neither did a sixth fewer vector operations.
template <int N>
__global__ __launch_bounds__(kBwdThreads) void k_light_moments(
    int64_t first, int64_t k, int64_t q, int tile, const float *__restrict__ grec,
    const float *__restrict__ qs, const float *__restrict__ gs,
    const int64_t *__restrict__ a_off, const uint32_t *__restrict__ a_key,
    const int32_t *__restrict__ a_ent, const int32_t *__restrict__ ent_tile,
    const uint8_t *__restrict__ act, float *__restrict__ mom, int32_t *__restrict__ ncount)
{
    using Lay = BwdLayout<N>;
    constexpr int T = Lay::T, R = Lay::R, NM = Lay::NM;
    constexpr int AL = N + T + 3, CO = N + T + 4;
    // a row: y (N) | w y (N) | 1 | G g (3); every moment is a product of two
    constexpr int ONE = 2 * N, RS = (2 * N + 4) | 1;
    constexpr int NE = (NM + kWave - 1) / kWave;
    __shared__ float s_row[kWavesPerBlock][kLightRows * RS];
    const int lane = lane_id(), w = uniform(int(threadIdx.x) / kWave);
    // neighbouring Gaussians, which share tiles, share an L2
    const int64_t g0 =
        ((first + xcd_block(blockIdx.x, gridDim.x)) * kWavesPerBlock + w) * kLightGaussians;
    if (g0 >= k) return;
    const int ng = int(k - g0 < kLightGaussians ? k - g0 : kLightGaussians);
    const int64_t off = a_off[g0 + (lane < ng ? lane : ng)];
    const int64_t b = uniform64(off);
    const int rel = int(off - b);   // this wave's entries: below 2^31
    const int ne = __builtin_amdgcn_readlane(rel, ng);
    const int mine = __shfl_down(rel, 1, kWave) - rel;   // lane < ng: its Gaussian's entries
    // lane < ng: its Gaussian's queries so far
    const bool none = light_none(k, a_off);
    int cnt = lane < ng && (none || mine > kLightEntries) ? kLightQueries + 1 : 0;
    // this lane's moments: lane, lane + 64
    int fa[NE], fb[NE];
    float acc[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = lane + i * kWave;
        fa[i] = fb[i] = ONE;
        acc[i] = 0.0f;
        if (e < N) {
            fa[i] = N + e;
        } else if (e < N + T) {
            int a = 0;
            while ((a + 1) * (a + 2) / 2 <= e - N) ++a;
            fa[i] = N + a;
            fb[i] = e - N - a * (a + 1) / 2;
        } else if (e < NM) {
            fa[i] = ONE + 1 + e - N - T;
        }
    }
    const ConstRec rec0 = const_rec(grec) + g0 * R;
    float *row = s_row[w];
    int cur = -1;
    auto flush = [&](int next) {   // the moments of Gaussian cur
        if (cur >= 0) {
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int e = lane + i * kWave;
                if (e < NM) mom[(g0 + cur) * NM + e] = acc[i];
                acc[i] = 0.0f;
            }
        }
        cur = next;
    };
    const int ngroups = (tile + kWave - 1) / kWave;
    for (int base = 0; base < ne; base += kWave) {
        // past the entries of Gaussians that go to items
        const uint64_t ahead =
            ballot(lane < ng && cnt <= kLightQueries && mine > 0 && rel + mine > base);
        if (ahead == 0) break;
        base = max(base, __builtin_amdgcn_readlane(rel, __builtin_ctzll(ahead)));
        int tl = 0, gl = 0;
        uint32_t fl = 0;   // bit g: group g kept
        if (base + lane < ne) {
            const int64_t e = b + base + lane;
            gl = int(a_key[e] - uint32_t(g0));
            const int64_t ent = a_ent[e];
            tl = ent_tile[ent];
            const uint8_t *af = act + ent * ngroups;
            if (ngroups == 4) {
                const uint32_t v = *reinterpret_cast<const uint32_t *>(af);
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) fl |= uint32_t(((v >> (8 * gq)) & 0xffu) != 0) << gq;
            } else {
                for (int gq = 0; gq < ngroups; ++gq) fl |= uint32_t(af[gq] != 0) << gq;
            }
        }
        if (__shfl(cnt, gl, kWave) > kLightQueries) fl = 0;
        for (uint64_t m = ballot(fl != 0); m != 0; m = ballot(fl != 0)) {
            const int l = __builtin_ctzll(m);
            const uint32_t bits = __builtin_amdgcn_readlane(fl, l);
            const int gq = __builtin_ctz(bits);
            if (lane == l) fl = bits & (bits - 1);
            const int gg = __builtin_amdgcn_readlane(gl, l);
            const int64_t t0 = int64_t(__builtin_amdgcn_readlane(tl, l)) * tile;
            const int sidx = gq * kWave + lane;
            const bool valid = (sidx < tile) && (t0 + sidx < q);
            // scalar bases and one offset, no 64-bit sums a lane (past the
            // end the group's first query)
            const uint32_t at = valid ? uint32_t(sidx) : uint32_t(gq * kWave);
            const ConstRec r = rec0 + gg * R;
            float x[N], d[N], y[N];
            const float *col = qs + t0;
#pragma unroll
            for (int a = 0; a < N; ++a, col += q) x[a] = col[at];
            const float *gt = gs + t0;
            const float gv[3] = {gt[at], (gt + q)[at], (gt + 2 * q)[at]};
            float msq = 0.0f;
#pragma unroll
            for (int a = 0; a < N; ++a) {
                d[a] = x[a] - r[a];
                float t = r[N + a * (a + 1) / 2] * d[0];
#pragma unroll
                for (int j = 1; j <= a; ++j) t = fmaf(r[N + a * (a + 1) / 2 + j], d[j], t);
                y[a] = t;
                msq = fmaf(t, t, msq);
            }
            const float G = __builtin_amdgcn_exp2f(-msq);
            const float wgt = r[AL] * G *
                              fmaf(gv[2], r[CO + 2], fmaf(gv[1], r[CO + 1], gv[0] * r[CO]));
            float h[3];
            bool none = wgt == 0.0f && msq < INFINITY;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                h[ch] = G * gv[ch];
                none &= h[ch] == 0.0f;
            }
            const bool counts = valid && !none;
            const uint64_t hit = ballot(counts);
            const int nh = __popcll(hit);
            int c = __builtin_amdgcn_readlane(cnt, gg) + nh;
            if (nh > kLightRows) c = kLightQueries + 1;
            if (lane == gg) cnt = c;
            if (c > kLightQueries) {
                if (gl == gg) fl = 0;
                continue;
            }
            if (nh == 0) continue;
            if (gg != cur) flush(gg);
            if (counts) {
                float *o = row + __popcll(hit & lanemask_lt()) * RS;
#pragma unroll
                for (int a = 0; a < N; ++a) {
                    o[a] = y[a];
                    o[N + a] = wgt * y[a];
                }
                o[ONE] = 1.0f;
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) o[ONE + 1 + ch] = h[ch];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int h = 0; h < nh; ++h) {
#pragma unroll
                for (int i = 0; i < NE; ++i)
                    acc[i] = fmaf(row[h * RS + fa[i]], row[h * RS + fb[i]], acc[i]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    flush(-1);
    if (lane < ng) ncount[g0 + lane] = cnt > kLightQueries ? -1 : cnt;
}

// The gradients of the Gaussians whose moments k_light_moments left: a lane
// applies S^T to its Gaussian's, a wave per 64 Gaussians.  Records and moments
// come, and gradients go, through LDS, consecutive lanes on consecutive words:
// written from the lanes, every store would touch 64 lines.  62 us at K =
// 262,144, n = 10, 3.5 TB/s (the pass of k_backward_finalize, which stores from
// its lanes, took 81).
template <int N>
__global__ __launch_bounds__(kWave, 2) void k_light_gradients(
    int64_t k, const float *__restrict__ grec, const float *__restrict__ mom,
    const int32_t *__restrict__ ncount, const int32_t *__restrict__ gperm,
    float *__restrict__ g_mean, float *__restrict__ g_factor, float *__restrict__ g_weight,
    float *__restrict__ g_colour)
{
    using Lay = BwdLayout<N>;
    constexpr int T = Lay::T, R = Lay::R, NM = Lay::NM;
    constexpr int F = N + T + 7;        // fields used of a record
    constexpr int ST = R + 1;           // odd: no bank conflicts
    static_assert(R % 4 == 0 && N + T + 4 <= R, "a lane's row");
    __shared__ float st[kWave * ST];
    __shared__ int32_t s_gi[kWave];
    const int lane = lane_id();
    const int64_t g0 = int64_t(blockIdx.x) * kWave, g = g0 + lane;
    const int n = g < k ? ncount[g] : -1;
    if (ballot(n >= 0) == 0) return;
    s_gi[lane] = n >= 0 ? gperm[g] : -1;
    const int rows = int(k - g0 < kWave ? k - g0 : kWave);
    {
        const float4 *src = reinterpret_cast<const float4 *>(grec + g0 * R);
#pragma unroll
        for (int i = 0; i < R / 4; ++i) {
            const int e = i * kWave + lane, j = e / (R / 4), u = e - j * (R / 4);
            if (j < rows) {
                const float4 v = src[e];
                float *o = st + j * ST + 4 * u;
                o[0] = v.x;
                o[1] = v.y;
                o[2] = v.z;
                o[3] = v.w;
            }
        }
    }
    __syncthreads();
    float r[F], mo[NM];
#pragma unroll
    for (int e = 0; e < F; ++e) r[e] = st[lane * ST + e];
    __syncthreads();
    {
        constexpr int V = (NM + 3) / 4;
        // (rows nobody wrote are read, below the buffer's end, and not used)
        const float4 *src = reinterpret_cast<const float4 *>(mom + g0 * NM);
        const int words = rows * NM;
        float4 v[V];
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int e = 4 * (i * kWave + lane);
            if (e + 3 < words) {
                v[i] = src[i * kWave + lane];
            } else {
                v[i].x = e < words ? mom[g0 * NM + e] : 0.0f;
                v[i].y = e + 1 < words ? mom[g0 * NM + e + 1] : 0.0f;
                v[i].z = e + 2 < words ? mom[g0 * NM + e + 2] : 0.0f;
                v[i].w = 0.0f;
            }
        }
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const float c[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = 4 * (i * kWave + lane) + u, j = e / NM;
                if (e < words) st[j * ST + e - j * NM] = c[u];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < NM; ++e) mo[e] = n > 0 ? st[lane * ST + e] : 0.0f;
    __syncthreads();
    constexpr int AL = N + T + 3, CO = N + T + 4;
    const float *b1 = mo, *b2 = mo + N;
    // dm | dL | dc | dalpha
    const float inv_c = float(1.0 / kHalfLog2e);
    const float inv_c15 = float(1.0 / (kHalfLog2e * kSqrtHalfLog2e));
    float *o = st + lane * ST;
#pragma unroll
    for (int a = 0; a < N; ++a) {
        float sum = 0.0f;
#pragma unroll
        for (int kk = a; kk < N; ++kk) sum = fmaf(r[N + kk * (kk + 1) / 2 + a], b1[kk], sum);
        o[a] = sum * inv_c;
#pragma unroll
        for (int c = 0; c <= a; ++c) {
            float t = 0.0f;
#pragma unroll
            for (int kk = a; kk < N; ++kk)
                t = fmaf(r[N + kk * (kk + 1) / 2 + a], b2[kk * (kk + 1) / 2 + c], t);
            o[N + a * (a + 1) / 2 + c] = t * inv_c15;
        }
    }
    const float h0 = mo[N + T], h1 = mo[N + T + 1], h2 = mo[N + T + 2];
    o[N + T + 0] = r[AL] * h0;
    o[N + T + 1] = r[AL] * h1;
    o[N + T + 2] = r[AL] * h2;
    o[N + T + 3] = fmaf(r[CO + 2], h2, fmaf(r[CO + 1], h1, r[CO] * h0));
    __syncthreads();
    auto put = [&](float *dst, auto width, int from) {
        constexpr int W = decltype(width)::value;
#pragma unroll 11
        for (int i = 0; i < W; ++i) {
            const int e = i * kWave + lane, j = e / W, c = e - j * W;
            const int64_t gi = s_gi[j];
            if (gi >= 0) dst[gi * W + c] = st[j * ST + from + c];
        }
    };
    put(g_mean, std::integral_constant<int, N>{}, 0);
    put(g_factor, std::integral_constant<int, T>{}, N);
    put(g_colour, std::integral_constant<int, 3>{}, N + T);
    put(g_weight, std::integral_constant<int, 1>{}, N + T + 3);
}

// Per sorted Gaussian: sum its items' moments in item order, then
//   dm = S'^T B1 / c, dL = tril(S'^T B2) / c^1.5, dalpha = c . H, dc = alpha H.
// light: not negative where a Gaussian has its gradients already (null: nowhere).
template <int N>
__global__ __launch_bounds__(kBwdThreads) void k_backward_finalize(
    int64_t k, const int32_t *__restrict__ light, const float *__restrict__ grec,
    const int64_t *__restrict__ gitem_off, const float *__restrict__ gpart,
    const int32_t *__restrict__ gflag,
    const int32_t *__restrict__ gperm, float *__restrict__ g_mean,
    float *__restrict__ g_factor, float *__restrict__ g_weight, float *__restrict__ g_colour)
{
    using Lay = BwdLayout<N>;
    constexpr int T = Lay::T, NM = Lay::NM;
    const int64_t g = int64_t(blockIdx.x) * kBwdThreads + threadIdx.x;
    if (g >= k || (light && light[g] >= 0)) return;
    const int64_t i0 = gitem_off[g], i1 = gitem_off[g + 1];
    float acc[NM];
#pragma unroll
    for (int e = 0; e < NM; ++e) acc[e] = 0.0f;
    for (int64_t i = i0; i < i1; ++i) {
        if (!gflag[i]) continue;
        const float *pp = gpart + i * NM;
#pragma unroll
        for (int e = 0; e < NM; ++e) acc[e] += pp[e];
    }
    const float *r = grec + g * Lay::R;
    const int64_t gi = gperm[g];
    const float inv_c = float(1.0 / kHalfLog2e);
    const float inv_c15 = float(1.0 / (kHalfLog2e * kSqrtHalfLog2e));
#pragma unroll
    for (int a = 0; a < N; ++a) {
        float s = 0.0f;
#pragma unroll
        for (int kk = a; kk < N; ++kk) s = fmaf(r[N + kk * (kk + 1) / 2 + a], acc[kk], s);
        g_mean[gi * N + a] = s * inv_c;
    }
#pragma unroll
    for (int a = 0; a < N; ++a) {
#pragma unroll
        for (int b = 0; b <= a; ++b) {
            float s = 0.0f;
#pragma unroll
            for (int kk = a; kk < N; ++kk)
                s = fmaf(r[N + kk * (kk + 1) / 2 + a], acc[N + kk * (kk + 1) / 2 + b], s);
            g_factor[gi * T + a * (a + 1) / 2 + b] = s * inv_c15;
        }
    }
    const float alpha = r[N + T + 3];
    const float h0 = acc[N + T], h1 = acc[N + T + 1], h2 = acc[N + T + 2];
    g_weight[gi] = fmaf(r[N + T + 6], h2, fmaf(r[N + T + 5], h1, r[N + T + 4] * h0));
    g_colour[gi * 3 + 0] = alpha * h0;
    g_colour[gi * 3 + 1] = alpha * h1;
    g_colour[gi * 3 + 2] = alpha * h2;
}

// The upstream gradient in tile order; also clears the k kept-entry counts.
__global__ __launch_bounds__(256) void k_gather_grad(int64_t q, const int32_t *__restrict__ perm,
                                                     const float *__restrict__ grad_out,
                                                     float *__restrict__ gs, int64_t k,
                                                     int32_t *__restrict__ a_cnt)
{
    const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (p < k) a_cnt[p] = 0;
    if (p >= q) return;
    const int64_t o = perm[p];
    gs[p] = grad_out[o * 3 + 0];
    gs[q + p] = grad_out[o * 3 + 1];
    gs[2 * q + p] = grad_out[o * 3 + 2];
}

template <int N>
hipError_t dense_n(const ngd_mixture *mix, const float *queries, int64_t q,
                   const float *grad_out, float *gm, float *gf, float *gw, float *gc,
                   hipStream_t s)
{
    // 16 waves per Gaussian (8 from n = 11, whose moments take more than the
    // 128 registers a lane of a 16-wave workgroup has) while that is what it
    // takes to fill the chip, then 4, and one where the Gaussians fill it by
    // themselves and a wave's sum over its lanes costs as much as its few
    // queries.  n = 10, 16 / 4 / 1 waves: K = 256, Q = 65,536 65 / 120 / 454 us;
    // K = 1,000, Q = 4,096 30 / 22 / 37; K = 4,096, Q = 8,192 - / 116 / 117 and
    // Q = 300 - / 23 / 17; K = 131,072, Q = 64 - / 418 / 186.
    auto go = [&](auto kern, int waves, int per = 1) {
        const int threads = waves * per * kWave;
        const int64_t blocks = (mix->k + per - 1) / per, most = max_grid(threads);
        for (int64_t b = 0; b < blocks; b += most)
            kern<<<unsigned(std::min(blocks - b, most)), threads, 0, s>>>(
                b, mix->k, q, mix->rec.as<float>(), queries, grad_out, gm, gf, gw, gc);
        return hipGetLastError();
    };
    if (q == 0) {   // no queries: zero gradients whatever the parameters
        hipError_t e = launch_zero_f32(gm, mix->k * N, s);
        if (e == hipSuccess) e = launch_zero_f32(gf, mix->k * (N * (N + 1) / 2), s);
        if (e == hipSuccess) e = launch_zero_f32(gw, mix->k, s);
        return e == hipSuccess ? launch_zero_f32(gc, mix->k * 3, s) : e;
    }
    if (mix->k < 512) {
        constexpr int W = N <= 10 ? 16 : 8;
        return go(k_backward_dense<N, W, 1>, W);
    }
    if (mix->k < 2048 || (mix->k < 32768 && q >= 4096)) return go(k_backward_dense<N, 4, 1>, 4);
    return go(k_backward_dense<N, 1, 4>, 1, 4);
}

template <int N>
hipError_t culled_n(const ngd_mixture *mix, ngd_cull *c, const float *grad_out, float *gm,
                    float *gf, float *gw, float *gc, hipStream_t s)
{
    k_gather_grad<<<unsigned((std::max(c->q, c->k) + 255) / 256), 256, 0, s>>>(
        c->q, c->perm.as<int32_t>(), grad_out, c->gs.as<float>(), c->k, c->a_cnt.as<int32_t>());
    hipError_t err = launch_backward_prepare(c, s);
    if (err != hipSuccess) return err;
    const int32_t *a_ent = c->a_ent_buf ? c->vals1.as<int32_t>() : c->vals0.as<int32_t>();
    // the Gaussians with a handful of queries first, by lanes
    const int32_t *light = nullptr;
    if (backward_light(c)) {
        // (their queries in gitem_cnt, which the items' offsets no longer need)
        int32_t *ncount = c->gitem_cnt.as<int32_t>();
        const int64_t per = int64_t(kWavesPerBlock) * kLightGaussians;
        const int64_t blocks = (mix->k + per - 1) / per, most = max_grid(kBwdThreads);
        for (int64_t b = 0; b < blocks; b += most)
            k_light_moments<N><<<unsigned(std::min(blocks - b, most)), kBwdThreads, 0, s>>>(
                b, mix->k, c->q, c->params.tile, c->grec.as<float>(), c->qs.as<float>(),
                c->gs.as<float>(), c->a_off.as<int64_t>(),
                c->a_ent_buf ? c->keys1.as<uint32_t>() : c->keys0.as<uint32_t>(), a_ent,
                c->ent_tile.as<int32_t>(), c->act.as<uint8_t>(), c->gpart.as<float>(), ncount);
        k_light_gradients<N><<<unsigned((mix->k + kWave - 1) / kWave), kWave, 0, s>>>(
            mix->k, c->grec.as<float>(), c->gpart.as<float>(), ncount, c->gperm.as<int32_t>(), gm,
            gf, gw, gc);
        light = ncount;
    }
    if ((err = launch_backward_items(c, light, s)) != hipSuccess) return err;
    if (c->gitems_cap > 0) {
        // about four rounds of resident waves (4 per SIMD at this kernel's
        // register count), each taking items a grid apart: 1,024 / 2,048 /
        // 4,096 blocks measured 327-343 / 319-326 / 293-305 us at 10-D,
        // 2^20 queries (8,192 and 16,384 alike), against 346-353 us with
        // one wave per item
        const unsigned blocks = unsigned(std::min<int64_t>(
            (c->gitems_cap + kWavesPerBlock - 1) / kWavesPerBlock, kBwdItemBlocks));
        k_backward_items<N><<<blocks, kBwdThreads, 0, s>>>(
            mix->k, c->q, c->params.tile, c->grec.as<float>(), c->qs.as<float>(),
            c->gs.as<float>(), c->a_off.as<int64_t>(), a_ent,
            c->ent_tile.as<int32_t>(), c->act.as<uint8_t>(), c->gitem_off.as<int64_t>(),
            c->gitem_g.as<int32_t>(), c->gpart.as<float>(), c->gflag.as<int32_t>());
    }
    const unsigned fb = unsigned((mix->k + kBwdThreads - 1) / kBwdThreads);
    k_backward_finalize<N><<<fb, kBwdThreads, 0, s>>>(
        mix->k, light, c->grec.as<float>(), c->gitem_off.as<int64_t>(), c->gpart.as<float>(),
        c->gflag.as<int32_t>(), c->gperm.as<int32_t>(), gm, gf, gw, gc);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_backward_dense(const ngd_mixture *mix, const float *queries, int64_t q,
                                 const float *grad_out, float *g_mean, float *g_factor,
                                 float *g_weight, float *g_colour, hipStream_t s)
{
    if (mix->k == 0) return hipSuccess;
    switch (mix->n) {
#define NGD_CASE(NN) \
    case NN: return dense_n<NN>(mix, queries, q, grad_out, g_mean, g_factor, g_weight, g_colour, s);
        NGD_CASE(1) NGD_CASE(2) NGD_CASE(3) NGD_CASE(4) NGD_CASE(5) NGD_CASE(6)
        NGD_CASE(7) NGD_CASE(8) NGD_CASE(9) NGD_CASE(10) NGD_CASE(11) NGD_CASE(12)
#undef NGD_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_backward_culled(const ngd_mixture *mix, ngd_cull *c, const float *grad_out,
                                  float *g_mean, float *g_factor, float *g_weight,
                                  float *g_colour, hipStream_t s)
{
    if (mix->k == 0) return hipSuccess;
    switch (mix->n) {
#define NGD_CASE(NN) \
    case NN: return culled_n<NN>(mix, c, grad_out, g_mean, g_factor, g_weight, g_colour, s);
        NGD_CASE(1) NGD_CASE(2) NGD_CASE(3) NGD_CASE(4) NGD_CASE(5) NGD_CASE(6)
        NGD_CASE(7) NGD_CASE(8) NGD_CASE(9) NGD_CASE(10) NGD_CASE(11) NGD_CASE(12)
#undef NGD_CASE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ngd
