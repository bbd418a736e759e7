// Culled forward: the pairs of every (tile, candidate) filtered by a
// matrix-core contraction, the survivors evaluated in float32.
//
// The quadratic form (Sec. 3.1, Eq. 1-2, in exp2 units, S' = sqrt(log2(e)/2)
// L^-1, P = S'^T S'):
//   M(x) = |S'(x - m)|^2
//        = sum_{i<=j} C_ij x'_i x'_j + sum_i b_i x'_i + a,
//   x' = x - c, m' = m - c, C_ii = P_ii, C_ij = 2 P_ij (i < j),
//   b = -2 P m',  a = m'^T P m',
// with c the centre of the tile's query box, so that the features stay small
// and the expanded form does not cancel away its own accuracy.  Features and
// coefficients are float16, one product each (v_mfma_f32_32x32x16_f16,
// float32 accumulation); a is held as a sum of two float16 values, and so is
// each b_i where the k-steps have room for it.
//
// The bound.  Per Gaussian, P is formed in float64 and rounded to float16
// (P~, relative 2^-11), and b and a follow from P~ in float32, so the
// contraction is that of (x - m)^T P~ (x - m) up to the rounding of the
// features (2^-11 each) and of b (2^-11 when it has one value).  With
// R = max row sum of |P| (at least the spectral norm of |P|), q = max |x'|
// and h = max |x'|_inf over a 64-query group, the result is off by at most
//   g (R ((|m'| + q)^2 + q^2) + k_b |b|_1 h),  g = 2^-11 * 1.25,
// k_b = 2 (1 where b has two values); the quarter covers the float32
// accumulation (96 terms: 2^-16.4), b's and a's own float32 rounding
// (2^-19), and x' and m' (2^-23).  A candidate is skipped for a whole group
// only when the group's smallest value minus that bound exceeds
// log2(1/tau) + 20, i.e. only pairs with G < tau 2^-20; every other pair is
// evaluated in float32 (lane = query) with the same threshold, so the colours
// are the float32 ones whatever the filter's rounding.
//
// Scales, powers of two all: s per Gaussian puts max |C| s in [2^7, 2^8);
// sigma per tile puts max |x'| sigma in (8, 16] (up to |x'| = 2^60: a tile that
// reaches further has no finite features, and an infinite bound), so the features
// (sigma x'_i)(sigma x'_j) stay within 2^8; the linear features carry 2^11
// and the constant one 2^15.  A column's accumulator is then K M with
// K = sigma^2 s.  `a` saturates (a smaller constant only keeps more); a
// Gaussian or tile outside the ranges (non-finite, b or K too large) gets an
// infinite bound and is never skipped.
//
// One product instead of the three of a hi / lo split costs 2.4% of the pairs
// passing instead of 1.5% (10-D, 2^20 queries), for a third of the matrix
// work and half the coefficients.
//
// The filter decides only what is evaluated.  Over 48 workloads drawn from n = 3
// to 10, K = 256 to 262,144, Q = 2,048 to 2^20 and tau = 1e-6 to 3 sigma it leaves
// the kept pairs of the forwards before it (per-coordinate boxes in float16,
// rounded outwards, ahead of the float32 distances; the bf16 hi / lo filter) and
// the float32 colours bit for bit.
//
// k_filter_items: one workgroup per item (a tile's queries, up to kItemCands of
// its candidates; four times as many spread the work too thin: 0.30 -> 0.32 and
// the image's 0.85 -> 1.14 ms), 4 waves of 64 queries.  256 candidates at a time:
// each wave brings 64 records into LDS (16-byte global-to-LDS loads), lane = candidate
// forms b, a and the bound terms beside them, then every wave contracts all
// 256 against its queries, 32 at a time, and writes the survivors as one bit
// per (candidate, group).  Nothing else per (tile, candidate) passes through
// memory.
// k_eval_items: the survivors in float32, a wave per (item, group), its queries
// in registers, records through scalar loads.  A kernel of its own because it
// needs the most waves in flight where the filter's LDS and registers leave
// three per SIMD: with the evaluation as the filter's last phase the 10-D image
// (K = 262,144, 800 x 800) took 6.15 ms, in two kernels 0.87 + 3.27.
//
// Measured against the forwards before it (a box test per group, or a bf16
// hi / lo filter over precomputed per-entry terms): 10-D, K = 262,144,
// Q = 2^20, 1.59 (float32) and 1.12 ms (bf16) -> 0.29 filter + 0.20 evaluation;
// the image, 22% of whose pairs are kept, 7.72 -> 4.14 ms.  The filter is
// bound by the gathers of its records (160 B a candidate and tile at 10-D),
// the evaluation of the image by its vector operations (80 of about 114 issue
// slots a pair).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "eval_common.hpp"
#include "ngd_internal.hpp"
#include "wave.hpp"

namespace ngd {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMThreads = 256;
constexpr int kWaves = kMThreads / kWave;
constexpr float kGamma = 1.25f / 2048.0f;
constexpr float kLinFeat = 2048.0f;      // 2^11
constexpr float kConstFeat = 32768.0f;   // 2^15
constexpr float kF16Max = 65504.0f;
constexpr int kItemChunks = kItemCands / kWave;   // 64-bit masks of an item and group
static_assert(kItemCands % kMThreads == 0, "whole rounds of columns");

// Slots of the contraction: T quadratic ones padded to units of 8, then the
// constant (two), the linear ones, and (LO) their low parts.  A record is QU
// units of 16 bytes of quadratic coefficients, then m (N), R s and s as
// floats; in LDS the linear units take the place of the latter.
template <int N> struct Filt {
    static constexpr int T = N * (N + 1) / 2;
    static constexpr int QU = (T + 7) / 8;
    static constexpr int KS = (8 * QU + 2 + N + 15) / 16;   // k-steps
    static constexpr int U = 2 * KS;                        // units of a column
    static constexpr int L0 = 8 * QU;                       // first constant slot
    static constexpr bool LO = L0 + 2 + 2 * N <= 16 * KS;
    static constexpr int MU = (N + 2 + 3) / 4;
    static constexpr int RU = QU + MU;                      // units of a record
    static constexpr int META = U > RU ? U : RU;            // the bound terms' unit
    static constexpr int ST = (META + 1) | 1;               // odd: no bank conflicts
};

// Quadratic slot q -> (i, j), i <= j, the upper triangle by rows; -1 past T.
template <int N> struct QuadTable {
    int i[Filt<N>::QU * 8];
    int j[Filt<N>::QU * 8];
    constexpr QuadTable() : i(), j()
    {
        int q = 0;
        for (int a = 0; a < N; ++a)
            for (int b = a; b < N; ++b) {
                i[q] = a;
                j[q] = b;
                ++q;
            }
        for (; q < Filt<N>::QU * 8; ++q) {
            i[q] = -1;
            j[q] = -1;
        }
    }
};
template <int N> inline constexpr QuadTable<N> kQuad{};

// Per ordered Gaussian: its record in the order, and that of the contraction, P
// formed in float64 from the record's S'.  A wave per 64 Gaussians: the records
// come and go as float4s, consecutive lanes on consecutive ones, through LDS.
// (Without the copy, the kernels reading the mixture's own records by the order,
// a step took as long: they lose what it costs.)
template <int N>
__global__ __launch_bounds__(kWave) void k_gauss_records(int64_t k, const float *__restrict__ rec,
                                                         const int32_t *__restrict__ gperm,
                                                         float *__restrict__ grec,
                                                         f16x8 *__restrict__ mrec)
{
    using Fi = Filt<N>;
    constexpr int R = RecLayout<N>::R, R4 = R / 4, kSt = R4 | 1;
    __shared__ f32x4 s_rec[kWave * kSt];
    const int lane = lane_id();
    const int64_t g0 = int64_t(blockIdx.x) * kWave, g = g0 + lane;
    const int cnt = int(k - g0 < kWave ? k - g0 : kWave);
    const int gp = lane < cnt ? gperm[g] : 0;
#pragma unroll
    for (int e = 0; e < R4; ++e) {
        const int sl = e * kWave + lane, j = sl / R4, f = sl - j * R4;
        const int src = __shfl(gp, j, kWave);
        if (j < cnt) {
            const f32x4 v = reinterpret_cast<const f32x4 *>(rec)[int64_t(src) * R4 + f];
            s_rec[j * kSt + f] = v;
            reinterpret_cast<f32x4 *>(grec)[g0 * R4 + sl] = v;
        }
    }
    __syncthreads();
    if (lane >= cnt) return;
    float r[R4 * 4];
#pragma unroll
    for (int e = 0; e < R4; ++e) {
        const f32x4 v = s_rec[lane * kSt + e];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[4 * e + i] = v[i];
    }
    double S[Fi::T];
#pragma unroll
    for (int e = 0; e < Fi::T; ++e) S[e] = double(r[N + e]);
    auto sidx = [](int row, int col) { return row * (row + 1) / 2 + col; };
    float cf[Fi::QU * 8];
    double rs[N];
    float cmax = 0.0f;
    bool ok = true;
#pragma unroll
    for (int a = 0; a < N; ++a) rs[a] = 0.0;
#pragma unroll
    for (int q = 0; q < Fi::QU * 8; ++q) {
        cf[q] = 0.0f;
        if (kQuad<N>.i[q] >= 0) {
            const int a = kQuad<N>.i[q], b = kQuad<N>.j[q];   // a <= b
            double p = 0.0;
#pragma unroll
            for (int row = 0; row < N; ++row)
                if (row >= b) p += S[sidx(row, a)] * S[sidx(row, b)];
            cf[q] = float(a == b ? p : 2.0 * p);
            rs[a] += fabs(p);
            if (a != b) rs[b] += fabs(p);
            cmax = fmaxf(cmax, fabsf(cf[q]));
            ok = ok && fabsf(cf[q]) < INFINITY;
        }
    }
    double best = 0.0;
#pragma unroll
    for (int a = 0; a < N; ++a) best = fmax(best, rs[a]);
    // s: the power of two that puts cmax s into [2^7, 2^8)
    const int e = int(__float_as_uint(cmax) >> 23) - 127;
    ok = ok && e > -90 && e < 90;
    const float s = ok ? __uint_as_float(uint32_t(7 - e + 127) << 23) : 1.0f;
    f16x8 *o = mrec + g * Fi::RU;
#pragma unroll
    for (int u = 0; u < Fi::QU; ++u) {
        f16x8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = ok ? _Float16(cf[8 * u + i] * s) : _Float16(0.0f);
        o[u] = v;
    }
    float mt[Fi::MU * 4];
#pragma unroll
    for (int i = 0; i < Fi::MU * 4; ++i) mt[i] = 0.0f;
#pragma unroll
    for (int a = 0; a < N; ++a) mt[a] = r[a];
    mt[N] = ok ? float(best * s * (1.0 + 1.0 / 1048576.0)) : INFINITY;   // rounded up
    mt[N + 1] = s;
#pragma unroll
    for (int u = 0; u < Fi::MU; ++u)
        o[Fi::QU + u] = __builtin_bit_cast(
            f16x8, f32x4{mt[4 * u], mt[4 * u + 1], mt[4 * u + 2], mt[4 * u + 3]});
}

// Feature of slot `slot` for sigma-scaled coordinates u.
template <int N, int SLOT> __device__ __forceinline__ float feature(const float (&u)[N], float one)
{
    using Fi = Filt<N>;
    if constexpr (SLOT < Fi::L0) {
        if constexpr (kQuad<N>.i[SLOT] >= 0)
            return u[kQuad<N>.i[SLOT]] * u[kQuad<N>.j[SLOT]];
        else
            return 0.0f;
    } else if constexpr (SLOT < Fi::L0 + 2) {
        return one;
    } else if constexpr (SLOT < Fi::L0 + 2 + N) {
        return u[SLOT - Fi::L0 - 2] * kLinFeat;
    } else if constexpr (Fi::LO && SLOT < Fi::L0 + 2 + 2 * N) {
        return u[SLOT - Fi::L0 - 2 - N] * kLinFeat;
    } else {
        return 0.0f;
    }
}

// masks: per (item, group) kItemChunks words, bit = candidate not skipped.
template <int N>
__global__ __launch_bounds__(kMThreads, 3) void k_filter_items(
    int64_t item0, int64_t q, int tile, const f16x8 *__restrict__ mrec, const float *__restrict__ tcen,
    const float *__restrict__ qs, const int64_t *__restrict__ tile_off,
    const int32_t *__restrict__ cand, const int32_t *__restrict__ item_tile,
    const int64_t *__restrict__ item_off, float skip, uint64_t *__restrict__ masks)
{
    using Fi = Filt<N>;
    constexpr int KS = Fi::KS, ST = Fi::ST;
    __shared__ f16x8 s_col[kMThreads * ST];
    __shared__ float s_hm[kWaves];

    const int64_t it = item0 + xcd_block(blockIdx.x, gridDim.x);   // neighbouring tiles share an L2
    const int64_t t = uniform(item_tile[it]);
    const int64_t c1 = uniform64(tile_off[t + 1]);
    const int64_t e0 = uniform64(tile_off[t]) + (it - uniform64(item_off[t])) * kItemCands;
    const int ne = uniform(int(c1 - e0 < kItemCands ? c1 - e0 : kItemCands));

    const int lane = lane_id(), w = uniform(int(threadIdx.x) / kWave), h = lane / 32;
    const int s = int(blockIdx.y) * kMThreads + int(threadIdx.x);
    const bool live = ballot(s < tile && t * tile + s < q) != 0;   // the wave has queries
    const int ngroups = (tile + kWave - 1) / kWave;
    uint64_t *__restrict__ mine_m = masks + (it * ngroups + s / kWave) * kItemChunks;

    float cen[N];
#pragma unroll
    for (int a = 0; a < N; ++a) cen[a] = tcen[t * N + a];
    // the wave's 64 rows, two blocks of 32; rows past the end repeat the
    // group's first query (a wave without queries: the tile's first)
    f16x8 fa[2][KS];
    float hq, hm;
    float sig;
    bool far;
    {
        float xr[2][N];
        float m1 = 0.0f, m2 = 0.0f;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
            const int sg = int(blockIdx.y) * kMThreads + w * kWave;
            const int sr = sg + rb * 32 + (lane % 32);
            const int64_t pr = t * tile + sr;
            const int64_t pc = (sr < tile && pr < q) ? pr : t * tile + (live ? sg : 0);
            float n2 = 0.0f;
#pragma unroll
            for (int a = 0; a < N; ++a) {
                xr[rb][a] = qs[a * q + pc] - cen[a];
                m1 = fmaxf(m1, fabsf(xr[rb][a]));
                n2 = fmaf(xr[rb][a], xr[rb][a], n2);
            }
            m2 = fmaxf(m2, n2);
        }
        hm = wave_max_nonneg(m1);
        hq = sqrtf(wave_max_nonneg(m2)) * (1.0f + 1.0f / 1048576.0f);
        if (lane == 0) s_hm[w] = hm;
        __syncthreads();
        float ht = s_hm[0];
#pragma unroll
        for (int i = 1; i < kWaves; ++i) ht = fmaxf(ht, s_hm[i]);
        // a tile much smaller than its distance from the origin: the scale
        // of that distance, so that b stays in range
#pragma unroll
        for (int a = 0; a < N; ++a) ht = fmaxf(ht, fabsf(cen[a]) * (1.0f / 1024.0f));
        // ht sigma in (8, 16]; beyond 2^60 the features would not be finite
        // and nothing is skipped
        const int e = int(__float_as_uint(ht) >> 23) - 127;
        far = e >= 60;
        sig = (e > -60 && !far) ? __uint_as_float(uint32_t(3 - e + 127) << 23) : 1.0f;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
            for (int a = 0; a < N; ++a) xr[rb][a] *= sig;
            // every lane forms all the features (indices known at compile time)
            // and keeps those of its half
            [&]<int... I>(std::integer_sequence<int, I...>) {
                float f[16 * KS] = {feature<N, I>(xr[rb], kConstFeat)...};
#pragma unroll
                for (int e = 0; e < 8 * KS; ++e) {
                    const float lo = f[e / 8 * 16 + e % 8], hi = f[e / 8 * 16 + 8 + e % 8];
                    fa[rb][e / 8][e % 8] = _Float16(h ? hi : lo);
                }
            }(std::make_integer_sequence<int, 16 * KS>{});
        }
    }

    for (int base = 0; base < ne; base += kMThreads) {
        if (base != 0) __syncthreads();   // the last chunk's readers are done
        // ---- columns: this wave's 64 candidates
        const int ew = base + w * kWave;
        const int nw = ne - ew < kWave ? ne - ew : kWave;   // may be <= 0
        if (nw > 0) {
            const int ci = lane < nw ? cand[e0 + ew + lane] : 0;
            f16x8 *col = s_col + w * kWave * ST;
#pragma unroll
            for (int i = 0; i < ST; ++i) {
                const int sl = i * kWave + lane;
                const int j = sl / ST, u = sl - j * ST;
                const int cj = __shfl(ci, j, kWave);
                if (u < Fi::RU && j < nw)
                    __builtin_amdgcn_global_load_lds(
                        (const __attribute__((address_space(1))) void *)(mrec +
                                                                         int64_t(cj) * Fi::RU + u),
                        (__attribute__((address_space(3))) void *)(col + i * kWave), 16, 0, 0);
            }
            __builtin_amdgcn_s_waitcnt(0);   // the wave reads only its own loads
            asm volatile("" ::: "memory");
            f16x8 *mine = col + lane * ST;
            float mt[Fi::MU * 4];
#pragma unroll
            for (int u = 0; u < Fi::MU; ++u) {
                const f32x4 v = __builtin_bit_cast(f32x4, mine[Fi::QU + u]);
#pragma unroll
                for (int i = 0; i < 4; ++i) mt[4 * u + i] = v[i];
            }
            const float Rs = mt[N], sc = mt[N + 1];
            float mp[N], tb[N];
            float mm = 0.0f;
#pragma unroll
            for (int a = 0; a < N; ++a) {
                mp[a] = mt[a] - cen[a];
                mm = fmaf(mp[a], mp[a], mm);
                tb[a] = 0.0f;
            }
            // tb = 2 s P~ m'
            [&]<int... QI>(std::integer_sequence<int, QI...>) {
                f16x8 v;
                ((
                     [&] {
                         if constexpr (QI % 8 == 0) v = mine[QI / 8];
                         if constexpr (kQuad<N>.i[QI] >= 0) {
                             constexpr int a = kQuad<N>.i[QI], b = kQuad<N>.j[QI];
                             const float cv = float(v[QI % 8]);
                             if constexpr (a == b) {
                                 tb[a] = fmaf(cv, mp[a] + mp[a], tb[a]);
                             } else {
                                 tb[a] = fmaf(cv, mp[b], tb[a]);
                                 tb[b] = fmaf(cv, mp[a], tb[b]);
                             }
                         }
                     }()),
                 ...);
            }(std::make_integer_sequence<int, 8 * Fi::QU>{});
            float as = 0.0f, b1 = 0.0f, bmax = 0.0f;
            float lin[8 * (Fi::U - Fi::QU)];
#pragma unroll
            for (int i = 0; i < 8 * (Fi::U - Fi::QU); ++i) lin[i] = 0.0f;
            const float bscale = -sig / kLinFeat;
#pragma unroll
            for (int a = 0; a < N; ++a) {
                as = fmaf(tb[a], mp[a], as);
                b1 += fabsf(tb[a]);
                const float v = tb[a] * bscale;
                bmax = fmaxf(bmax, fabsf(v));
                lin[2 + a] = v;
                if constexpr (Fi::LO) lin[2 + N + a] = v - float(_Float16(v));
            }
            const float sig2 = sig * sig;
            const float ac = fmaxf(0.5f * as * sig2 * (1.0f / kConstFeat), 0.0f);
            lin[0] = fminf(ac, kF16Max);
            lin[1] = fminf(ac - float(_Float16(lin[0])), kF16Max);
#pragma unroll
            for (int u = 0; u < Fi::U - Fi::QU; ++u) {
                f16x8 v;
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = _Float16(lin[8 * u + i]);
                mine[Fi::QU + u] = v;
            }
            // skip iff the minimum exceeds T0 + T1 q + T2 q^2 + T3 h; the 1
            // covers float16's least steps (values below 2^-14)
            const float K = sig2 * sc, rk = kGamma * Rs * sig2;
            float t0 = fmaf(rk, mm, fmaf(skip, K, 1.0f));
            if (far || !(bmax < 65000.0f) || !(K > 0x1p-60f && K < 0x1p60f)) t0 = INFINITY;
            mine[Fi::META] = __builtin_bit_cast(
                f16x8, f32x4{t0, 2.0f * rk * sqrtf(mm), 2.0f * rk,
                             (Fi::LO ? 1.0f : 2.0f) * kGamma * b1 * sig2});
        }
        __syncthreads();
        // ---- the contraction: 32 columns at a time against the wave's rows
        const int nb = ne - base < kMThreads ? ne - base : kMThreads;
        if (live) {
            uint32_t lowm = 0;
            for (int cb = 0; cb < nb; cb += 32) {
                const int jl = cb + (lane % 32);
                const f16x8 *colp = s_col + jl * ST;
                f32x16 acc0 = {}, acc1 = {};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const f16x8 b = colp[2 * ks + h];
                    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[0][ks], b, acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[1][ks], b, acc1, 0, 0, 0);
                }
                const f32x4 bd = __builtin_bit_cast(f32x4, colp[Fi::META]);
                const float thr =
                    fmaf(bd[3], hm, fmaf(fmaf(bd[2], hq, bd[1]), hq, bd[0]));
                // the smallest value over the group's rows as a signed-integer
                // minimum of the float bits: exact among non-negative values,
                // and any negative one (rounding below 0) stays negative,
                // which keeps the candidate, as it must
                int mi = 0x7f800000;   // +inf
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    mi = min(mi, min(__float_as_int(acc0[r]), __float_as_int(acc1[r])));
                const bool pass = jl < nb && !(__int_as_float(mi) > thr);
                const uint64_t bal = ballot(pass);
                const uint32_t both = uint32_t(bal) | uint32_t(bal >> 32);
                if (cb & 32) {
                    if (lane == 0) mine_m[(base + cb) / kWave] = uint64_t(both) << 32 | lowm;
                } else {
                    lowm = both;
                    if (cb + 32 >= nb && lane == 0) mine_m[(base + cb) / kWave] = lowm;
                }
            }
        }
    }
}

// A record's fields in order -- m, S' by rows, alpha c -- as NP parts of PS
// floats, each one run of scalar loads; two parts (64 to 80 scalar registers)
// are held at a time, the one in use and the one in flight.
template <int N> struct Parts {
    static constexpr int F = N + N * (N + 1) / 2 + 3;
    static constexpr int NP = F <= 40 ? 1 : (F <= 72 ? 2 : 3);
    static constexpr int PS = ((F + NP - 1) / NP + 3) / 4 * 4;
    static_assert(NP * PS <= RecLayout<N>::R && F - 3 >= (NP - 1) * PS, "parts");
};

template <int N, int P>
__device__ __forceinline__ void load_part(float (&blk)[Parts<N>::PS], ConstRec r)
{
#pragma unroll
    for (int e = 0; e < Parts<N>::PS; ++e) blk[e] = r[P * Parts<N>::PS + e];
}

// Waits for the part in flight, then sends for the next one; the scheduler
// keeps the arithmetic of the one that has arrived behind the loads.
template <int N, int P>
__device__ __forceinline__ void next_part(float (&blk)[Parts<N>::PS], ConstRec &r)
{
    __builtin_amdgcn_sched_barrier(0);
    wait_scalar_then(r);
    load_part<N, P>(blk, r);
    __builtin_amdgcn_sched_barrier(0);
}

// One lane's evaluation of a pair, field by field; the sums are those of rows
// y_r = sum_j S'_rj d_j, msq = sum_r y_r^2 in ascending order.
template <int N> struct PairState {
    float d[N], acc, msq;
    bool c1, c2;   // COUNT: the wave passed the checks after 3 and 6 rows
};

template <int N, int E, bool COUNT>
__device__ __forceinline__ void pair_field(PairState<N> &st, const float (&x)[N], float v,
                                           uint64_t vmask, float skip)
{
    constexpr int T = N * (N + 1) / 2;
    if constexpr (E < N) {
        st.d[E] = x[E] - v;
    } else if constexpr (E < N + T) {
        constexpr int f = E - N;
        constexpr int row = [] {
            int r = 0;
            while ((r + 1) * (r + 2) / 2 <= f) ++r;
            return r;
        }();
        constexpr int col = f - row * (row + 1) / 2;
        st.acc = col == 0 ? v * st.d[0] : fmaf(v, st.d[col], st.acc);
        if constexpr (col == row) st.msq = row == 0 ? st.acc * st.acc : fmaf(st.acc, st.acc, st.msq);
        if constexpr (COUNT && col == row) {
            if constexpr (row + 1 == 3 && N > 3) st.c1 = (ballot(st.msq <= skip) & vmask) != 0;
            if constexpr (row + 1 == 6 && N > 6) st.c2 = (ballot(st.msq <= skip) & vmask) != 0;
        }
    }
}

template <int N, int P, bool COUNT>
__device__ __forceinline__ void pair_part(PairState<N> &st, const float (&x)[N],
                                          const float (&blk)[Parts<N>::PS], uint64_t vmask,
                                          float skip)
{
    [&]<int... I>(std::integer_sequence<int, I...>) {
        (pair_field<N, P * Parts<N>::PS + I, COUNT>(st, x, blk[I], vmask, skip), ...);
    }(std::make_integer_sequence<int, Parts<N>::PS>{});
}

// masks: the filter's; null: every candidate is evaluated.
// OUT: the colours are accumulated; otherwise only the (entry, group) flags.
// COUNT (with OUT = false): the first five of a slot of stats += (pairs examined,
// not skipped by the filter, below the threshold after 3 rows, after 6 rows, kept).
template <int N, bool OUT, bool COUNT>
__global__ __launch_bounds__(kMThreads, 7) void k_eval_items(
    int64_t item0, int64_t q, int tile, const uint64_t *__restrict__ masks, const float *__restrict__ qs,
    const float *__restrict__ grec, const int64_t *__restrict__ tile_off,
    const int32_t *__restrict__ cand, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ item_tile, const int64_t *__restrict__ item_off, float skip,
    uint8_t *__restrict__ act, float *__restrict__ out, float *__restrict__ part,
    unsigned long long *__restrict__ stats)
{
    using Pa = Parts<N>;
    constexpr int R = RecLayout<N>::R, AC = N + N * (N + 1) / 2;
    __shared__ int32_t s_idx[kWaves][kItemCands];    // the survivors' Gaussians
    __shared__ uint16_t s_pos[kWaves][kItemCands];   // their places in the item
    __shared__ uint32_t s_kept[kWaves][kItemCands / 32];
    const int64_t it = item0 + xcd_block(blockIdx.x, gridDim.x);
    const int64_t t = uniform(item_tile[it]);
    const int64_t i0 = uniform64(item_off[t]);
    const int64_t nit = uniform64(item_off[t + 1]) - i0;
    const int64_t c1 = uniform64(tile_off[t + 1]);
    const int64_t e0 = uniform64(tile_off[t]) + (it - i0) * kItemCands;
    const int ne = uniform(int(c1 - e0 < kItemCands ? c1 - e0 : kItemCands));
    const int lane = lane_id(), w = uniform(int(threadIdx.x) / kWave);
    const int s = int(blockIdx.y) * kMThreads + int(threadIdx.x);
    const int64_t p = t * tile + s;
    const bool valid = (s < tile) && (p < q);
    const uint64_t vmask = ballot(valid);
    const int ngroups = (tile + kWave - 1) / kWave;
    const int grp = uniform(s / kWave);
    if (vmask == 0) {   // a group past the end keeps nothing; its pairs count as examined
        if (grp < ngroups) {
            for (int o = lane; o < ne; o += kWave) act[(e0 + o) * ngroups + grp] = 0;
            if constexpr (COUNT) {
                if (lane == 0) atomicAdd(&stats[it % kStatSlots * 8], (unsigned long long)(ne));
            }
        }
        return;
    }
    float x[N];
    {
        const int64_t pc = valid ? p : t * tile;
#pragma unroll
        for (int a = 0; a < N; ++a) x[a] = qs[a * q + pc];
    }
    // the survivors listed first (this wave's part of LDS only), so that the
    // evaluation below runs through them without stopping at each word
    int cnt = 0;
    {
        int32_t cv[kItemChunks];
#pragma unroll
        for (int c = 0; c < kItemChunks; ++c)
            cv[c] = c * kWave + lane < ne ? cand[e0 + c * kWave + lane] : 0;
#pragma unroll
        for (int c = 0; c < kItemChunks; ++c) {
            if (c * kWave < ne) {
                const uint64_t m =
                    masks ? uint64_t(uniform64(
                                int64_t(masks[(it * ngroups + grp) * kItemChunks + c])))
                          : ballot(c * kWave + lane < ne);
                if ((m >> lane) & 1) {
                    const int o = cnt + __popcll(m & lanemask_lt());
                    s_idx[w][o] = cv[c];
                    s_pos[w][o] = uint16_t(c * kWave + lane);
                }
                cnt += __builtin_popcountll(m);
            }
        }
        if (lane < kItemCands / 32) s_kept[w][lane] = 0;
    }
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");

    float f0 = 0.0f, f1 = 0.0f, f2 = 0.0f;
    uint32_t n1 = 0, n2 = 0, nk = 0;
    const ConstRec recs = const_rec(grec);
    for (int li = 0; li < cnt; li += kWave) {
        const int n = cnt - li < kWave ? cnt - li : kWave;
        const int vidx = lane < n ? s_idx[w][li + lane] : 0;
        uint64_t km = 0;
        // the pair's last part in blk: the decision, and the colours
        auto finish = [&](const PairState<N> &st, const float(&blk)[Pa::PS], int j) {
            const bool kept = (ballot(st.msq <= skip) & vmask) != 0;
            if constexpr (COUNT) {
                const bool k1 = N > 3 ? st.c1 : true, k2 = N > 6 ? st.c2 : k1;
                n1 += k1;
                n2 += k2;
                nk += kept;
            }
            if (!kept) return;
            km |= uint64_t(1) << j;
            if constexpr (OUT) {
                constexpr int o = AC - (Pa::NP - 1) * Pa::PS;
                const float g = __builtin_amdgcn_exp2f(-st.msq);
                f0 = fmaf(g, blk[o + 0], f0);
                f1 = fmaf(g, blk[o + 1], f1);
                f2 = fmaf(g, blk[o + 2], f2);
            }
        };
        // past the last survivor the first one's record again (not used)
        auto rec_of = [&](int j) {
            return recs + int64_t(__builtin_amdgcn_readlane(vidx, j < n ? j : 0)) * R;
        };
        ConstRec r = rec_of(0);
        float b0[Pa::PS], b1[Pa::PS];
        load_part<N, 0>(b0, r);
        if constexpr (Pa::NP == 1) {
            for (int j = 0; j < n; j += 2) {
                PairState<N> st;
                ConstRec r1 = rec_of(j + 1);
                next_part<N, 0>(b1, r1);
                pair_part<N, 0, COUNT>(st, x, b0, vmask, skip);
                finish(st, b0, j);
                if (j + 1 >= n) break;
                r = rec_of(j + 2);
                next_part<N, 0>(b0, r);
                pair_part<N, 0, COUNT>(st, x, b1, vmask, skip);
                finish(st, b1, j + 1);
            }
        } else {
            for (int j = 0; j < n; ++j) {
                PairState<N> st;
                next_part<N, 1>(b1, r);
                pair_part<N, 0, COUNT>(st, x, b0, vmask, skip);
                if constexpr (Pa::NP == 3) {
                    next_part<N, 2>(b0, r);
                    pair_part<N, 1, COUNT>(st, x, b1, vmask, skip);
                    r = rec_of(j + 1);
                    next_part<N, 0>(b1, r);
                    pair_part<N, 2, COUNT>(st, x, b0, vmask, skip);
                    finish(st, b0, j);
#pragma unroll
                    for (int e = 0; e < Pa::PS; ++e) b0[e] = b1[e];
                } else {
                    r = rec_of(j + 1);
                    next_part<N, 0>(b0, r);
                    pair_part<N, 1, COUNT>(st, x, b1, vmask, skip);
                    finish(st, b1, j);
                }
            }
        }
        if ((km >> lane) & 1) {
            const int o = s_pos[w][li + lane];
            atomicOr(&s_kept[w][o / 32], 1u << (o % 32));
        }
    }
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < kItemChunks; ++c) {
        const int o = c * kWave + lane;
        if (o < ne) act[(e0 + o) * ngroups + grp] = uint8_t((s_kept[w][o / 32] >> (o % 32)) & 1u);
    }
    if constexpr (COUNT) {
        if (lane == 0) {
            unsigned long long *sl = stats + it % kStatSlots * 8;
            atomicAdd(&sl[0], static_cast<unsigned long long>(ne));
            atomicAdd(&sl[1], static_cast<unsigned long long>(cnt));
            atomicAdd(&sl[2], static_cast<unsigned long long>(n1));
            atomicAdd(&sl[3], static_cast<unsigned long long>(n2));
            atomicAdd(&sl[4], static_cast<unsigned long long>(nk));
        }
    }
    if constexpr (!OUT) return;
    if (!valid) return;
    if (nit == 1) {
        const int64_t o = perm[p];
        out[o * 3 + 0] = f0;
        out[o * 3 + 1] = f1;
        out[o * 3 + 2] = f2;
    } else {
        float *pp = part + it * 3 * int64_t(tile);
        pp[s] = f0;
        pp[tile + s] = f1;
        pp[2 * tile + s] = f2;
    }
}

template <int N> hipError_t records_n(const ngd_mixture *mix, ngd_cull *c, hipStream_t s)
{
    k_gauss_records<N><<<unsigned((c->k + kWave - 1) / kWave), kWave, 0, s>>>(
        c->k, mix->rec.as<float>(), c->gperm.as<int32_t>(), c->grec.as<float>(),
        c->mrec.as<f16x8>());
    return hipGetLastError();
}

template <int N>
hipError_t culled_n(const ngd_cull *c, float *out, unsigned long long *stats, hipStream_t s)
{
    const int tile = c->params.tile;
    const unsigned gy = unsigned((tile + kMThreads - 1) / kMThreads);
    const float skip = float(-std::log2(double(c->params.tau)) + kSkipLog2Margin);
    // A handful of candidates an item are evaluated at once, and so are all in
    // one dimension, whose tiles keep nearly every candidate.  Without the filter
    // and with it: n = 10, Q = 2^20, K = 200 (4.9 candidates an item) 31 and 54 us,
    // K = 1,000 (24) 73 and 53; Q = 2^18, K = 500 (20) 28 and 19; K = 4,096, Q =
    // 32,768 in tiles of one (1.3) 32 and 137, of 4 (11) 36 and 60, of 16 (70) 55
    // and 26; n = 12, Q = 2^20, K = 300 (8.2) 45 and 65; n = 4, Q = 2^18, K = 300
    // (7.8) 13 and 17; n = 3, Q = 2^20, K = 60 (60) 42 and 47, Q = 30,000, K = 2,000
    // (160) 41 and 29; n = 1, K = 500, Q = 30,000 (121) 23 and 27.
    const bool filter = N > 1 && c->total > (N <= 3 ? 64 : 12) * c->nitems;
    // no idle waves for tiles of fewer than 256 queries
    const int threads = tile < kMThreads ? (tile + kWave - 1) / kWave * kWave : kMThreads;
    for (int64_t i0 = 0; i0 < c->nitems; i0 += max_grid(kMThreads)) {
        const dim3 grid(unsigned(std::min(c->nitems - i0, max_grid(kMThreads))), gy);
        if (filter)
            k_filter_items<N><<<grid, kMThreads, 0, s>>>(
                i0, c->q, tile, c->mrec.as<f16x8>(), c->tcen.as<float>(), c->qs.as<float>(),
                c->tile_off.as<int64_t>(), c->cand.as<int32_t>(), c->item_tile.as<int32_t>(),
                c->item_off.as<int64_t>(), skip, c->fmask.as<uint64_t>());
        auto go = [&](auto kern) {
            kern<<<grid, threads, 0, s>>>(
                i0, c->q, tile, filter ? c->fmask.as<uint64_t>() : nullptr, c->qs.as<float>(),
                c->grec.as<float>(), c->tile_off.as<int64_t>(), c->cand.as<int32_t>(),
                c->perm.as<int32_t>(), c->item_tile.as<int32_t>(), c->item_off.as<int64_t>(),
                skip, c->act.as<uint8_t>(), out, c->fpart.as<float>(), stats);
        };
        if (stats)
            go(k_eval_items<N, false, true>);
        else if (out)
            go(k_eval_items<N, true, false>);
        else
            go(k_eval_items<N, false, false>);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !out) return e;
    // as many items as tiles and none with two: every tile has written its own
    if (c->nitems == c->ntiles && c->max_per_tile <= kItemCands) return hipSuccess;
    return launch_eval_reduce(c, out, s);
}

}  // namespace

size_t mfma_rec_bytes(int n)
{
    return size_t((tri(n) + 7) / 8 + (n + 2 + 3) / 4) * sizeof(f16x8);
}

hipError_t launch_gauss_records(const ngd_mixture *mix, ngd_cull *c, hipStream_t s)
{
    if (c->k == 0) return hipSuccess;
    switch (mix->n) {
#define NGD_CASE(NN) \
    case NN: return records_n<NN>(mix, c, s);
        NGD_CASE(1) NGD_CASE(2) NGD_CASE(3) NGD_CASE(4) NGD_CASE(5) NGD_CASE(6)
        NGD_CASE(7) NGD_CASE(8) NGD_CASE(9) NGD_CASE(10) NGD_CASE(11) NGD_CASE(12)
#undef NGD_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_eval_culled(const ngd_mixture *mix, const ngd_cull *c, float *out,
                              unsigned long long *stats, hipStream_t s)
{
    if (c->q == 0 || c->ntiles == 0) return hipSuccess;
    switch (mix->n) {
#define NGD_CASE(NN) \
    case NN: return culled_n<NN>(c, out, stats, s);
        NGD_CASE(1) NGD_CASE(2) NGD_CASE(3) NGD_CASE(4) NGD_CASE(5) NGD_CASE(6)
        NGD_CASE(7) NGD_CASE(8) NGD_CASE(9) NGD_CASE(10) NGD_CASE(11) NGD_CASE(12)
#undef NGD_CASE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ngd
