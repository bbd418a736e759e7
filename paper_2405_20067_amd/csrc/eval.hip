// Forward evaluation of the mixture colour (Sec. 4.1, Eq. 8):
//   f(x) = sum_i exp2(-|S'_i (x - m_i)|^2) alpha_i c_i,  S' = sqrt(log2(e)/2) L^-1
//
// without a cull: the plain direct sum over all Gaussians, lane = query, the
// records through scalar loads.  The culled forward is in eval_mfma.hip; the
// sum over the items of a tile that has several is here.
#include "eval_common.hpp"
#include "ngd_internal.hpp"
#include "wave.hpp"

namespace ngd {
namespace {

constexpr int kEvalThreads = 256;

// The plain direct sum.  A lane holds NQ queries, so that a record's scalar
// loads and their waits serve NQ distances; records alternate between two
// register blocks, the next one's load issued after the wait for the current.
// SPLIT: the workgroup's W waves take the same 64 NQ queries and split the
// Gaussians into W consecutive ranges; the partial sums are added in float64 and
// range order through LDS, so the result does not depend on scheduling (in
// float32 sixteen of them had a larger error than four: K = 256, n = 4 8.9e-8
// root mean square against 8.2e-8, now 7.0e-8).  Otherwise
// each wave has its own queries and sums all Gaussians.
// Bound by the vector operations (N = 4: 25 issue slots a pair with the exp).
// K = 256, Q = 65,536, n = 4, one query a lane, 16 waves: 13.5 us, 10 of them
// vector issue (15.2 with four queries a lane); with 4 waves whose records came
// through vector loads 41.9 us.
template <int N, int NQ, int W, bool SPLIT>
__global__ __launch_bounds__(W *kWave) void k_eval_dense(int64_t k, int64_t q,
                                                         const float *__restrict__ rec,
                                                         const float *__restrict__ queries,
                                                         float *__restrict__ out)
{
    using Lay = RecLayout<N>;
    constexpr int kQ = NQ * kWave;   // queries of a wave
    const int w = int(threadIdx.x) / kWave, lane = lane_id();
    const int64_t p0 = (SPLIT ? int64_t(blockIdx.x) : int64_t(blockIdx.x) * W + w) * kQ;
    float x[NQ][N], f[NQ][3];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int64_t p = p0 + u * kWave + lane;
#pragma unroll
        for (int a = 0; a < N; ++a) x[u][a] = p < q ? queries[p * N + a] : 0.0f;
        f[u][0] = f[u][1] = f[u][2] = 0.0f;
    }
    // 32-bit uniform indices (k < 2^31) and unconditional loads (past the
    // range, its last record again): the records then go through scalar loads
    const int per = uniform(int(SPLIT ? (k + W - 1) / W : k));
    const int i0 = SPLIT ? uniform(w) * per : 0;
    const int n = uniform(int(i0 >= k ? 0 : (k - i0 < per ? k - i0 : per)));
    float bufA[Lay::PF], bufB[Lay::PF];
    auto add = [&](const float(&blk)[Lay::PF], ConstRec r) {
#pragma unroll
        for (int u = 0; u < NQ; ++u)
            eval_pair<N>(blk, r, x[u], f[u][0], f[u][1], f[u][2]);
    };
    if (n > 0) {
        ConstRec r = const_rec(rec) + int64_t(i0) * Lay::R;
        ConstRec last = r + int64_t(n - 1) * Lay::R;
        load_block<N>(bufA, r);
        for (int left = n; left > 0; left -= 2) {
            ConstRec r1 = left > 1 ? r + Lay::R : last;
            ConstRec r2 = left > 2 ? r + 2 * Lay::R : last;
            wait_scalar_then(r1);
            load_block<N>(bufB, r1);
            add(bufA, r);
            if (left == 1) break;
            wait_scalar_then(r2);
            load_block<N>(bufA, r2);
            add(bufB, r1);
            r = r2;
        }
    }
    if constexpr (SPLIT) {
        __shared__ float part[W][3][kQ];
#pragma unroll
        for (int u = 0; u < NQ; ++u)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) part[w][ch][u * kWave + lane] = f[u][ch];
        __syncthreads();
        // consecutive threads on consecutive outputs
        for (int e = int(threadIdx.x); e < 3 * kQ; e += W * kWave) {
            const int s = e / 3, ch = e - 3 * s;
            if (p0 + s >= q) break;
            double acc = part[0][ch][s];
#pragma unroll
            for (int v = 1; v < W; ++v) acc += double(part[v][ch][s]);
            out[p0 * 3 + e] = float(acc);
        }
    } else {
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int64_t p = p0 + u * kWave + lane;
            if (p >= q) break;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) out[p * 3 + ch] = f[u][ch];
        }
    }
}

// Tiles with no item (no candidates) get zeros; tiles with two or more items
// get the sum of their items' partials in item order.
__global__ __launch_bounds__(kEvalThreads) void k_eval_reduce(
    int64_t q, int tile, const int32_t *__restrict__ perm, const int64_t *__restrict__ item_off,
    const float *__restrict__ part, float *__restrict__ out)
{
    const int64_t t = blockIdx.x;
    const int64_t i0 = item_off[t], i1 = item_off[t + 1];
    if (i1 - i0 == 1) return;
    const int s = int(blockIdx.y) * kEvalThreads + int(threadIdx.x);
    const int64_t p = t * tile + s;
    if (s >= tile || p >= q) return;
    float f0 = 0.0f, f1 = 0.0f, f2 = 0.0f;
    for (int64_t i = i0; i < i1; ++i) {
        const float *pp = part + i * 3 * int64_t(tile);
        f0 += pp[s];
        f1 += pp[tile + s];
        f2 += pp[2 * tile + s];
    }
    const int64_t o = perm[p];
    out[o * 3 + 0] = f0;
    out[o * 3 + 1] = f1;
    out[o * 3 + 2] = f2;
}

template <int N>
hipError_t dense_n(const ngd_mixture *mix, const float *queries, int64_t q, float *out,
                   hipStream_t s)
{
    auto go = [&](auto kern, int per_block, int waves) {
        kern<<<unsigned((q + per_block - 1) / per_block), waves * kWave, 0, s>>>(
            mix->k, q, mix->rec.as<float>(), queries, out);
        return hipGetLastError();
    };
    // Too few Gaussians to share, or few and many queries: a wave per 64 queries.
    // Otherwise four waves share the Gaussians, sixteen where the queries alone
    // leave the chip idle.  n = 8, 4 / 16 waves: K = 1,000, Q = 2,000 67 / 34 us,
    // 70,000 137 / 118, 2^18 367 / 353; K = 64, Q = 2^17 18 / 32; n = 10: K = 1,000,
    // Q = 70,000 186 / 198, 2^18 516 / 632.  n = 8, K = 16, Q = 2^20: one wave 34,
    // four 61; n = 4, K = 15, Q = 2^18 - 1: one 11.3 with its launch, sixteen 18.8.
    // Four queries a lane pay in one dimension only, whose pairs are cheaper than
    // the waits for their records (K = 1,000: Q = 2^20 268 us against 292, 2^18 67
    // against 82; n = 10, 2^20 2,204 against 1,966).
    // Records beyond an XCD's L2 (4 MiB) bind by their own reading, which two or
    // four queries a lane share: K = 262,144, Q = 2^18 150 ms with two and four
    // waves, 180 with one; Q = 2^16 42 with four and sixteen, 54; K = 20,000, Q =
    // 2^16 - 1 3.2 with two and sixteen, 3.8.
    if (mix->k * int64_t(RecLayout<N>::R * sizeof(float)) > (int64_t(4) << 20) &&
        q >= (int64_t(1) << 15)) {
        if (q >= (int64_t(1) << 18)) return go(k_eval_dense<N, 2, 4, true>, 2 * kWave, 4);
        if (q >= (int64_t(1) << 16)) return go(k_eval_dense<N, 4, 16, true>, 4 * kWave, 16);
        return go(k_eval_dense<N, 2, 16, true>, 2 * kWave, 16);
    }
    if constexpr (N == 1) {
        if (mix->k >= 64 && q >= (int64_t(1) << 16)) {
            if (q >= (int64_t(1) << 20)) return go(k_eval_dense<N, 4, 4, false>, 16 * kWave, 4);
            if (q >= (int64_t(1) << 18)) return go(k_eval_dense<N, 4, 4, true>, 4 * kWave, 4);
            return go(k_eval_dense<N, 4, 16, true>, 4 * kWave, 16);
        }
    }
    if (mix->k < 16 || (mix->k < 64 && q >= (int64_t(1) << 19)))
        return go(k_eval_dense<N, 1, 4, false>, 4 * kWave, 4);
    const int64_t few = N < 10 ? int64_t(1) << 17 : int64_t(1) << 16;
    if (mix->k < 256 || q >= few) return go(k_eval_dense<N, 1, 4, true>, kWave, 4);
    return go(k_eval_dense<N, 1, 16, true>, kWave, 16);
}

}  // namespace

hipError_t launch_eval_reduce(const ngd_cull *c, float *out, hipStream_t s)
{
    const int tile = c->params.tile;
    const int per = tile < kEvalThreads ? (tile + 63) / 64 * 64 : kEvalThreads;
    const unsigned gy = unsigned((tile + kEvalThreads - 1) / kEvalThreads);
    k_eval_reduce<<<dim3(unsigned(c->ntiles), gy), per, 0, s>>>(
        c->q, tile, c->perm.as<int32_t>(), c->item_off.as<int64_t>(), c->fpart.as<float>(), out);
    return hipGetLastError();
}

hipError_t launch_eval_dense(const ngd_mixture *mix, const float *queries, int64_t q, float *out,
                             hipStream_t s)
{
    if (q == 0) return hipSuccess;
    switch (mix->n) {
#define NGD_CASE(NN) \
    case NN: return dense_n<NN>(mix, queries, q, out, s);
        NGD_CASE(1) NGD_CASE(2) NGD_CASE(3) NGD_CASE(4) NGD_CASE(5) NGD_CASE(6)
        NGD_CASE(7) NGD_CASE(8) NGD_CASE(9) NGD_CASE(10) NGD_CASE(11) NGD_CASE(12)
#undef NGD_CASE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ngd
