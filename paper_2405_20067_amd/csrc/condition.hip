// Conditioning of every Gaussian of a mixture on fixed values of its
// trailing dimensions (the paper's global conditioning, Sec. 3.2: when all
// inputs but the world position are constant over an image, the N-D
// Gaussians are conditioned on them and culled and evaluated as 3-D ones).
// With V = L L^T split into the kept dimensions 0..p-1 and the fixed ones
// p..n-1, the textbook Schur complement gives, for every x_p,
//   G_n(x_p, x_c) = exp(-M_c / 2) G_p(x_p),
//   G_p: mean  m_p + V_pc V_cc^-1 (x_c - m_c),
//        cov   V_pp - V_pc V_cc^-1 V_cp,
//   M_c = (x_c - m_c)^T V_cc^-1 (x_c - m_c),
// so the conditioned mixture (weights alpha exp(-M_c / 2), colours as they
// are) takes the same values over x_p as the N-D one at (x_p, x_c).
// Float64 throughout, one thread per Gaussian.  The fixed dimensions are
// conditioned on one at a time, the last first: with d = V_jj and the residual
// r = x_j - m_j,
//   M_c += r^2 / d,  m_i += V_ij r / d,  V_ik -= V_ij V_kj / d   (i, k < j),
// which is the block formula above by the chain rule of conditioning (the
// elimination of V_cc from its last row up).  The output factor is the
// Cholesky factor of the p x p block that is left.
//
// The kernel is bound by its reads (4 (2N + T) bytes per Gaussian) as long as
// V stays in registers: every loop runs over compile-time indices with
// wave-uniform tests of p.  With run-time loop bounds V, F and Z lay in
// scratch, 3,360 bytes a lane at N = 10 (K = 262,144, p = 3: 325 us, now
// 23 us, 3.3 TB/s of reads and writes).
#include "ngd_internal.hpp"

namespace ngd {
namespace {

constexpr int kThreads = 128;

struct CondArgs {
    float xc[NGD_MAX_N];
};

template <int N>
__global__ __launch_bounds__(kThreads) void k_condition(
    int64_t k, int p, CondArgs args, const float *__restrict__ rec,
    const float *__restrict__ lfac, float *__restrict__ mean_out,
    float *__restrict__ factor_out, float *__restrict__ weight_out,
    float *__restrict__ colour_out)
{
    constexpr int T = N * (N + 1) / 2;
    constexpr int R = (N + T + 7 + 3) / 4 * 4;
    const int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= k) return;
    const int tp = p * (p + 1) / 2;
    const float *rc = rec + i * R;
    double mu[N];
#pragma unroll
    for (int a = 0; a < N; ++a) mu[a] = double(rc[a]);
    // V = L L^T, lower triangle by rows
    double V[T];
    {
        double L[T];
#pragma unroll
        for (int e = 0; e < T; ++e) L[e] = double(lfac[i * T + e]);
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int c = 0; c <= r; ++c) {
                double acc = 0.0;
#pragma unroll
                for (int q = 0; q <= c; ++q)
                    acc = fma(L[r * (r + 1) / 2 + q], L[c * (c + 1) / 2 + q], acc);
                V[r * (r + 1) / 2 + c] = acc;
            }
    }
    bool bad = false;
    // the fixed dimensions, last one first (p is the same for every lane)
    double mc = 0.0;
#pragma unroll
    for (int j = N - 1; j >= 1; --j) {
        if (j >= p) {
            const int row = j * (j + 1) / 2;
            double d = V[row + j];
            bad |= !(d > 0.0);
            d = d > 0.0 ? d : 1.0;
            const double inv = 1.0 / d;
            const double res = double(args.xc[j - p]) - mu[j];
            mc = fma(res * res, inv, mc);
#pragma unroll
            for (int r = 0; r < j; ++r) {
                const double g = V[row + r] * inv;
                mu[r] = fma(g, res, mu[r]);
#pragma unroll
                for (int c = 0; c <= r; ++c)
                    V[r * (r + 1) / 2 + c] = fma(-g, V[row + c], V[r * (r + 1) / 2 + c]);
            }
        }
    }
    // the Cholesky factor of what is left (positive diagonal), in place
#pragma unroll
    for (int r = 0; r < N - 1; ++r) {
        if (r < p) {
            mean_out[i * p + r] = float(mu[r]);
#pragma unroll
            for (int c = 0; c <= r; ++c) {
                double acc = V[r * (r + 1) / 2 + c];
#pragma unroll
                for (int q = 0; q < c; ++q)
                    acc = fma(-V[r * (r + 1) / 2 + q], V[c * (c + 1) / 2 + q], acc);
                if (r == c) {
                    bad |= !(acc > 0.0);
                    acc = sqrt(acc > 0.0 ? acc : 1.0);
                } else {
                    acc /= V[c * (c + 1) / 2 + c];
                }
                V[r * (r + 1) / 2 + c] = acc;
                factor_out[i * tp + r * (r + 1) / 2 + c] = float(acc);
            }
        }
    }
    const double alpha = double(rc[N + T + 3]);
    weight_out[i] = float(alpha * exp(-0.5 * mc));
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) colour_out[i * 3 + ch] = rc[N + T + 4 + ch];
    if (bad) {
        // a conditional covariance that is not positive in float64: the
        // output factor gets a zero diagonal, which ngd_mixture_update of the
        // conditioned mixture reports (ngd_mixture_validate: NGD_E_SINGULAR)
        for (int r = 0; r < p; ++r) factor_out[i * tp + r * (r + 1) / 2 + r] = 0.0f;
    }
}

template <int N>
hipError_t condition_n(const ngd_mixture *mix, int p, const CondArgs &a, float *mean_out,
                       float *factor_out, float *weight_out, float *colour_out, hipStream_t s)
{
    k_condition<N><<<unsigned((mix->k + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        mix->k, p, a, mix->rec.as<float>(), mix->lfac.as<float>(), mean_out, factor_out,
        weight_out, colour_out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_condition(const ngd_mixture *mix, int p, const float *xc, float *mean_out,
                            float *factor_out, float *weight_out, float *colour_out,
                            hipStream_t s)
{
    if (mix->k == 0) return hipSuccess;
    CondArgs a{};
    for (int j = 0; j < mix->n - p; ++j) a.xc[j] = xc[j];
    switch (mix->n) {
#define NGD_CASE(NN) \
    case NN: return condition_n<NN>(mix, p, a, mean_out, factor_out, weight_out, colour_out, s);
        NGD_CASE(2) NGD_CASE(3) NGD_CASE(4) NGD_CASE(5) NGD_CASE(6)
        NGD_CASE(7) NGD_CASE(8) NGD_CASE(9) NGD_CASE(10) NGD_CASE(11) NGD_CASE(12)
#undef NGD_CASE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ngd
