// Shared by the forward kernels (eval.hip, eval_mfma.hip): record layout, the
// rows of y = S'(x - m), and the uniform record loads.
#pragma once

#include <utility>

#include "ngd_internal.hpp"
#include "wave.hpp"

namespace ngd {

// s_waitcnt immediate that waits for all scalar-memory (and LDS) loads only:
// vmcnt and expcnt at their maxima, lgkmcnt 0.
constexpr int kWaitScalar = 0xC07F;

template <int N> struct RecLayout {
    static constexpr int T = N * (N + 1) / 2;
    static constexpr int R = (N + T + 7 + 3) / 4 * 4;
    static constexpr int AC = N + T;
    static constexpr int PF = R < 32 ? R : 32;   // floats loaded ahead
};

// A record as constant memory: a wave-uniform address then always takes a
// scalar load, also inside a loop whose waits the compiler takes for stores.
typedef const __attribute__((address_space(4))) float *ConstRec;
__device__ __forceinline__ ConstRec const_rec(const float *r)
{
    return reinterpret_cast<ConstRec>(reinterpret_cast<uintptr_t>(r));
}

// Record field e: from the prefetched block when e < PF, else from memory.
template <int N, int E, class P>
__device__ __forceinline__ float field(const float (&blk)[RecLayout<N>::PF], P r)
{
    if constexpr (E < RecLayout<N>::PF)
        return blk[E];
    else
        return r[E];
}

// Rows [R0, R1) of y = S'(x - m), accumulated into msq; d holds x - m.
template <int N, int R0, int R1, class P>
__device__ __forceinline__ void rows(const float (&blk)[RecLayout<N>::PF], P r,
                                     const float (&x)[N], float (&d)[N], float (&y)[N],
                                     float &msq)
{
    if constexpr (R0 < R1) {
        d[R0] = x[R0] - field<N, R0>(blk, r);
        constexpr int base = N + R0 * (R0 + 1) / 2;
        float acc = field<N, base>(blk, r) * d[0];
        [&]<int... J>(std::integer_sequence<int, J...>) {
            ((acc = fmaf(field<N, base + 1 + J>(blk, r), d[1 + J], acc)), ...);
        }(std::make_integer_sequence<int, R0>{});
        y[R0] = acc;
        msq = fmaf(acc, acc, msq);
        rows<N, R0 + 1, R1>(blk, r, x, d, y, msq);
    }
}

// Accumulates one Gaussian into f for this lane's query x.
template <int N, class P>
__device__ __forceinline__ void eval_pair(const float (&blk)[RecLayout<N>::PF], P r,
                                          const float (&x)[N], float &f0, float &f1, float &f2)
{
    using Lay = RecLayout<N>;
    float d[N], y[N];
    float msq = 0.0f;
    rows<N, 0, N>(blk, r, x, d, y, msq);
    const float g = __builtin_amdgcn_exp2f(-msq);
    f0 = fmaf(g, field<N, Lay::AC + 0>(blk, r), f0);
    f1 = fmaf(g, field<N, Lay::AC + 1>(blk, r), f1);
    f2 = fmaf(g, field<N, Lay::AC + 2>(blk, r), f2);
}

// Waits for every scalar load in flight; loads through `next` stay behind the
// wait (the pointer is made anew after it), so that the wait never covers
// them -- scalar loads complete out of order and can only be waited for all
// together.
__device__ __forceinline__ void wait_scalar_then(ConstRec &next)
{
    uintptr_t u = reinterpret_cast<uintptr_t>(next);
    __builtin_amdgcn_s_waitcnt(kWaitScalar);
    asm volatile("" : "+s"(u));
    next = reinterpret_cast<ConstRec>(u);
}

template <int N, class P>
__device__ __forceinline__ void load_block(float (&blk)[RecLayout<N>::PF], P r)
{
#pragma unroll
    for (int e = 0; e < RecLayout<N>::PF; ++e) blk[e] = r[e];
}

}  // namespace ngd
