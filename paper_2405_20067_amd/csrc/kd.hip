// k-d ordering of points in projection space, the tiling of the cull.
//
// Definition (shared with the CPU re-implementation): a run of n points is
// cut in units of u = leaf while n > leaf, else of u = sub (sub <= leaf);
// it needs T = ceil(n/u) units, and its first ceil(T/2)*u points in the
// order (value on the split projection, then position in the run) go left
// and the rest right, each side keeping its relative order.  The split
// projection is the one of largest extent (max - min) over the run, the
// first such on ties.  Runs of at most `sub` points are leaves; the runs of
// at most `leaf` points (tiles) are those of a split with sub = leaf, the
// finer splits only reorder inside them.  Because every split is an exact
// rank split on a stable order, run boundaries depend only on
// (n, leaf, sub), and the host lays them out level by level.
//
// Levels with a node of more than kNodeMax points run one level at a time
// over all of the level's nodes, each node cut into slices (one workgroup
// each), in five launches:
//   hist 0   per slice of kHistSlice points: the node's split projection
//            (largest extent, from the node's min / max accumulated by the
//            previous level's scatter; for the root from the projections'
//            kernel's partials), then the histogram of the first radix digit (11, 11,
//            10 bits of the order-preserving key), added into the node's
//            round-0 histogram
//   hist 1,2 per slice: the bin of the previous round's histogram that holds
//            the rank n_left (every workgroup of the node finds the same; the
//            node's first records it), then the histogram of the next digit
//            among the points that match the digits found so far
//   count    per slice of kSlice points: the last digit's bin, which
//            completes the pivot key (the first point that goes right); the
//            points below / equal to it
//   scatter  per slice: offsets from the node's earlier slices' counts,
//            stable ranks by workgroup prefix sums in position order; index
//            and projection values move to the next buffer, the children's
//            min / max are accumulated for the next split, and the node's
//            histograms are cleared for the next level
// Levels of nodes of at most kNodeMax points take two launches: the selection
// by a workgroup per node (k_kd_select), with the node's keys in registers and
// the histograms in LDS, and the same scatter.
// Subtrees finish in one workgroup each: nodes of at most kSubMax points in
// k_kd_subtree, which holds the points' keys in LDS, for up to 16 projections
// and runs that start at multiples of 64 points; otherwise nodes of at most
// kLocalMax points in k_kd_local, where every level of the subtree is one
// bitonic sort of (run, key, position) over blocks of the smallest
// power-of-two length that holds every run.
#include <algorithm>
#include <map>
#include <vector>

#include "ngd_internal.hpp"
#include "wave.hpp"

namespace ngd {
namespace {

constexpr int kThreads = 256;
constexpr int kSlice = 1024;        // points per scatter / count workgroup
constexpr int kHistSlice = 4096;    // points per histogram workgroup
constexpr int kBins = 2048;
constexpr int kShift[3] = {21, 10, 0};
constexpr int kWidth[3] = {11, 11, 10};

constexpr int kHistThreads = 512;

constexpr int kLocalMax = 1024;    // points per subtree workgroup (<= 4096: 12-bit positions)
constexpr unsigned kWideLocalBlocks = 512;   // subtrees for the 512-thread variant
// Min / max key slots come in kExtRep planes of max_nodes x P x 2: a
// workgroup merges into plane (blockIdx.x mod kExtRep), so that the atomics
// of the many workgroups of one node (all of them, at the root) spread over
// as many cache lines; readers reduce the planes.
constexpr int kExtRep = 16;
constexpr int kLocalRuns = 128;     // runs per subtree (8-bit run ids)
// Nodes selected by one workgroup, in 10 to 18 us, where three histogram
// rounds and a count take 21 and their gaps; at 32,768 points it took 35.
constexpr int kNodeMax = 16384;
constexpr int kNodeThreads = 1024;
static_assert(kNodeMax == 16 * kNodeThreads, "16 keys a thread");
constexpr int kSubMax = 2048;
constexpr int kSubThreads = 1024;
constexpr int kSubProj = 16;
constexpr int kSubChunks = kSubMax / kWave;
constexpr int kLocalSplit = 64;     // runs split at one level of a subtree

// node table row: start, size, n_left (-1: leaf), first slice, end slice,
// first child's index in the next level (-1: none), first histogram slice,
// end histogram slice
constexpr int kNodeCols = 8;
// slice table row: start, length, node
constexpr int kSliceCols = 3;

// The plane of min / max key slots a workgroup merges into.
__device__ __forceinline__ uint32_t *ext_plane(uint32_t *ext, int64_t max_nodes, int P)
{
    return ext + int64_t(blockIdx.x % kExtRep) * max_nodes * 2 * P;
}

// The root's extents from per-block partials: block (j, 0) reduces projection
// j into plane 0 and puts the other planes at their identities; the blocks
// (., y > 0) clear the histograms.
__global__ __launch_bounds__(kThreads) void k_kd_root(int64_t nparts, int P,
                                                      const uint32_t *__restrict__ part,
                                                      uint32_t *__restrict__ ext,
                                                      int64_t max_nodes,
                                                      int32_t *__restrict__ hist, int64_t nhist)
{
    if (blockIdx.y > 0) {
        const int64_t step = int64_t(gridDim.x) * (gridDim.y - 1) * kThreads;
        for (int64_t i = (int64_t(blockIdx.y - 1) * gridDim.x + blockIdx.x) * kThreads +
                         threadIdx.x;
             i < nhist; i += step)
            hist[i] = 0;
        return;
    }
    __shared__ uint32_t slo[kThreads / kWave], shi[kThreads / kWave];
    const int j = blockIdx.x;
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (int64_t b = threadIdx.x; b < nparts; b += kThreads) {
        lo = min(lo, part[(b * P + j) * 2 + 0]);
        hi = max(hi, part[(b * P + j) * 2 + 1]);
    }
    lo = wave_umin_dpp(lo);
    hi = wave_umax_dpp(hi);
    if (lane_id() == kWave - 1) {
        slo[threadIdx.x / kWave] = lo;
        shi[threadIdx.x / kWave] = hi;
    }
    __syncthreads();
    if (threadIdx.x >= kExtRep) return;
    lo = 0xffffffffu, hi = 0u;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < kThreads / kWave; ++i) {
            lo = min(lo, slo[i]);
            hi = max(hi, shi[i]);
        }
    }
    uint32_t *e = ext + int64_t(threadIdx.x) * max_nodes * 2 * P + 2 * j;
    e[0] = lo;
    e[1] = hi;
}

// Block exclusive scan of one count per thread (THREADS threads).  Every
// caller scans counts of points of one node, whose wave sums stay below
// 2^31 (the point count is): the wave scan runs in 32 bits by DPP, the
// workgroup's combination in 64.
template <int THREADS = kThreads>
__device__ int64_t block_exscan(int64_t v, int64_t *total)
{
    __shared__ int64_t wt[THREADS / kWave];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const int64_t inc = wave_inclusive_scan(int(v));
    if (lane == kWave - 1) wt[w] = inc;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < THREADS / kWave; ++i) {
        before += (i < w) ? wt[i] : 0;
        all += wt[i];
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

// One round of the radix selection, by a whole workgroup: the bin of the
// node's histogram h (2^width bins, of the points matching `pre`) that holds
// rank r; returns the extended prefix and the rank inside that bin.
template <int THREADS>
__device__ void block_select(const int32_t *__restrict__ h, int width, uint32_t pre, int64_t r,
                             uint32_t *out_pre, int64_t *out_rank)
{
    __shared__ uint32_t s_pre;
    __shared__ int64_t s_rank;
    constexpr int kMaxPer = kBins / THREADS;
    const int per = (1 << width) / THREADS;
    int32_t cnt[kMaxPer];
    int64_t mine = 0;
#pragma unroll
    for (int i = 0; i < kMaxPer; ++i) {
        cnt[i] = i < per ? h[threadIdx.x * per + i] : 0;
        mine += cnt[i];
    }
    int64_t tot;
    int64_t cum = block_exscan<THREADS>(mine, &tot);
#pragma unroll
    for (int i = 0; i < kMaxPer; ++i) {
        if (i < per && r >= cum && r < cum + cnt[i]) {
            s_pre = (pre << width) | uint32_t(threadIdx.x * per + i);
            s_rank = r - cum;
        }
        cum += cnt[i];
    }
    __syncthreads();
    *out_pre = s_pre;
    *out_rank = s_rank;
}

// Per slice of kHistSlice points, one round of the radix selection of the
// node's pivot.  Round 0 first picks the node's split projection (its
// first slice records it and resets the children's min / max slots);
// rounds 1 and 2 first finish the previous round (its first slice records
// the prefix and rank).  The histogram of the round's digit among the
// points that match the prefix is added into the node's histogram of the
// round (integer atomics: the sum does not depend on their order).
// sel_pre / sel_rank: 3 x max_nodes, the state after rounds 0, 1, 2.
__global__ __launch_bounds__(kHistThreads) void k_kd_hist(
    const int64_t *__restrict__ nodes, const int64_t *__restrict__ slices, int64_t node0,
    int64_t hslice0, int64_t max_nodes, int64_t hist_nodes, int64_t n, int P, int round,
    const float *__restrict__ vin, const uint32_t *__restrict__ ext,
    uint32_t *__restrict__ ext_next, int32_t *__restrict__ dim, uint32_t *__restrict__ sel_pre,
    int64_t *__restrict__ sel_rank, int32_t *__restrict__ hist)
{
    __shared__ int h[kBins];
    __shared__ float s_ext[32];
    __shared__ int s_dim;
    const int64_t sl = blockIdx.x;
    const int64_t s0 = slices[sl * kSliceCols + 0], len = slices[sl * kSliceCols + 1];
    const int64_t nd = slices[sl * kSliceCols + 2] - node0;
    const int64_t *row = nodes + nd * kNodeCols;
    const int64_t nleft = row[2];
    const bool first = sl + hslice0 == row[6];
    if (nleft < 0) {   // a leaf (uniform over the workgroup)
        if (round == 0 && first && threadIdx.x == 0) dim[nd] = -1;
        return;
    }
    // the slice's keys of projection d, loaded before the previous round's
    // selection so that the two latencies overlap
    constexpr int kPer = kHistSlice / kHistThreads;
    uint32_t keys[kPer];
    auto load_keys = [&](int d) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int64_t i = threadIdx.x + int64_t(u) * kHistThreads;
            keys[u] = i < len ? orderable(vin[int64_t(d) * n + s0 + i]) : 0u;
        }
    };
    uint32_t pre = 0u;
    int d;
    if (round == 0) {
        // the projection of largest extent, the first on ties
        if (int(threadIdx.x) < P) {
            const int j = threadIdx.x;
            uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll 4
            for (int e = 0; e < kExtRep; ++e) {
                const uint32_t *x = ext + int64_t(e) * max_nodes * 2 * P + (nd * P + j) * 2;
                lo = min(lo, x[0]);
                hi = max(hi, x[1]);
            }
            s_ext[j] = from_orderable(hi) - from_orderable(lo);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int best = 0;
            for (int j = 1; j < P; ++j)
                if (s_ext[j] > s_ext[best]) best = j;
            s_dim = best;
        }
        __syncthreads();
        d = s_dim;
        load_keys(d);
        if (first) {
            if (threadIdx.x == 0) dim[nd] = d;
            const int64_t ch = row[5];
            if (ext_next && ch >= 0) {   // both children's slots, every plane
                for (int t = threadIdx.x; t < 2 * P * kExtRep; t += kHistThreads) {
                    uint32_t *x = ext_next + int64_t(t / (2 * P)) * max_nodes * 2 * P +
                                  (ch * P + t % (2 * P)) * 2;
                    x[0] = 0xffffffffu;
                    x[1] = 0u;
                }
            }
        }
    } else {
        d = dim[nd];
        load_keys(d);
        const uint32_t p0 = round == 1 ? 0u : sel_pre[nd];
        const int64_t r0 = round == 1 ? nleft : sel_rank[nd];
        int64_t r1;
        block_select<kHistThreads>(hist + ((round - 1) * hist_nodes + nd) * kBins,
                                   kWidth[round - 1], p0, r0, &pre, &r1);
        if (first && threadIdx.x == 0) {
            sel_pre[(round - 1) * max_nodes + nd] = pre;
            sel_rank[(round - 1) * max_nodes + nd] = r1;
        }
    }
    for (int b = threadIdx.x; b < kBins; b += kHistThreads) h[b] = 0;
    __syncthreads();
    const int shift = kShift[round], width = kWidth[round];
    const uint32_t mask = (1u << width) - 1u;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t key = keys[u];
        const bool valid = threadIdx.x + int64_t(u) * kHistThreads < len;
        const bool match = (round == 0) || ((key >> (shift + width)) == pre);
        if (valid && match) atomicAdd(&h[(key >> shift) & mask], 1);
    }
    __syncthreads();
    int32_t *nh = hist + (round * hist_nodes + nd) * kBins;
    for (int b = threadIdx.x; b < kBins; b += kHistThreads)
        if (h[b]) atomicAdd(&nh[b], h[b]);
}

// Per slice of kSlice points: the last round of the selection (the node's
// first slice records the pivot key and the number of pivot-equal points
// that go left), then the slice's points below and equal to the pivot.
__global__ __launch_bounds__(kThreads) void k_kd_count(
    const int64_t *__restrict__ nodes, const int64_t *__restrict__ slices, int64_t node0,
    int64_t slice0, int64_t max_nodes, int64_t hist_nodes, int64_t n,
    const float *__restrict__ vin, const int32_t *__restrict__ dim, uint32_t *__restrict__ sel_pre,
    int64_t *__restrict__ sel_rank, const int32_t *__restrict__ hist, int64_t *__restrict__ cnt)
{
    const int64_t sl = blockIdx.x;
    const int64_t s0 = slices[sl * kSliceCols + 0], len = slices[sl * kSliceCols + 1];
    const int64_t nd = slices[sl * kSliceCols + 2] - node0;
    const int d = dim[nd];
    int64_t less = 0, eq = 0;
    if (d >= 0) {   // uniform
        // the slice's keys first: their loads overlap the selection
        constexpr int kPer = kSlice / kThreads;
        uint32_t keys[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int64_t i = threadIdx.x + int64_t(u) * kThreads;
            keys[u] = i < len ? orderable(vin[int64_t(d) * n + s0 + i]) : 0u;
        }
        uint32_t pivot;
        int64_t r;
        block_select<kThreads>(hist + (2 * hist_nodes + nd) * kBins, kWidth[2],
                               sel_pre[max_nodes + nd], sel_rank[max_nodes + nd], &pivot, &r);
        if (sl + slice0 == nodes[nd * kNodeCols + 3] && threadIdx.x == 0) {
            sel_pre[2 * max_nodes + nd] = pivot;
            sel_rank[2 * max_nodes + nd] = r;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const bool valid = threadIdx.x + int64_t(u) * kThreads < len;
            less += valid && keys[u] < pivot;
            eq += valid && keys[u] == pivot;
        }
    }
    int64_t tl, te;
    block_exscan(less, &tl);
    block_exscan(eq, &te);
    if (threadIdx.x == 0) {
        cnt[sl * 2 + 0] = tl;
        cnt[sl * 2 + 1] = te;
    }
}

// Minima (MAX: maxima) over the wave of V keys per lane, scattered as
// wave_reduce_scatter does: lane 16 r + 15 holds those of keys
// [r V/4, (r + 1) V/4) in v[0 .. V/4).
template <int V, bool MAX = false> __device__ __forceinline__ void wave_umin_scatter(uint32_t (&v)[V])
{
    static_assert(V % 4 == 0, "keys in four equal rows");
    constexpr int H = V / 2, Q = V / 4;
    auto pick = [](uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); };
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(v[i], v[i + H], false, false);
        v[i] = pick(uint32_t(r[0]), uint32_t(r[1]));
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(v[i], v[i + Q], false, false);
        v[i] = pick(uint32_t(r[0]), uint32_t(r[1]));
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if constexpr (MAX) {
            v[i] = dpp_umax_row<kDppRowShr1>(v[i]);
            v[i] = dpp_umax_row<kDppRowShr2>(v[i]);
            v[i] = dpp_umax_row<kDppRowShr4>(v[i]);
            v[i] = dpp_umax_row<kDppRowShr8>(v[i]);
        } else {
            v[i] = dpp_umin<kDppRowShr1>(v[i]);
            v[i] = dpp_umin<kDppRowShr2>(v[i]);
            v[i] = dpp_umin<kDppRowShr4>(v[i]);
            v[i] = dpp_umin<kDppRowShr8>(v[i]);
        }
    }
}

// Each lane's minimum (maximum) with the lanes 16, 32 and 48 apart.
template <bool MAX> __device__ __forceinline__ uint32_t rows_pick(uint32_t v)
{
    auto pick = [](uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); };
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = pick(uint32_t(r[0]), uint32_t(r[1]));
    const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return pick(uint32_t(q[0]), uint32_t(q[1]));
}

// Moves a slice's points to their node's children: ranks inside the slice by
// ballots, the projections four at a time (a thread's four points of each: 16
// loads in flight), the children's min / max on the way.  Bound by the 2 x 68 B
// a point.
template <int PMAX>
__global__ __launch_bounds__(kThreads) void k_kd_scatter(
    const int64_t *__restrict__ nodes, const int64_t *__restrict__ slices, int64_t node0,
    int64_t slice0, int64_t n, int P, const int32_t *__restrict__ idx_in,
    const float *__restrict__ vin, const int32_t *__restrict__ dim,
    const uint32_t *__restrict__ prefix, const int64_t *__restrict__ rank,
    const int64_t *__restrict__ cnt, int32_t *__restrict__ idx_out, float *__restrict__ vout,
    uint32_t *__restrict__ ext_next, int32_t *__restrict__ hist, int64_t max_nodes,
    int64_t hist_nodes)
{
    constexpr int S = kSlice / kThreads, W = kThreads / kWave, JU = 4;
    static_assert(S * W == 16, "one row of lanes scans the (strip, wave) counts");
    __shared__ int lw[S * W], ew[S * W];
    __shared__ uint32_t e4[W][4 * PMAX];
    const int64_t sl = blockIdx.x;
    const int64_t s0 = slices[sl * kSliceCols + 0];
    const int len = int(slices[sl * kSliceCols + 1]);
    const int64_t nd = slices[sl * kSliceCols + 2] - node0;
    const int64_t *row = nodes + nd * kNodeCols;
    const int64_t start = row[0], size = row[1], nleft = row[2];
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    const int d = dim[nd];
    if (d < 0) {   // a leaf: its points stay where they are
        for (int64_t i = tid; i < len; i += kThreads) {
            const int64_t pos = s0 + i;
            idx_out[pos] = idx_in ? idx_in[pos] : int32_t(pos);
#pragma unroll
            for (int j = 0; j < PMAX; ++j)
                if (j < P) vout[int64_t(j) * n + pos] = vin[int64_t(j) * n + pos];
        }
        return;
    }
    uint32_t key[S];
    int32_t id[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int i = u * kThreads + tid;
        key[u] = i < len ? orderable(vin[int64_t(d) * n + s0 + i]) : 0u;
        id[u] = i < len ? (idx_in ? idx_in[s0 + i] : int32_t(s0 + i)) : 0;
    }
    const int64_t sb = row[3] - slice0;   // the node's first slice
    if (hist && sl == sb) {   // the node's histograms, clean for the next level
        for (int r = 0; r < 3; ++r)
            for (int b = tid; b < kBins; b += kThreads) hist[(r * hist_nodes + nd) * kBins + b] = 0;
    }
    // points below the pivot, and equal to it, in the node's earlier slices
    int64_t l_mine = 0, e_mine = 0;
    for (int64_t s = sb + tid; s < sl; s += kThreads) {
        l_mine += cnt[s * 2 + 0];
        e_mine += cnt[s * 2 + 1];
    }
    const uint32_t pivot = prefix[nd];
    const int64_t need = rank[nd];   // pivot-equal points that go left
    uint64_t bl[S], be[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const bool valid = u * kThreads + tid < len;
        bl[u] = ballot(valid && key[u] < pivot);
        be[u] = ballot(valid && key[u] == pivot);
        if (lane == 0) {
            lw[u * W + w] = __popcll(bl[u]);
            ew[u * W + w] = __popcll(be[u]);
        }
    }
    int64_t l_before, e_before;   // the scans' barriers publish lw and ew too
    block_exscan(l_mine, &l_before);
    block_exscan(e_mine, &e_before);
    const int lv = lw[lane & 15], ev = ew[lane & 15];
    const int lx = wave_inclusive_scan(lane < 16 ? lv : 0) - lv;
    const int ex = wave_inclusive_scan(lane < 16 ? ev : 0) - ev;
    int64_t dst[S];
    bool left[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int i = u * kThreads + tid;
        const int at = uniform(u * W + w);
        const bool less = (bl[u] >> lane) & 1, eq = (be[u] >> lane) & 1;
        const int64_t lb =
            l_before + __builtin_amdgcn_readlane(lx, at) + __popcll(bl[u] & lanemask_lt());
        const int64_t eb =
            e_before + __builtin_amdgcn_readlane(ex, at) + __popcll(be[u] & lanemask_lt());
        left[u] = less || (eq && eb < need);
        const int64_t lr = lb + (eb < need ? eb : need);
        dst[u] = left[u] ? start + lr : start + nleft + (s0 + i - start - lr);
        // every destination lies in the node's own run (the counts agree);
        // the test only guards the buffers should they ever not
        if (i >= len || dst[u] < start || dst[u] >= start + size) dst[u] = -1;
        if (dst[u] >= 0) idx_out[dst[u]] = id[u];
    }
    const int64_t ch = row[5];
    const bool track = ext_next != nullptr && ch >= 0;
#pragma unroll
    for (int j0 = 0; j0 < PMAX; j0 += JU) {
        if (j0 >= P) break;   // uniform
        float v[JU][S];
#pragma unroll
        for (int jj = 0; jj < JU; ++jj)
#pragma unroll
            for (int u = 0; u < S; ++u) {
                const int i = u * kThreads + tid;
                v[jj][u] = (j0 + jj < P && i < len) ? vin[int64_t(j0 + jj) * n + s0 + i] : 0.0f;
            }
        // left min, left ~max, right min, right ~max
        uint32_t mm[4 * JU];
#pragma unroll
        for (int e = 0; e < 4 * JU; ++e) mm[e] = 0xffffffffu;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            if (dst[u] < 0) continue;
#pragma unroll
            for (int jj = 0; jj < JU; ++jj) {
                if (j0 + jj < P) vout[int64_t(j0 + jj) * n + dst[u]] = v[jj][u];
                const uint32_t k = orderable(v[jj][u]);
                mm[4 * jj + 0] = min(mm[4 * jj + 0], left[u] ? k : 0xffffffffu);
                mm[4 * jj + 1] = min(mm[4 * jj + 1], left[u] ? ~k : 0xffffffffu);
                mm[4 * jj + 2] = min(mm[4 * jj + 2], left[u] ? 0xffffffffu : k);
                mm[4 * jj + 3] = min(mm[4 * jj + 3], left[u] ? 0xffffffffu : ~k);
            }
        }
        if (track) {
            wave_umin_scatter<4 * JU>(mm);
            if ((lane & 15) == 15)
#pragma unroll
                for (int e = 0; e < JU; ++e) e4[w][4 * j0 + (lane >> 4) * JU + e] = mm[e];
        }
    }
    if (!track) return;   // uniform
    __syncthreads();
    uint32_t *plane = ext_plane(ext_next, max_nodes, P);
    for (int t = tid; t < 4 * P; t += kThreads) {
        uint32_t m = 0xffffffffu;
#pragma unroll
        for (int i = 0; i < W; ++i) m = min(m, e4[i][t]);
        if (m == 0xffffffffu) continue;   // no point on that side
        uint32_t *x = &plane[((ch + (t & 3) / 2) * P + t / 4) * 2 + (t & 1)];
        if (t & 1)
            atomicMax(x, ~m);
        else
            atomicMin(x, m);
    }
}

// The selection of a level whose nodes have at most S x 1024 points, a
// workgroup per node, its keys in registers: split projection from the node's
// extents; a histogram of 2,048 equal steps over the node's range on it, in
// floats (a monotone map: its rounding only moves equal values together); the
// points of the bin that holds the pivot's rank, ranked by (key, position).
// More than kListMax of them (ties, infinite ranges) are resolved by radix
// rounds instead, whose first digit, mostly exponent, puts most of a wave's
// counts on a few LDS words.  Then the slices' counts.
constexpr int kListMax = 256;
template <int S>
__global__ __launch_bounds__(kNodeThreads) void k_kd_select(
    int64_t node_first, const int64_t *__restrict__ nodes, int64_t slice0, int64_t n, int P,
    const float *__restrict__ vin, const uint32_t *__restrict__ ext, int64_t max_nodes,
    uint32_t *__restrict__ ext_next, int32_t *__restrict__ dim, uint32_t *__restrict__ pre_out,
    int64_t *__restrict__ rank_out, int64_t *__restrict__ cnt)
{
    constexpr int W = kNodeThreads / kWave;
    static_assert(kNodeThreads == kSlice, "a strip of points is a slice");
    __shared__ int h[kBins];
    __shared__ int lcnt[S][W], ecnt[S][W];
    __shared__ float s_ext[32], s_lo[32];
    __shared__ uint64_t s_list[kListMax];
    __shared__ int s_num, s_need;
    __shared__ uint32_t s_pivot;
    const int64_t nd = node_first + blockIdx.x;
    const int64_t *row = nodes + nd * kNodeCols;
    const int64_t start = row[0];
    const int size = int(row[1]), nleft = int(row[2]);
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    if (nleft < 0) {   // a leaf
        if (tid == 0) dim[nd] = -1;
        return;
    }
    // the projection of largest extent, the first on ties: 16 lanes per
    // projection, one for each plane of its slots
    static_assert(kExtRep == 16, "a row of lanes reduces the planes");
    if (tid < 16 * P) {
        const int j = tid / 16;
        const uint32_t *x = ext + int64_t(tid % 16) * max_nodes * 2 * P + (nd * P + j) * 2;
        uint32_t lo = x[0], nhi = ~x[1];
        lo = dpp_umin<kDppRowShr1>(lo), nhi = dpp_umin<kDppRowShr1>(nhi);
        lo = dpp_umin<kDppRowShr2>(lo), nhi = dpp_umin<kDppRowShr2>(nhi);
        lo = dpp_umin<kDppRowShr4>(lo), nhi = dpp_umin<kDppRowShr4>(nhi);
        lo = dpp_umin<kDppRowShr8>(lo), nhi = dpp_umin<kDppRowShr8>(nhi);
        if (tid % 16 == 15) {
            s_ext[j] = from_orderable(~nhi) - from_orderable(lo);
            s_lo[j] = from_orderable(lo);
        }
    }
    for (int b = tid; b < kBins; b += kNodeThreads) h[b] = 0;
    if (tid == 0) s_num = 0;
    __syncthreads();
    int d = 0;
    {
        // an extent that is not a number counts only in the first place
        const float e = lane < P ? s_ext[lane & 31] : 0.0f;
        uint32_t ek = e == e ? orderable(e) : (lane == 0 ? 0xffffffffu : 0u);
        if (lane >= P) ek = 0u;
        const uint32_t best = __builtin_amdgcn_readlane(wave_umax_dpp(ek), kWave - 1);
        d = __builtin_ctzll(ballot(ek == best));
    }
    const float *vd = vin + int64_t(d) * n + start;
    uint32_t key[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int i = s * kNodeThreads + tid;
        key[s] = i < size ? orderable(vd[i]) : 0u;
    }
    if (tid == 0) dim[nd] = d;
    const int64_t ch = row[5];
    if (ext_next && ch >= 0) {   // both children's slots, every plane
        for (int t = tid; t < 2 * P * kExtRep; t += kNodeThreads) {
            uint32_t *x = ext_next + int64_t(t / (2 * P)) * max_nodes * 2 * P +
                          (ch * P + t % (2 * P)) * 2;
            x[0] = 0xffffffffu;
            x[1] = 0u;
        }
    }
    // the key of rank nleft, and how many of its equals go left
    uint32_t pivot = 0;
    int64_t need = nleft;
    const float vlo = s_lo[d], ve = s_ext[d];
    float scale = (ve > 0.0f && ve < INFINITY) ? float(kBins) / ve : 0.0f;
    if (!(scale < INFINITY)) scale = 0.0f;
    auto bin_of = [&](uint32_t k) {
        const float t = (from_orderable(k) - vlo) * scale;
        return t > 0.0f ? min(int(t), kBins - 1) : 0;   // not a number: 0
    };
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s * kNodeThreads + tid < size) atomicAdd(&h[bin_of(key[s])], 1);
    __syncthreads();
    uint32_t bin;
    int64_t r;
    block_select<kNodeThreads>(h, 11, 0u, nleft, &bin, &r);
    const int num = h[bin];
    if (num <= kListMax) {   // uniform
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int i = s * kNodeThreads + tid;
            if (i < size && bin_of(key[s]) == int(bin)) {
                const int slot = atomicAdd(&s_num, 1);
                if (slot < kListMax) s_list[slot] = uint64_t(key[s]) << 32 | uint32_t(i);
            }
        }
        __syncthreads();
        if (tid < num) {
            const uint64_t mine = s_list[tid];
            int rank = 0, eq = 0;
            for (int i = 0; i < num; ++i) {
                const uint64_t x = s_list[i];
                rank += x < mine;
                eq += x < mine && (x >> 32) == (mine >> 32);
            }
            if (rank == r) {
                s_pivot = uint32_t(mine >> 32);
                s_need = eq;
            }
        }
        __syncthreads();
        pivot = s_pivot;
        need = s_need;
    } else {
#pragma unroll
        for (int rd = 0; rd < 3; ++rd) {
            __syncthreads();
            for (int b = tid; b < kBins; b += kNodeThreads) h[b] = 0;
            __syncthreads();
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (s * kNodeThreads + tid < size &&
                    (rd == 0 || (key[s] >> ((kShift[rd] + kWidth[rd]) & 31)) == pivot))
                    atomicAdd(&h[(key[s] >> kShift[rd]) & ((1u << kWidth[rd]) - 1u)], 1);
            __syncthreads();
            uint32_t pre;
            int64_t rank;
            block_select<kNodeThreads>(h, kWidth[rd], pivot, need, &pre, &rank);
            pivot = pre;
            need = rank;
        }
    }
    if (tid == 0) {
        pre_out[nd] = pivot;
        rank_out[nd] = need;
    }
    // the slices' points below and equal to the pivot
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const bool valid = s * kNodeThreads + tid < size;
        const uint64_t bl = ballot(valid && key[s] < pivot), be = ballot(valid && key[s] == pivot);
        if (lane == 0) {
            lcnt[s][w] = __popcll(bl);
            ecnt[s][w] = __popcll(be);
        }
    }
    __syncthreads();
    if (tid < S && int64_t(tid) * kSlice < size) {
        int l = 0, e = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            l += lcnt[tid][i];
            e += ecnt[tid][i];
        }
        const int64_t sl = row[3] - slice0 + tid;
        cnt[sl * 2 + 0] = l;
        cnt[sl * 2 + 1] = e;
    }
}

// ---- subtrees of at most kLocalMax points, one workgroup each -------------

template <int THREADS>
__device__ int local_exscan(int v, int *total)
{
    __shared__ int wt[THREADS / kWave];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const int inc = wave_inclusive_scan(v);
    if (lane == kWave - 1) wt[w] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < THREADS / kWave; ++i) {
        before += (i < w) ? wt[i] : 0;
        all += wt[i];
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

template <int PMAX, int kLocalThreads>
__global__ __launch_bounds__(kLocalThreads) void k_kd_local(
    const int64_t *__restrict__ nodes, int64_t n, int P, int leaf, int sub,
    const int32_t *__restrict__ idx_in, const float *__restrict__ vin,
    int32_t *__restrict__ idx_out, float *__restrict__ vout)
{
    __shared__ uint16_t ord[2][kLocalMax];
    __shared__ uint16_t lpre[kLocalMax];
    __shared__ uint8_t flag[kLocalMax];
    __shared__ uint8_t run_of[kLocalMax];
    __shared__ int rs[kLocalRuns], rl[kLocalRuns], rn[kLocalRuns], rd[kLocalRuns], rsi[kLocalRuns];
    __shared__ int split_list[kLocalSplit];
    // min / max slots of the splitting runs; during the sort (after the
    // split projections are chosen) the same memory exchanges keys between
    // waves
    __shared__ uint32_t ext_buf[2][kLocalSplit][PMAX];
    static_assert(sizeof(ext_buf) >= kLocalMax * sizeof(uint64_t), "key exchange fits");
    auto &emin = ext_buf[0];
    auto &emax = ext_buf[1];
    uint64_t *keys = reinterpret_cast<uint64_t *>(&ext_buf[0][0][0]);
    __shared__ int nruns_s, nsplit_s, sortlen_s;

    const int64_t *row = nodes + int64_t(blockIdx.x) * kNodeCols;
    const int64_t start = row[0];
    const int m = int(row[1]);   // <= kLocalMax, with at most kLocalRuns leaves (host plan)
    const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    constexpr int kWaves = kLocalThreads / kWave;
    int m2 = 1;
    while (m2 < m) m2 <<= 1;
    constexpr int kPer = kLocalMax / kLocalThreads;   // positions per thread
    constexpr int kSpan = kPer * kWave;   // elements per wave
    static_assert(kPer * kLocalThreads == kLocalMax, "elements: lane, register, wave bits");

    for (int i = tid; i < m; i += kLocalThreads) {
        ord[0][i] = uint16_t(i);
        run_of[i] = 0;
    }
    if (tid == 0) {
        rs[0] = 0;
        rl[0] = m;
        nruns_s = 1;
    }
    __syncthreads();
    int cur = 0;
    while (true) {
        // runs that split at this level, and where
        if (tid == 0) {
            int ns = 0;
            for (int b = 0; b < nruns_s; ++b) {
                const int len = rl[b];
                if (len > sub && ns < kLocalSplit) {
                    const int u = len > leaf ? leaf : sub;
                    const int T = (len + u - 1) / u;
                    rn[b] = ((T + 1) / 2) * u;
                    rsi[b] = ns;
                    split_list[ns++] = b;
                } else {
                    rn[b] = -1;
                    rsi[b] = -1;
                }
            }
            nsplit_s = ns;
            // every run inside one aligned block of L positions (L a power
            // of two): sorting each block sorts every run
            int maxlen = 1;
            for (int b = 0; b < nruns_s; ++b) maxlen = rl[b] > maxlen ? rl[b] : maxlen;
            int L = 1;
            while (L < maxlen) L <<= 1;
            for (int b = 0; b < nruns_s; ++b)
                if (rs[b] / L != (rs[b] + rl[b] - 1) / L) L = m2;
            sortlen_s = L < m2 ? L : m2;
        }
        __syncthreads();
        const int nsplit = nsplit_s;
        if (nsplit == 0) break;
        // extent of every projection over every splitting run.  Each wave
        // covers kSpan consecutive positions, each lane kPer consecutive ones
        // of them: when every lane's positions lie in one splitting run (or
        // past the end), which holds for runs aligned to kPer, the lane first
        // reduces its own positions in registers; otherwise the wave takes
        // its span 64 positions at a time.  Then one DPP min / max per run
        // present in the wave and projection, merged by LDS atomics.
        for (int t = tid; t < nsplit * PMAX; t += kLocalThreads) {
            emin[t / PMAX][t % PMAX] = 0xffffffffu;
            emax[t / PMAX][t % PMAX] = 0u;
        }
        __syncthreads();
        {
            auto merge = [&](int si, const uint32_t (&lo)[PMAX], const uint32_t (&hi)[PMAX]) {
                uint64_t todo = ballot(si >= 0);
                while (todo) {
                    const int src = __ffsll((unsigned long long)todo) - 1;
                    const int cur_si = __builtin_amdgcn_readlane(si, src);
                    const bool mine = si == cur_si;
                    todo &= ~ballot(mine);
#pragma unroll
                    for (int j = 0; j < PMAX; ++j) {
                        if (j < P) {
                            const uint32_t a = wave_umin_dpp(mine ? lo[j] : 0xffffffffu);
                            const uint32_t c = wave_umax_dpp(mine ? hi[j] : 0u);
                            if (lane == kWave - 1) {
                                atomicMin(&emin[cur_si][j], a);
                                atomicMax(&emax[cur_si][j], c);
                            }
                        }
                    }
                }
            };
            const int p0 = w * kSpan + lane * kPer;
            int sl[kPer];
            int lr = -1;
            bool same = true;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                sl[u] = p0 + u < m ? rsi[run_of[p0 + u]] : -1;
                if (sl[u] >= 0) {
                    if (lr < 0) lr = sl[u];
                    else if (sl[u] != lr) same = false;
                }
            }
            if (ballot(!same) == 0) {
                uint32_t lo[PMAX], hi[PMAX];
#pragma unroll
                for (int j = 0; j < PMAX; ++j) {
                    lo[j] = 0xffffffffu;
                    hi[j] = 0u;
                }
                // all of the lane's loads issued together (positions outside
                // a splitting run read a valid point and are left out)
                int ou[kPer];
                bool in[kPer];
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    in[u] = p0 + u < m && sl[u] >= 0;
                    ou[u] = in[u] ? ord[cur][p0 + u] : 0;
                }
                // four projections per round: the workgroup's gathers then
                // stay within 4 x 4 KB of the subtree's values at a time,
                // which the L2 keeps while every lane reads them
#pragma unroll
                for (int j0 = 0; j0 < PMAX; j0 += 4) {
                    float v[4][kPer];
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                        for (int u = 0; u < kPer; ++u)
                            v[jj][u] = j0 + jj < P ? vin[int64_t(j0 + jj) * n + start + ou[u]] : 0.0f;
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        const int j = j0 + jj;
                        if (j >= P) continue;
#pragma unroll
                        for (int u = 0; u < kPer; ++u) {
                            if (!in[u]) continue;
                            const uint32_t k = orderable(v[jj][u]);
                            lo[j] = min(lo[j], k);
                            hi[j] = max(hi[j], k);
                        }
                    }
                    // each round's loads complete before the next round's
                    // are issued
                    __builtin_amdgcn_s_waitcnt(0);
                }
                merge(lr, lo, hi);
            } else {
#pragma unroll 1
                for (int u = 0; u < kPer; ++u) {
                    const int i = w * kSpan + u * kWave + lane;
                    const int si = i < m ? rsi[run_of[i]] : -1;
                    uint32_t kv[PMAX];
#pragma unroll
                    for (int j = 0; j < PMAX; ++j)
                        kv[j] = (j < P && si >= 0)
                                    ? orderable(vin[int64_t(j) * n + start + ord[cur][i]])
                                    : 0u;
                    merge(si, kv, kv);
                }
            }
        }
        __syncthreads();
        for (int si = tid; si < nsplit; si += kLocalThreads) {
            int best = 0;
            float best_ext = 0.0f;
            for (int j = 0; j < P; ++j) {
                const float e = from_orderable(emax[si][j]) - from_orderable(emin[si][j]);
                if (j == 0 || e > best_ext) {
                    best = j;
                    best_ext = e;
                }
            }
            rd[split_list[si]] = best;
        }
        __syncthreads();
        // sort keys (run, key on the run's split projection, position); runs
        // that do not split sort by (run, position), i.e. stay in place.
        // Element e = w * kSpan + r * 64 + lane is register r of that lane.
        uint64_t kr[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int i = w * kSpan + r * kWave + lane;
            uint64_t key = ~uint64_t(0);
            if (i < m) {
                const int b = run_of[i];
                key = (uint64_t(b) << 44) | uint64_t(i);
                if (rn[b] >= 0) {
                    const float v = vin[int64_t(rd[b]) * n + start + ord[cur][i]];
                    key |= uint64_t(orderable(v)) << 12;
                }
            }
            kr[r] = key;
        }
        // bitonic sort of every aligned block of L keys, ascending (the last
        // merge of a block sorts it up whatever its position); elements past
        // m2 hold the largest key and stay in their own blocks.  Partners at
        // distance j < 64 are lanes of the wave, at j < kSpan registers of
        // the thread, further off other waves (through LDS).
        const int L = sortlen_s;
        for (int k = 2; k <= L; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                if (j >= kSpan) {   // uniform
#pragma unroll
                    for (int r = 0; r < kPer; ++r) keys[w * kSpan + r * kWave + lane] = kr[r];
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < kPer; ++r) {
                        const int e = w * kSpan + r * kWave + lane;
                        const uint64_t o = keys[e ^ j];
                        const bool up = k == L || (e & k) == 0;
                        const bool keep_min = ((e & j) == 0) == up;
                        kr[r] = keep_min ? (kr[r] < o ? kr[r] : o) : (kr[r] > o ? kr[r] : o);
                    }
                    __syncthreads();
                } else if (j >= kWave) {
                    const int rj = j / kWave;
#pragma unroll
                    for (int r = 0; r < kPer; ++r) {
                        if (r & rj) continue;
                        const int e = w * kSpan + r * kWave + lane;
                        const bool up = k == L || (e & k) == 0;
                        const uint64_t a = kr[r], c = kr[r | rj];
                        if ((a > c) == up) {
                            kr[r] = c;
                            kr[r | rj] = a;
                        }
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < kPer; ++r) {
                        const int e = w * kSpan + r * kWave + lane;
                        const uint64_t o = __shfl_xor(kr[r], j, kWave);
                        const bool up = k == L || (e & k) == 0;
                        const bool keep_min = ((e & j) == 0) == up;
                        kr[r] = keep_min ? (kr[r] < o ? kr[r] : o) : (kr[r] > o ? kr[r] : o);
                    }
                }
            }
        }
        // left flags by old position: sorted rank inside the run < n_left
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int rank = w * kSpan + r * kWave + lane;
            if (rank >= m) continue;
            const uint64_t key = kr[r];
            const int i = int(key & 0xfffu), b = int(key >> 44);
            flag[i] = (rn[b] >= 0 && rank - rs[b] < rn[b]) ? 1 : 0;
        }
        __syncthreads();
        {
            int c[4], sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * tid + q;
                c[q] = i < m ? flag[i] : 0;
                sum += c[q];
            }
            int tot;
            int run = local_exscan<kLocalThreads>(sum, &tot);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * tid + q;
                if (i < m) lpre[i] = uint16_t(run);
                run += c[q];
            }
        }
        __syncthreads();
        // stable partition of every splitting run
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int i = tid + q * kLocalThreads;
            if (i >= m) break;
            const int b = run_of[i];
            int np = i;
            if (rn[b] >= 0) {
                const int s = rs[b];
                const int lb = int(lpre[i]) - int(lpre[s]);
                np = flag[i] ? s + lb : s + rn[b] + (i - s - lb);
            }
            ord[cur ^ 1][np] = ord[cur][i];
        }
        __syncthreads();
        cur ^= 1;
        // next level's runs, in order of their starts
        if (tid == 0) {
            const int nr = nruns_s;
            int out = nr + nsplit;   // every splitting run becomes two
            for (int b = nr - 1; b >= 0; --b) {
                if (rn[b] >= 0) {
                    out -= 2;
                    const int s = rs[b], len = rl[b], nl = rn[b];
                    rs[out + 1] = s + nl;
                    rl[out + 1] = len - nl;
                    rs[out] = s;
                    rl[out] = nl;
                } else {
                    out -= 1;
                    rs[out] = rs[b];
                    rl[out] = rl[b];
                }
            }
            nruns_s = nr + nsplit;
        }
        __syncthreads();
        for (int b = w; b < nruns_s; b += kWaves)
            for (int i = rs[b] + lane; i < rs[b] + rl[b]; i += kWave) run_of[i] = uint8_t(b);
        __syncthreads();
    }
    // the subtree's points in their final order; the values move four
    // projections at a time, as the extents read them
    int64_t of[kPer];
    bool pin[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = tid + q * kLocalThreads;
        pin[q] = p < m;
        of[q] = start + (pin[q] ? ord[cur][p] : 0);
        if (pin[q]) idx_out[start + p] = idx_in ? idx_in[of[q]] : int32_t(of[q]);
    }
    if (vout) {
#pragma unroll
        for (int j0 = 0; j0 < PMAX; j0 += 4) {
            float v[4][kPer];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int q = 0; q < kPer; ++q)
                    v[jj][q] = j0 + jj < P ? vin[int64_t(j0 + jj) * n + of[q]] : 0.0f;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int q = 0; q < kPer; ++q)
                    if (j0 + jj < P && pin[q])
                        vout[int64_t(j0 + jj) * n + start + tid + q * kLocalThreads] = v[jj][q];
        }
    }
}

// ---- subtrees of at most kSubMax points, one workgroup each ----------------
// For runs that start at multiples of 64 points: a chunk of 64 positions then
// lies in one run, and a wave holds two chunks, a lane one point of each.  The
// points' keys stay in LDS where they were loaded (16 projections x 2,048
// points: 128 KB, one workgroup per CU); the order is an array of 16-bit
// indices.  Per level: chunk extents by wave minima, the run's split
// projection from them; a histogram of 256 equal steps over the run's range on
// it, in floats (a monotone map, so that any rounding only moves points
// between bins the same way for all), whose bin holding the pivot's rank
// leaves a handful of points that one wave ranks; more than 64 of them take a
// second histogram over the bin, and if they remain (ties, infinite ranges) a
// radix descent (the Gaussians of an 800 x 800 10-D image, where far ones
// squeeze the rest into a few bins: 206 -> 66 us by the second histogram).
// Stable partition by (key, position) against the pivot's.  Bound by its
// vector operations and the chain of these steps: 36 us for one subtree, 100
// for 512 (two rounds of the CUs; 10-D, 2^20 queries; 107 with a reduction per
// chunk instead of one for a wave's two), where the sorts of k_kd_local
// took 58 to 100 and, with the level above that they left, 300.
__global__ __launch_bounds__(kSubThreads) void k_kd_subtree(
    const int64_t *__restrict__ nodes, int64_t n, int P, int leaf,
    const int32_t *__restrict__ idx_in, const float *__restrict__ vin,
    int32_t *__restrict__ idx_out, float *__restrict__ vout)
{
    constexpr int kRuns = kSubChunks;           // at most one run per chunk
    constexpr int kSplits = kSubChunks / 2;     // a run that splits has two chunks
    constexpr int kHBins = 256;
    __shared__ uint32_t val[kSubProj][kSubMax];
    __shared__ uint16_t ord[2][kSubMax];
    // histograms of the splitting runs; then the pivot bin's points of each
    __shared__ __attribute__((aligned(16))) uint32_t hist[kSplits][kHBins];
    __shared__ uint32_t cext[kSubChunks][2 * kSubProj];   // minima, maxima
    __shared__ int rs[2][kRuns], rl[2][kRuns], rn[2][kRuns], rsi[2][kRuns];
    __shared__ int nruns[2], nsplit[2];
    __shared__ int srun[2][kSplits];                      // a splitting run's index
    __shared__ int sbin[kSplits], srank[kSplits], scnt[kSplits], lcnt[kSplits];
    __shared__ int sdim[kSplits], sbin2[kSplits];   // sbin2: -1 without a second histogram
    __shared__ int s_again;
    __shared__ uint32_t s_starts;
    __shared__ uint64_t spiv[kSplits];
    __shared__ int ccnt[kSubChunks];
    __shared__ int crun[2][kSubChunks];
    const int64_t *row = nodes + int64_t(blockIdx.x) * kNodeCols;
    const int64_t start = row[0];
    const int m = int(row[1]);
    const int tid = threadIdx.x, w = uniform(tid / kWave), lane = lane_id();
    constexpr int kPer = kSubMax / kSubThreads;   // chunks per wave
    static_assert(kPer == 2, "two chunks per wave");

    // a run of length len: n_left when it splits, -1 when it does not
    auto split_of = [&](int len) {
        if (len <= kWave) return -1;
        const int u = len > leaf ? leaf : kWave;
        return ((len + u - 1) / u + 1) / 2 * u;
    };
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kSubThreads;
#pragma unroll
        for (int j = 0; j < kSubProj; ++j)
            if (j < P && i < m) val[j][i] = orderable(vin[int64_t(j) * n + start + i]);
        ord[0][i] = uint16_t(i);
    }
    for (int b = tid; b < kSplits * kHBins; b += kSubThreads) (&hist[0][0])[b] = 0;
    // chunks past the end stay in run 0, without points
    if (tid < 2 * kSubChunks) crun[tid / kSubChunks][tid % kSubChunks] = 0;
    if (tid == 0) {
        rs[0][0] = 0;
        rl[0][0] = m;
        rn[0][0] = split_of(m);
        rsi[0][0] = rn[0][0] >= 0 ? 0 : -1;
        srun[0][0] = 0;
        nruns[0] = 1;
        nsplit[0] = rn[0][0] >= 0 ? 1 : 0;
    }
    __syncthreads();
    int cur = 0;
    while (true) {
        const int ns = nsplit[cur];
        if (ns == 0) break;   // uniform
        int o[kPer], run[kPer], si[kPer];
        bool in[kPer];
        // the chunks' extents (lanes past the end repeat the last point, which
        // is in the same run; keys of projections past P are not looked at)
        bool have[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int c = kPer * w + u, pos = c * kWave + lane;
            run[u] = uniform(crun[cur][c]);
            si[u] = uniform(rsi[cur][run[u]]);
            in[u] = pos < m;
            o[u] = ord[cur][in[u] ? pos : m - 1];
            have[u] = si[u] >= 0 && c * kWave < m;   // uniform
        }
        {
            auto put = [&](uint32_t (&lo)[kSubProj], uint32_t (&hi)[kSubProj], int c) {
                wave_umin_scatter<kSubProj>(lo);
                wave_umin_scatter<kSubProj, true>(hi);
                if ((lane & 15) == 15)
#pragma unroll
                    for (int e = 0; e < kSubProj / 4; ++e) {
                        cext[c][(lane >> 4) * (kSubProj / 4) + e] = lo[e];
                        cext[c][kSubProj + (lane >> 4) * (kSubProj / 4) + e] = hi[e];
                    }
            };
            uint32_t lo[kSubProj], hi[kSubProj];
            if (have[0] && have[1] && run[0] == run[1]) {   // one reduction for both
#pragma unroll
                for (int j = 0; j < kSubProj; ++j) {
                    const uint32_t a = val[j][o[0]], b = val[j][o[1]];
                    lo[j] = min(a, b);
                    hi[j] = max(a, b);
                }
                if (lane < 2 * kSubProj)
                    cext[kPer * w + 1][lane] = lane < kSubProj ? 0xffffffffu : 0u;
                put(lo, hi, kPer * w);
            } else {
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    if (!have[u]) continue;
#pragma unroll
                    for (int j = 0; j < kSubProj; ++j) lo[j] = hi[j] = val[j][o[u]];
                    put(lo, hi, kPer * w + u);
                }
            }
        }
        if (tid == 0) s_again = 0;
        __syncthreads();
        // split projections; histograms over the runs' ranges on them
        uint32_t key[kPer];
        int bin[kPer], bin2[kPer];
        float t[kPer];
        int dim = 0;
        float vlo = 0.0f, scale = 0.0f;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            key[u] = 0;
            bin[u] = bin2[u] = -1;
            if (!have[u]) continue;   // uniform
            if (u == 0 || !have[0] || run[u] != run[0]) {
                const int c0 = rs[cur][run[u]] / kWave;
                const int c1 = (rs[cur][run[u]] + rl[cur][run[u]] + kWave - 1) / kWave;
                // lane: projection lane mod 16, every fourth chunk (past the
                // last, it again)
                const int j = lane & 15;
                uint32_t lo = 0xffffffffu, hi = 0u;
                for (int b = c0 + (lane >> 4); b < c1 + (lane >> 4); b += 16) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int c = min(b + 4 * e, c1 - 1);
                        lo = min(lo, cext[c][j]);
                        hi = max(hi, cext[c][kSubProj + j]);
                    }
                }
                lo = rows_pick<false>(lo);
                hi = rows_pick<true>(hi);
                // the largest extent, the first on ties; one that is not a
                // number counts only in the first place
                const float flo = from_orderable(lo);
                const float e = from_orderable(hi) - flo;
                uint32_t ek = e == e ? orderable(e) : (j == 0 ? 0xffffffffu : 0u);
                if (j >= P) ek = 0u;
                const uint32_t best = __builtin_amdgcn_readlane(wave_umax_dpp(ek), kWave - 1);
                const int l = __builtin_ctzll(ballot(ek == best));
                dim = l & 15;
                vlo = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(flo), l));
                const float ext = __uint_as_float(
                    __builtin_amdgcn_readlane(__float_as_uint(e), l));
                scale = (ext > 0.0f && ext < INFINITY) ? float(kHBins) / ext : 0.0f;
                if (!(scale < INFINITY)) scale = 0.0f;
                if (lane == 0) sdim[si[u]] = dim;
            }
            key[u] = val[dim][o[u]];
            t[u] = (from_orderable(key[u]) - vlo) * scale;
            if (in[u]) {
                bin[u] = t[u] > 0.0f ? min(int(t[u]), kHBins - 1) : 0;   // not a number: 0
                atomicAdd(&hist[si[u]][bin[u]], 1u);
            }
        }
        __syncthreads();
        // the bin of run w's histogram that holds rank `want`
        auto pick_bin = [&](int want, int *out) {
            const uint4 c4 = *reinterpret_cast<const uint4 *>(&hist[w][4 * lane]);
            const int c[4] = {int(c4.x), int(c4.y), int(c4.z), int(c4.w)};
            const int sum = c[0] + c[1] + c[2] + c[3];
            int cum = wave_inclusive_scan(sum) - sum;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (want >= cum && want < cum + c[i]) {
                    out[w] = 4 * lane + i;
                    srank[w] = want - cum;
                    scnt[w] = c[i];
                    if (out == sbin && c[i] > kWave) s_again = 1;
                }
                cum += c[i];
            }
        };
        // the bin of each splitting run's pivot, a wave per run; the run
        // tables of the next level, wave 15 (runs in order of their starts)
        if (w < ns) {
            pick_bin(rn[cur][srun[cur][w]], sbin);
            if (lane == 0) {
                lcnt[w] = 0;
                sbin2[w] = -1;
            }
        }
        if (w == kSubThreads / kWave - 1) {
            const int nr = nruns[cur];
            const bool has = lane < nr;
            const int s0 = has ? rs[cur][lane] : 0, len = has ? rl[cur][lane] : 0;
            const int nl = has ? rn[cur][lane] : -1;
            const uint64_t sp = ballot(nl >= 0);
            const int at = lane + __popcll(sp & lanemask_lt());
            const int l0 = nl >= 0 ? nl : len, l1 = len - l0;
            const int n0 = split_of(l0), n1 = split_of(l1);
            const uint64_t b0 = ballot(has && n0 >= 0), b1 = ballot(has && nl >= 0 && n1 >= 0);
            const int k0 = __popcll(b0 & lanemask_lt()) + __popcll(b1 & lanemask_lt());
            const int nx = cur ^ 1;
            if (has) {
                rs[nx][at] = s0;
                rl[nx][at] = l0;
                rn[nx][at] = n0;
                rsi[nx][at] = n0 >= 0 ? k0 : -1;
                if (n0 >= 0) srun[nx][k0] = at;
                if (nl >= 0) {
                    const int k1 = k0 + (n0 >= 0 ? 1 : 0);
                    rs[nx][at + 1] = s0 + l0;
                    rl[nx][at + 1] = l1;
                    rn[nx][at + 1] = n1;
                    rsi[nx][at + 1] = n1 >= 0 ? k1 : -1;
                    if (n1 >= 0) srun[nx][k1] = at + 1;
                }
            }
            // a chunk's run: the runs that start at or before it
            if (lane == 0) s_starts = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (has)
                atomicOr(&s_starts, 1u << (s0 / kWave) | (nl >= 0 ? 1u << ((s0 + l0) / kWave) : 0u));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const uint32_t starts = s_starts;
            if (lane < kSubChunks)
                crun[nx][lane] = __popc(starts & (0xffffffffu >> (31 - lane))) - 1;
            if (lane == 0) {
                nruns[nx] = nr + __popcll(sp);
                nsplit[nx] = __popcll(b0) + __popcll(b1);
            }
        }
        __syncthreads();
        // bins of more points than a wave ranks: a second histogram over the
        // bin's own range (the same map, of what it left)
        if (s_again) {   // uniform
            if (w < ns && scnt[w] > kWave) {
                *reinterpret_cast<uint4 *>(&hist[w][4 * lane]) = make_uint4(0, 0, 0, 0);
                if (lane == 0) sbin2[w] = 0;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                if (bin[u] >= 0 && sbin2[si[u]] >= 0 && bin[u] == sbin[si[u]]) {
                    const float f = (t[u] - float(bin[u])) * float(kHBins);
                    bin2[u] = f > 0.0f ? min(int(f), kHBins - 1) : 0;
                    atomicAdd(&hist[si[u]][bin2[u]], 1u);
                }
            }
            __syncthreads();
            if (w < ns && sbin2[w] >= 0) pick_bin(srank[w], sbin2);
            __syncthreads();
        }
        // that bin's points, listed over the run's histogram
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (bin[u] >= 0 && bin[u] == sbin[si[u]] && bin2[u] == sbin2[si[u]]) {
                const int slot = atomicAdd(&lcnt[si[u]], 1);
                if (slot < kWave)
                    reinterpret_cast<uint64_t *>(hist[si[u]])[slot] =
                        uint64_t(key[u]) << 16 | uint32_t((kPer * w + u) * kWave + lane);
            }
        }
        __syncthreads();
        // each run's pivot (key, position): the first point that goes right
        if (w < ns) {
            const int cnt = scnt[w];
            uint64_t piv = 0;
            if (cnt <= kWave) {
                const uint64_t e =
                    lane < cnt ? reinterpret_cast<const uint64_t *>(hist[w])[lane] : ~uint64_t(0);
                int rank = 0;
                for (int i = 0; i < cnt; ++i) {
                    const uint64_t x =
                        uint64_t(uint32_t(__builtin_amdgcn_readlane(uint32_t(e >> 32), i))) << 32 |
                        uint32_t(__builtin_amdgcn_readlane(uint32_t(e), i));
                    rank += x < e;
                }
                const int l = __builtin_ctzll(ballot(lane < cnt && rank == srank[w]) |
                                              uint64_t(1) << 63);
                piv = uint64_t(uint32_t(__builtin_amdgcn_readlane(uint32_t(e >> 32), l))) << 32 |
                      uint32_t(__builtin_amdgcn_readlane(uint32_t(e), l));
            } else {
                // bit by bit over the run's keys, then the position among
                // the keys equal to the pivot's
                const int r = srun[cur][w], d = sdim[w];
                const int s0 = rs[cur][r], s1 = s0 + rl[cur][r];
                uint32_t pre = 0;
                int rank = rn[cur][r];
                for (int bit = 31; bit >= 0; --bit) {
                    int zeros = 0;
                    for (int b = s0; b < s1; b += kWave) {
                        const uint32_t k = b + lane < s1 ? val[d][ord[cur][b + lane]] : 0u;
                        const bool z = b + lane < s1 && (k >> bit) == (pre << 1);
                        zeros += __popcll(ballot(z));
                    }
                    pre <<= 1;
                    if (rank >= zeros) {
                        rank -= zeros;
                        pre |= 1u;
                    }
                }
                int at = s0;
                for (int b = s0; b < s1; b += kWave) {
                    const bool q = b + lane < s1 && val[d][ord[cur][b + lane]] == pre;
                    const uint64_t bq = ballot(q);
                    const int c = __popcll(bq);
                    if (rank >= 0 && rank < c) {
                        const uint64_t hit =
                            ballot(q && __popcll(bq & lanemask_lt()) == rank);
                        at = b + __builtin_ctzll(hit);
                    }
                    rank -= c;
                }
                piv = uint64_t(pre) << 16 | uint32_t(at);
            }
            if (lane == 0) spiv[w] = piv;
            // clean for the next level
            *reinterpret_cast<uint4 *>(&hist[w][4 * lane]) = make_uint4(0, 0, 0, 0);
        }
        __syncthreads();
        // stable partition of every splitting run
        uint64_t bl[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int c = kPer * w + u;
            const uint64_t mine = uint64_t(key[u]) << 16 | uint32_t(c * kWave + lane);
            bl[u] = have[u] ? ballot(in[u] && mine < spiv[si[u]]) : 0;
            if (lane == 0) ccnt[c] = __popcll(bl[u]);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int c = kPer * w + u, pos = c * kWave + lane;
            int np = pos;
            if (have[u]) {   // uniform
                const int s0 = rs[cur][run[u]];
                const int v = lane >= s0 / kWave && lane < c ? ccnt[lane & (kSubChunks - 1)] : 0;
                const int before = wave_last(wave_inclusive_scan(v));
                const int lr = before + __popcll(bl[u] & lanemask_lt());
                np = (bl[u] >> lane) & 1 ? s0 + lr : s0 + rn[cur][run[u]] + (pos - s0 - lr);
            }
            if (in[u] && np < m) ord[cur ^ 1][np] = uint16_t(o[u]);
        }
        __syncthreads();
        cur ^= 1;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kSubThreads;
        if (i >= m) break;
        const int o = ord[cur][i];
        idx_out[start + i] = idx_in ? idx_in[start + o] : int32_t(start + o);
        if (vout) {
#pragma unroll
            for (int j = 0; j < kSubProj; ++j)
                if (j < P) vout[int64_t(j) * n + start + i] = from_orderable(val[j][o]);
        }
    }
}

inline unsigned nb(int64_t n, int per) { return unsigned((n + per - 1) / per); }

// Leaves of a run of `size` points (the split rule above).
int64_t count_leaves(int64_t size, int leaf, int sub, std::map<int64_t, int64_t> &memo)
{
    if (size <= sub) return 1;
    auto it = memo.find(size);
    if (it != memo.end()) return it->second;
    const int64_t u = size > leaf ? leaf : sub;
    const int64_t T = (size + u - 1) / u, nl = ((T + 1) / 2) * u;
    const int64_t r = count_leaves(nl, leaf, sub, memo) + count_leaves(size - nl, leaf, sub, memo);
    memo[size] = r;
    return r;
}

}  // namespace

bool kd_plan(KdPlan &pl, int64_t n, int leaf, int sub, int P)
{
    // subtrees in k_kd_subtree: every run then starts at a multiple of 64
    const bool subtree = P <= kSubProj && sub == kWave && leaf % kWave == 0;
    if (pl.n == n && pl.leaf == leaf && pl.sub == sub && pl.subtree == subtree) return true;
    pl.n = n;
    pl.leaf = leaf;
    pl.sub = sub;
    pl.subtree = subtree;
    pl.levels.clear();
    pl.local = KdLevel{};
    pl.has_local = false;
    std::vector<int64_t> nodes, slices;
    std::vector<std::pair<int64_t, int64_t>> cur;
    if (n > 0) cur.push_back({0, n});
    int64_t max_nodes = 0, max_slices = 0, hist_nodes = 0;
    std::map<int64_t, int64_t> memo;
    while (true) {
        bool any = false;
        int64_t biggest = 0, most_leaves = 0;
        for (auto &nd : cur) {
            any |= nd.second > sub;
            biggest = std::max(biggest, nd.second);
            if (!subtree && nd.second <= kLocalMax)
                most_leaves = std::max(most_leaves, count_leaves(nd.second, leaf, sub, memo));
        }
        if (!any) break;
        if (subtree ? biggest <= kSubMax : biggest <= kLocalMax && most_leaves <= kLocalRuns) {
            // the rest of every subtree in one workgroup each
            pl.local.node0 = int64_t(nodes.size()) / kNodeCols;
            for (auto &nd : cur)
                nodes.insert(nodes.end(), {nd.first, nd.second, -1, 0, 0, -1, 0, 0});
            pl.local.node1 = int64_t(nodes.size()) / kNodeCols;
            pl.has_local = true;
            break;
        }
        KdLevel lv;
        lv.biggest = biggest;
        const bool sliced = biggest > kNodeMax;
        lv.node0 = int64_t(nodes.size()) / kNodeCols;
        lv.slice0 = int64_t(slices.size()) / kSliceCols;
        std::vector<std::pair<int64_t, int64_t>> next;
        for (auto &nd : cur) {
            const int64_t st = nd.first, sz = nd.second;
            const int64_t node_id = int64_t(nodes.size()) / kNodeCols;
            int64_t nl = -1, child = -1;
            if (sz > sub) {
                const int64_t u = sz > leaf ? leaf : sub;
                const int64_t T = (sz + u - 1) / u;
                nl = ((T + 1) / 2) * u;
                child = int64_t(next.size());
                next.push_back({st, nl});
                next.push_back({st + nl, sz - nl});
            } else {
                next.push_back({st, sz});
            }
            const int64_t sb = int64_t(slices.size()) / kSliceCols;
            for (int64_t s = st; s < st + sz; s += kSlice) {
                slices.push_back(s);
                slices.push_back(std::min<int64_t>(kSlice, st + sz - s));
                slices.push_back(node_id);
            }
            const int64_t se = int64_t(slices.size()) / kSliceCols;
            nodes.insert(nodes.end(), {st, sz, nl, sb, se, child, 0, 0});
        }
        lv.node1 = int64_t(nodes.size()) / kNodeCols;
        lv.slice1 = int64_t(slices.size()) / kSliceCols;
        // the histogram slices of the level's nodes, after its slices
        lv.hslice0 = lv.slice1;
        for (int64_t nd = lv.node0; nd < lv.node1; ++nd) {
            const int64_t st = nodes[nd * kNodeCols + 0], sz = nodes[nd * kNodeCols + 1];
            nodes[nd * kNodeCols + 6] = int64_t(slices.size()) / kSliceCols;
            for (int64_t s = st; sliced && s < st + sz; s += kHistSlice) {
                slices.push_back(s);
                slices.push_back(std::min<int64_t>(kHistSlice, st + sz - s));
                slices.push_back(nd);
            }
            nodes[nd * kNodeCols + 7] = int64_t(slices.size()) / kSliceCols;
        }
        lv.hslice1 = int64_t(slices.size()) / kSliceCols;
        max_nodes = std::max(max_nodes, lv.node1 - lv.node0);
        if (sliced) hist_nodes = std::max(hist_nodes, lv.node1 - lv.node0);
        max_slices = std::max(max_slices, lv.slice1 - lv.slice0);
        pl.levels.push_back(lv);
        cur.swap(next);
    }
    // the last upper level's children are not upper-level nodes: no slots
    if (!pl.levels.empty()) {
        const KdLevel &last = pl.levels.back();
        for (int64_t i = last.node0; i < last.node1; ++i) nodes[i * kNodeCols + 5] = -1;
    }
    pl.max_nodes = max_nodes;
    pl.max_slices = max_slices;
    pl.hist_nodes = hist_nodes;
    if (!pl.node_tab.ensure(sizeof(int64_t) * std::max<size_t>(nodes.size(), 1)) ||
        !pl.slice_tab.ensure(sizeof(int64_t) * std::max<size_t>(slices.size(), 1))) {
        pl.n = -1;
        return false;
    }
    if ((!nodes.empty() && hipMemcpy(pl.node_tab.p, nodes.data(), sizeof(int64_t) * nodes.size(),
                                     hipMemcpyHostToDevice) != hipSuccess) ||
        (!slices.empty() && hipMemcpy(pl.slice_tab.p, slices.data(),
                                      sizeof(int64_t) * slices.size(),
                                      hipMemcpyHostToDevice) != hipSuccess)) {
        pl.n = -1;
        return false;
    }
    return true;
}

bool kd_reserve(KdWork &w, const KdPlan &pl, int64_t n, int P)
{
    const int64_t nn = std::max<int64_t>(n, 1);
    const int64_t ms = std::max<int64_t>(pl.max_slices, 1), mn = std::max<int64_t>(pl.max_nodes, 1);
    const int64_t mh = std::max<int64_t>(pl.hist_nodes, 1);
    bool ok = true;
    ok &= w.idx[0].ensure(sizeof(int32_t) * nn);
    ok &= w.idx[1].ensure(sizeof(int32_t) * nn);
    ok &= w.val[0].ensure(sizeof(float) * P * nn);
    ok &= w.val[1].ensure(sizeof(float) * P * nn);
    ok &= w.ext[0].ensure(sizeof(uint32_t) * 2 * P * mn * kExtRep);
    ok &= w.ext[1].ensure(sizeof(uint32_t) * 2 * P * mn * kExtRep);
    ok &= w.hist.ensure(sizeof(int32_t) * 3 * kBins * mh);
    ok &= w.cnt.ensure(sizeof(int64_t) * 2 * ms);
    ok &= w.dim.ensure(sizeof(int32_t) * mn);
    ok &= w.prefix.ensure(sizeof(uint32_t) * 3 * mn);
    ok &= w.rank.ensure(sizeof(int64_t) * 3 * mn);
    return ok;
}

hipError_t launch_kd_root(const KdPlan &pl, KdWork &w, int P, int64_t nparts, const void *part,
                          hipStream_t s)
{
    if (pl.levels.empty()) return hipSuccess;   // one subtree: it finds its extents itself
    const int64_t mn = std::max<int64_t>(pl.max_nodes, 1);
    if (w.ext[0].cap < sizeof(uint32_t) * 2 * P * size_t(mn) * kExtRep ||
        w.hist.cap < sizeof(int32_t) * 3 * kBins * size_t(pl.hist_nodes))
        return hipErrorInvalidValue;
    k_kd_root<<<dim3(unsigned(P), pl.hist_nodes > 0 ? 17 : 1), kThreads, 0, s>>>(
        nparts, P, static_cast<const uint32_t *>(part), w.ext[0].as<uint32_t>(), mn,
        w.hist.as<int32_t>(), 3 * kBins * pl.hist_nodes);
    return hipGetLastError();
}

hipError_t kd_start(KdRun &r, const KdPlan &pl, KdWork &w, int P, const float *vals, int64_t n,
                    int32_t *perm, float *vals_sorted, hipStream_t s)
{
    r = KdRun{};
    r.pl = &pl;
    r.w = &w;
    r.P = P;
    r.vals = vals;
    r.n = n;
    r.perm = perm;
    r.vals_sorted = vals_sorted;
    r.s = s;
    r.vin = vals;
    r.done = n == 0;
    if (n == 0) return hipSuccess;
    const int64_t mn = std::max<int64_t>(pl.max_nodes, 1), ms = std::max<int64_t>(pl.max_slices, 1);
    const int64_t mh = std::max<int64_t>(pl.hist_nodes, 1);
    if (pl.n != n || (pl.levels.empty() && !pl.has_local) || P < 1 || P > 32 ||
        w.idx[0].cap < sizeof(int32_t) * size_t(n) || w.idx[1].cap < sizeof(int32_t) * size_t(n) ||
        w.val[0].cap < sizeof(float) * P * size_t(n) ||
        w.val[1].cap < sizeof(float) * P * size_t(n) ||
        w.ext[0].cap < sizeof(uint32_t) * 2 * P * size_t(mn) * kExtRep ||
        w.ext[1].cap < sizeof(uint32_t) * 2 * P * size_t(mn) * kExtRep ||
        w.hist.cap < sizeof(int32_t) * 3 * kBins * size_t(mh) ||
        w.cnt.cap < sizeof(int64_t) * 2 * size_t(ms) || w.dim.cap < sizeof(int32_t) * size_t(mn) ||
        w.prefix.cap < sizeof(uint32_t) * 3 * size_t(mn) ||
        w.rank.cap < sizeof(int64_t) * 3 * size_t(mn) || (pl.subtree && P > kSubProj)) {
        r.done = true;
        return hipErrorInvalidValue;
    }
    return hipSuccess;
}

hipError_t kd_step(KdRun &r)
{
    if (r.done) return hipSuccess;
    const KdPlan &pl = *r.pl;
    KdWork &w = *r.w;
    const int P = r.P;
    const int64_t n = r.n;
    const hipStream_t s = r.s;
    const int64_t mn = std::max<int64_t>(pl.max_nodes, 1);
    const int64_t mh = std::max<int64_t>(pl.hist_nodes, 1);
    const int64_t *nodes = pl.node_tab.as<int64_t>();
    const int64_t *slices = pl.slice_tab.as<int64_t>();
    int32_t *hist = w.hist.as<int32_t>();
    int32_t *dim = w.dim.as<int32_t>();
    uint32_t *prefix = w.prefix.as<uint32_t>();
    int64_t *rank = w.rank.as<int64_t>();
    int64_t *cnt = w.cnt.as<int64_t>();
    const size_t nlev = pl.levels.size();
    const size_t phase = r.phase++;
    if (phase < nlev) {   // an upper level
        const size_t li = phase;
        const KdLevel &lv = pl.levels[li];
        const int64_t *nt = nodes + lv.node0 * kNodeCols;
        const int64_t *st = slices + lv.slice0 * kSliceCols;
        uint32_t *ext = w.ext[li & 1].as<uint32_t>();
        uint32_t *ext_next = (li + 1 < nlev) ? w.ext[(li + 1) & 1].as<uint32_t>() : nullptr;
        int32_t *idx_out = w.idx[r.cur].as<int32_t>();
        float *vout = w.val[r.cur].as<float>();
        const int64_t ns = lv.slice1 - lv.slice0;
        const int64_t *hst = slices + lv.hslice0 * kSliceCols;
        const unsigned nhs = unsigned(lv.hslice1 - lv.hslice0);
        const bool one = lv.biggest <= kNodeMax;   // the selection in one launch
        if (one) {
            auto go = [&](auto kern) {
                const int64_t nn = lv.node1 - lv.node0, most = max_grid(kNodeThreads);
                for (int64_t b = 0; b < nn; b += most)
                    kern<<<unsigned(std::min(nn - b, most)), kNodeThreads, 0, s>>>(
                        b, nt, lv.slice0, n, P, r.vin, ext, mn, ext_next, dim, prefix + 2 * mn,
                        rank + 2 * mn, cnt);
            };
            if (lv.biggest <= 4 * kNodeThreads) go(k_kd_select<4>);
            else go(k_kd_select<16>);
        }
        for (int rd = 0; !one && rd < 3; ++rd)
            k_kd_hist<<<nhs, kHistThreads, 0, s>>>(nt, hst, lv.node0, lv.hslice0, mn, mh, n, P, rd,
                                                   r.vin, ext, ext_next, dim, prefix, rank, hist);
        if (!one) k_kd_count<<<unsigned(ns), kThreads, 0, s>>>(nt, st, lv.node0, lv.slice0, mn, mh, n, r.vin,
                                                     dim, prefix, rank, hist, cnt);
        if (P <= 16)
            k_kd_scatter<16><<<unsigned(ns), kThreads, 0, s>>>(
                nt, st, lv.node0, lv.slice0, n, P, r.idx_in, r.vin, dim, prefix + 2 * mn,
                rank + 2 * mn, cnt, idx_out, vout, ext_next, one ? nullptr : hist, mn, mh);
        else
            k_kd_scatter<32><<<unsigned(ns), kThreads, 0, s>>>(
                nt, st, lv.node0, lv.slice0, n, P, r.idx_in, r.vin, dim, prefix + 2 * mn,
                rank + 2 * mn, cnt, idx_out, vout, ext_next, one ? nullptr : hist, mn, mh);
        r.idx_in = idx_out;
        r.vin = vout;
        r.cur ^= 1;
        return hipGetLastError();
    }
    // the subtrees, or the order out as it stands
    r.done = true;
    if (pl.has_local) {
        const int64_t *nt = nodes + pl.local.node0 * kNodeCols;
        const unsigned nl = unsigned(pl.local.node1 - pl.local.node0);
        if (pl.subtree) {
            k_kd_subtree<<<nl, kSubThreads, 0, s>>>(nt, n, P, pl.leaf, r.idx_in, r.vin, r.perm,
                                                    r.vals_sorted);
            return hipGetLastError();
        }
        // 512 threads per subtree when every subtree's workgroup is resident
        // at once with them (three per CU), else 256 (seven per CU)
        auto go = [&](auto kern, int threads) {
            kern<<<nl, threads, 0, s>>>(nt, n, P, pl.leaf, pl.sub, r.idx_in, r.vin, r.perm,
                                        r.vals_sorted);
        };
        const bool wide = nl <= kWideLocalBlocks;
        if (P <= 16)
            wide ? go(k_kd_local<16, 512>, 512) : go(k_kd_local<16, 256>, 256);
        else
            wide ? go(k_kd_local<32, 512>, 512) : go(k_kd_local<32, 256>, 256);
        return hipGetLastError();
    }
    hipError_t e =
        hipMemcpyAsync(r.perm, r.idx_in, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess && r.vals_sorted)
        e = hipMemcpyAsync(r.vals_sorted, r.vin, sizeof(float) * P * n, hipMemcpyDeviceToDevice,
                           s);
    return e;
}

}  // namespace ngd
