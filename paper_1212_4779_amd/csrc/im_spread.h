// im_spread.h -- spread evaluator: f(T) = sum_r |R_r(T)| (the snapshot estimator
// of Sec. 3.1, times R) for the prefixes of a seed sequence, on snapshots of
// any seed, so a seed set can be scored on snapshots independent of those that
// chose it (the evaluation protocol of Sec. 5.2).
//
// One workgroup takes one snapshot at a time and covers the seeds in order:
// each seed's search leaves out what the earlier ones reached, so the nodes
// it adds are its marginal gain. Only the arcs of reached nodes have their
// coin drawn, where drawing whole masks first costs m draws per snapshot and a
// round trip through memory, and the snapshots are independent, where one
// workgroup per word of 64 left a device of 256 CUs with R / 64 of them. A
// level costs a row load, a 16-byte record per arc and the draw (about 20
// integer operations); with thousands of snapshots the draws are the bound,
// with a few hundred the levels. 50 seeds on 15,000 nodes, 59,000 arcs: R =
// 20,000 9.0 -> 2.06 ms, R = 300 3.7 -> 0.53 ms; on 10^6 nodes, 10^7 arcs, R =
// 256: 11.7 -> 1.4 ms.
#pragma once

#include "im_bfs.h"

// what a draw needs of an arc: its key, floor(p 2^32) - 1 and its head
// (IM_EMPTY: the arc is never live)
struct __align__(16) ArcCoin {
    uint64_t key;
    uint32_t last, head;
};

__device__ __forceinline__ ArcCoin arc_coin(const uint32_t *col, const float *prob, uint64_t seed, uint64_t e)
{
    const uint64_t thr = (uint64_t)((double)prob[e] * 4294967296.0);   // 0 .. 2^32
    ArcCoin c;
    c.key = sm64_finalise(seed + (e + 1ull) * IM_GOLDEN);
    c.last = (uint32_t)(thr - 1ull);
    c.head = thr ? col[e] : IM_EMPTY;
    return c;
}

__global__ __launch_bounds__(256) void k_arc_coins(const uint32_t *col, const float *prob, uint64_t m,
                                                   uint64_t seed, ArcCoin *coin)
{
    for (uint64_t e = blockIdx.x * 256ull + threadIdx.x; e < m; e += (uint64_t)gridDim.x * 256u)
        coin[e] = arc_coin(col, prob, seed, e);
}

struct SpreadArgs {
    const uint32_t *row;
    const ArcCoin *coin;         // a record per arc; without (RECORDS false) it is made for each draw
    const uint32_t *col;
    const float *prob;
    uint64_t seed;
    uint32_t n, R;
    const uint32_t *S;
    uint32_t nS, group;          // seeds per search
    uint32_t *queue;             // [workgroups][n]
    uint32_t *bits;              // [workgroups][ceil(n / 32)], zero at rest; LDS is used if null
    unsigned long long *marg;    // [ceil(nS / group)] (accumulated over snapshots) or nullptr
    bool sum_here;               // ... per workgroup first, in 32 bits: at most SPR_ACC seeds,
                                 // and its snapshots' nodes below 2^32 in all
    uint32_t *per_snapshot;      // [R] or nullptr
};

constexpr int SPR_Q = 1024;      // queue entries kept in LDS as well
constexpr int SPR_ACC = 256;     // marginals added up per workgroup up to this many seeds
constexpr int SPR_U = 4;         // arcs in flight per lane

template <int NT, bool RECORDS>
__global__ __launch_bounds__(NT) void k_spread(SpreadArgs a)
{
    extern __shared__ uint32_t lds_bits[];   // [ceil(n / 32)] unless a.bits
    __shared__ uint32_t q[SPR_Q], ex[NT], rs[NT], wsum[NT / 64 + 1], cnt;
    __shared__ uint32_t acc[SPR_ACC];
    const uint32_t tid = threadIdx.x, words = (a.n + 31) / 32;
    uint32_t *bits = a.bits ? a.bits + (uint64_t)blockIdx.x * words : lds_bits;
    uint32_t *queue = a.queue + (uint64_t)blockIdx.x * a.n;
    if (!a.bits)
        for (uint32_t i = tid; i < words; i += NT) bits[i] = 0;
    const bool sum_here = a.marg && a.sum_here;
    for (uint32_t i = tid; i < (uint32_t)SPR_ACC; i += NT) acc[i] = 0;
    auto visit = [&](uint32_t v) {
        const uint32_t bit = 1u << (v & 31u);
        if (atomicOr(&bits[v >> 5], bit) & bit) return;
        const uint32_t p = atomicAdd(&cnt, 1u);
        if (p < (uint32_t)SPR_Q) q[p] = v;
        else queue[p] = v;
    };
    auto entry = [&](uint32_t i) { return i < (uint32_t)SPR_Q ? q[i] : queue[i]; };
    for (uint32_t r = blockIdx.x; r < a.R; r += gridDim.x) {
        const uint64_t step = ((uint64_t)r + 1ull) * IM_GOLDEN;
        if (tid == 0) cnt = 0;
        __syncthreads();
        uint32_t head = 0;
        for (uint32_t g0 = 0; g0 < a.nS; g0 += a.group) {
            const uint32_t before = head;
            for (uint32_t i = g0 + tid; i < min(g0 + a.group, a.nS); i += NT) visit(a.S[i]);
            __syncthreads();
            for (;;) {
                const uint32_t end = cnt;
                __syncthreads();   // (cnt grows from here on)
                if (head == end) break;
                for (; head < end; head += NT) {
                    const uint32_t i = head + tid;
                    uint32_t r0 = 0, deg = 0;
                    if (i < end) {
                        const uint32_t x = entry(i);
                        r0 = a.row[x];
                        deg = a.row[x + 1] - r0;
                    }
                    uint32_t total;
                    ex[tid] = group_excl_scan<NT>(deg, wsum, &total);
                    rs[tid] = r0;
                    __syncthreads();
                    for (uint32_t j0 = tid; j0 < total; j0 += NT * SPR_U) {
                        ArcCoin c[SPR_U];
#pragma unroll
                        for (int u = 0; u < SPR_U; u++) {
                            const uint32_t j = j0 + (uint32_t)u * NT;
                            c[u].head = IM_EMPTY;
                            c[u].key = 0; c[u].last = 0;
                            if (j < total && j >= j0) {
                                const int k = upper_index<NT>(ex, j);
                                const uint32_t e = rs[k] + (j - ex[k]);
                                c[u] = RECORDS ? a.coin[e] : arc_coin(a.col, a.prob, a.seed, e);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < SPR_U; u++)
                            if (c[u].head != IM_EMPTY &&
                                (uint32_t)(sm64_finalise(c[u].key + step) >> 32) <= c[u].last)
                                visit(c[u].head);
                    }
                    __syncthreads();
                }
                head = end;
            }
            if (tid == 0 && a.marg && head != before) {   // (marginals: one seed per search)
                if (sum_here) acc[g0] += head - before;
                else atomicAdd(&a.marg[g0], (unsigned long long)(head - before));
            }
        }
        if (tid == 0 && a.per_snapshot) a.per_snapshot[r] = head;
        // back to zero for the next snapshot
        for (uint32_t i = tid; i < head; i += NT) bits[entry(i) >> 5] = 0;
        __syncthreads();
    }
    if (sum_here)
        for (uint32_t i = tid; i < a.nS; i += NT)
            if (acc[i]) atomicAdd(&a.marg[i], (unsigned long long)acc[i]);
}
