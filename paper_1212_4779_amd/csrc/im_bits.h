// im_bits.h -- the largest initial-count tasks, one snapshot bit per wavefront.
//
// A task (node, word) that outgrew the LDS tables reaches hundreds to tens of
// thousands of nodes. On near-critical graphs its 64 snapshots hardly share
// them (1.2 snapshot bits per reached node on a weighted-cascade graph of
// 60,000 nodes), so searching them together saves nothing, while its dense
// state (16 bytes per node and task) makes every relaxation an atomic on
// memory that no cache holds. Here each wavefront searches one snapshot over
// its live lists with the visited nodes as a bitmap in LDS (n / 8 bytes; on
// graphs too large for that as a table of CB_CS nodes, with which a hub's
// snapshots fit and a task that outgrows it goes to the dense tier), and the
// workgroup's wavefronts mark what any of them reached in a shared bitmap (LDS
// or memory), which gives the task's (node, word) counts. Per level: list offsets, listed
// heads, two LDS atomics. Bound: those two dependent loads, times the levels
// of 64 / (wavefronts per workgroup) searches.
// Where the snapshots do share their nodes (supercritical graphs), one search
// of the word does less: after the first search of every wavefront the task is
// handed to the dense tier if they reached more than twice the nodes of their
// union (the source aside).
// Measured (tier 2 of the initial counts): see run_tiers.
#pragma once

#include "im_rev.h"

constexpr int CB_WAVES = 8;      // most wavefronts (bits at a time) per workgroup
constexpr int CB_Q = 128;        // queue entries per wavefront kept in LDS as well
constexpr int CB_CS = 4096, CB_LIM = 3072;   // table entries per wavefront, most nodes in it

struct BitsArgs {
    SnapGraph g;
    uint32_t R;
    const uint32_t *node_inst, *inst_R, *inst_off;   // batches (nullptr: one graph)
    uint32_t *gain;
    const uint32_t *in_q, *in_n;
    uint32_t *out_q, *out_n;     // tasks for the dense tier
    uint32_t *grab;
    uint32_t *queue;             // [workgroups][wavefronts][nmax] (bitmaps) or [..][CB_CS] (tables)
    uint32_t *any;               // tables: [workgroups][words of the largest instance], zero at rest
    uint32_t nmax;               // nodes of the largest instance
    unsigned long long *stats;
};

// orders a wavefront's own LDS and memory accesses for the compiler (the
// hardware keeps them in order)
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

struct WaveBig {
    uint32_t ex[64], start[64], kind[64];
};

// rev_expand for one wavefront: visit(v) for every live head of the lanes' spans
template <typename Visit>
__device__ __forceinline__ void wave_expand(WaveBig &B, const SnapGraph &a, uint32_t w, uint32_t b,
                                            const RevSpan &sp, Visit visit, uint64_t &arcs)
{
    const uint32_t lane = threadIdx.x & 63u;
    const bool big = sp.len > (uint32_t)REV_SMALL;
    const uint64_t bal = __ballot(big);
    rev_small(a, w, b, big ? 0u : sp.len, sp, visit);
    arcs += sp.len;
    if (!bal) return;
    const uint32_t nb = (uint32_t)__popcll(bal);
    const uint32_t q = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
    if (big) { B.ex[q] = sp.len; B.start[q] = sp.start; B.kind[q] = sp.kind; }
    wave_order();
    const uint32_t len = lane < nb ? B.ex[lane] : 0u;
    const uint32_t incl = wave_incl_scan(len);
    const uint32_t total = __shfl(incl, 63, 64);
    B.ex[lane] = incl - len;
    wave_order();
    for (uint32_t j0 = lane; j0 < total; j0 += 64 * REV_U) {
        uint32_t v[REV_U];
        bool live[REV_U];
#pragma unroll
        for (int u = 0; u < REV_U; u++) {
            const uint32_t j = j0 + 64u * (uint32_t)u;
            live[u] = false; v[u] = 0;
            if (j < total) {
                const int k = upper_index<64>(B.ex, j);
                live[u] = rev_head(a, w, b, B.kind[k], B.start[k] + (j - B.ex[k]), v[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < REV_U; u++)
            if (live[u]) visit(v[u]);
    }
    wave_order();
}

template <bool TABLE>
__global__ __launch_bounds__(CB_WAVES * 64) void k_cnt_bits(BitsArgs a)
{
    // bitmaps: [wavefronts + 1][words of the largest instance]; tables:
    // [wavefronts][CB_CS] nodes
    extern __shared__ uint32_t maps[];
    __shared__ WaveBig B[CB_WAVES];
    __shared__ uint32_t q[CB_WAVES][CB_Q], cnt[CB_WAVES], s_task, s_sum, s_union, s_next, s_over;
    __shared__ unsigned long long red[CB_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, nw = blockDim.x >> 6;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t words = (a.nmax + 31) / 32;
    const uint32_t per = TABLE ? (uint32_t)CB_CS : words;          // words per wavefront
    uint32_t *mine = maps + (uint64_t)wv * per;
    uint32_t *any = TABLE ? a.any + (uint64_t)blockIdx.x * words : maps + (uint64_t)nw * words;
    uint32_t *queue = a.queue + ((uint64_t)blockIdx.x * nw + wv) * (TABLE ? (uint32_t)CB_CS : a.nmax);
    const uint32_t nt = *a.in_n;
    if (blockIdx.x >= nt) return;
    for (uint32_t i = tid; i < (TABLE ? nw * per : (nw + 1) * words); i += blockDim.x)
        maps[i] = TABLE ? IM_EMPTY : 0u;
    if (tid == 0) { s_sum = 0; s_union = 0; s_next = nw; s_over = 0; }
    uint64_t t_relax = 0, t_reached = 0, t_trav = 0, t_arcs = 0;   // of the finished tasks
    uint32_t ran = 0;
    __syncthreads();
    for (uint32_t t = blockIdx.x; t < nt;) {
        const uint32_t task = __builtin_amdgcn_readfirstlane(a.in_q[t]);
        const uint32_t w = task / a.g.n, src = task - w * a.g.n;
        const uint32_t inst = a.node_inst ? a.node_inst[src] : 0u;
        const uint32_t base = a.node_inst ? a.inst_off[inst] : 0u;
        const uint64_t valid = im_valid_bits(a.node_inst ? a.inst_R[inst] : a.R, w);
        uint64_t relax = 0, reached = 0, trav = 0, arcs = 0;
        uint32_t sum = 0;
        // queue entries are nodes (bitmaps) or table positions
        auto entry = [&](uint32_t i) { return i < (uint32_t)CB_Q ? q[wv][i] : queue[i]; };
        auto push = [&](uint32_t x) {
            const uint32_t p = atomicAdd(&cnt[wv], 1u);
            if (p < (uint32_t)CB_Q) q[wv][p] = x;
            else queue[p] = x;
        };
        auto visit = [&](uint32_t v) {
            if constexpr (TABLE) {
                uint32_t h = slot_hash(v) >> (32 - __builtin_ctz(CB_CS));
                // (a full table is left as it is: the task is handed over)
                if (*(volatile uint32_t *)&cnt[wv] >= (uint32_t)CB_LIM) { s_over = 1; return; }
                for (;;) {
                    const uint32_t key = atomicCAS(&mine[h], IM_EMPTY, v);
                    if (key == v) return;
                    if (key == IM_EMPTY) break;
                    h = (h + 1) & (CB_CS - 1);
                }
                push(h);
            } else {
                const uint32_t i = v - base, bit = 1u << (i & 31u);
                if (!(atomicOr(&mine[i >> 5], bit) & bit)) push(v);
            }
        };
        bool over = false;
        for (uint32_t b = wv; b < 64;) {
            if ((valid >> b) & 1ull) {
                if (lane == 0) {
                    cnt[wv] = 0;
                    visit(src);
                }
                wave_order();
                uint32_t head = 0;
                for (;;) {
                    const uint32_t end = cnt[wv];
                    if (head == end) break;
                    for (; head < end; head += 64) {
                        RevSpan sp = {0, 0, 0};
                        if (head + lane < end) {
                            const uint32_t e = entry(head + lane), x = TABLE ? mine[e] : e;
                            sp = rev_span(a.g, w, b, x);
                            const uint32_t dg = a.g.row[x + 1] - a.g.row[x];
                            const uint32_t i = x - base, bit = 1u << (i & 31u);
                            trav += dg;
                            if (!(atomicOr(&any[i >> 5], bit) & bit)) { relax += dg; reached++; }
                        }
                        wave_expand(B[wv], a.g, w, b, sp, visit, arcs);
                    }
                    head = end;
                    wave_order();
                }
                sum += head;
                for (uint32_t i = lane; i < head; i += 64) {
                    if (TABLE) mine[entry(i)] = IM_EMPTY;
                    else mine[(entry(i) - base) >> 5] = 0;
                }
                wave_order();
            }
            if (b == wv) {   // the first searches: do the snapshots share their nodes?
                const uint64_t r = wave_sum_u64(reached);
                if (lane == 0) {
                    atomicAdd(&s_sum, sum - ((valid >> b) & 1ull ? 1u : 0u));
                    atomicAdd(&s_union, (uint32_t)r);
                }
                __syncthreads();
                over = s_sum > 2u * s_union + 64u;
                __syncthreads();
                if (over) break;
            }
            if (lane == 0) b = atomicAdd(&s_next, 1u);
            b = __builtin_amdgcn_readfirstlane(b);   // (scalar: list and mask bases are, too)
        }
        __syncthreads();
        over = over || s_over != 0;
        __syncthreads();
        if (tid == 0) { s_sum = 0; s_union = 0; s_next = nw; s_over = 0; }
        for (uint32_t i = tid; i < words; i += blockDim.x) any[i] = 0;
        if (over) {
            if (tid == 0) a.out_q[atomicAdd(a.out_n, 1u)] = task;
        } else {
            if (lane == 0) atomicAdd(&a.gain[src], sum);
            t_relax += relax; t_reached += reached; t_trav += trav; t_arcs += arcs;
            ran = 1;
        }
        if (tid == 0) s_task = gridDim.x + atomicAdd(a.grab, 1u);
        __syncthreads();
        t = s_task;
        __syncthreads();
    }
    auto total = [&](uint64_t v) -> unsigned long long {
        v = wave_sum_u64(v);
        if (lane == 0) red[wv] = v;
        __syncthreads();
        unsigned long long s = 0;
        for (uint32_t i = 0; i < nw; i++) s += red[i];
        __syncthreads();
        return s;
    };
    const unsigned long long r0 = total(t_relax), r1 = total(t_reached), r2 = total(t_trav), r3 = total(t_arcs);
    if (tid == 0 && ran) {
        stat_add(a.stats, st_tier(PASS_INIT, 2, F_RELAX), r0);
        stat_add(a.stats, st_tier(PASS_INIT, 2, F_REACHED), r1);
        stat_add(a.stats, ST_TRAV_INIT, r2);
        stat_add(a.stats, st_tier(PASS_INIT, 2, F_ARCS), r3);
    }
}
