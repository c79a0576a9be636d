// im_bits.h -- the largest initial-count tasks, one snapshot bit per wavefront.
//
// A task (node, word) that outgrew the LDS tables reaches hundreds to tens of
// thousands of nodes. On near-critical graphs its 64 snapshots hardly share
// them (1.2 snapshot bits per reached node on a weighted-cascade graph of
// 60,000 nodes), so searching them together saves nothing, while its dense
// state (16 bytes per node and task) makes every relaxation an atomic on
// memory that no cache holds. Here each wavefront searches one snapshot over
// its live lists with the visited nodes as a bitmap in LDS (n / 8 bytes; on
// graphs too large for that in a table, of CB_CS1 entries in a first launch and
// of CB_CS2, with which a hub's snapshots fit, in a second for the tasks that
// outgrew it; the dense tier takes what is left), and marks
// what any snapshot of the task reached in a bitmap of the task (LDS or
// memory), which gives its (node, word) counts.
// Bound: the two dependent loads of a level (list offsets, listed heads), times
// the levels, over the searches that the bitmaps leave room for (13 per CU at
// 60,000 nodes): the wavefronts wait three quarters of their time, and taking
// the L2 misses out (lists of eight snapshots per XCD) did not change it while a
// workgroup still ended its tasks one by one. All 64 frontiers of a task in one
// LDS table, level by level, were slower too (27 -> 28 to 46 ms).
// Where the snapshots do share their nodes (supercritical graphs), one search
// of the word does less: the task is handed to the dense tier if its first
// CB_PROBE searches reached more than twice the nodes that the task had marked
// by then (the sources aside). On a graph whose tasks nearly all share three
// quarters and more, the probes themselves cost up to one and a half times the
// dense tier: once CB_JUDGED tasks were judged (every fourth is) and seven eighths
// of them shared that much, only one in 16 is still probed, as a sample, and the
// others go on without (ms of this step; probing all -> sampling; the dense tier alone):
//   20,000 nodes, 2*10^5 arcs, p = 1, R = 64      445 -> 231; 178
//   8,000 nodes, 3.2*10^5 arcs, p = 0.6, R = 64   227 -> 166; 139
//   8,000 nodes, 8*10^4 arcs, p = 0.6 / 0.2       118 -> 100; 85 / 72 -> 73; 113
//   weighted cascade, 60,000 nodes, R = 128       18.7 -> 18.7; 61
// (Two counter loads per task, before it or at its probe, instead of the sums of
// every fourth judged: 210, 156 and 95 ms, but 2 to 3 % on weighted-cascade graphs.)
// (Judged at twice instead of six times the marks, p = 0.05 on the denser graph
// took 144 ms instead of 119.)
// Measured (tier 2 of the initial counts): see cnt_bits.
#pragma once

#include "im_rev.h"

constexpr int CB_WAVES = 16;     // most wavefronts (bits at a time) per workgroup
constexpr int CB_Q = 64;         // queue entries per wavefront kept in LDS as well
constexpr uint32_t CB_LIST = 4096;   // tables: words of a task's marks that are listed
constexpr int CB_TASKS = 8;      // most tasks in progress per workgroup
// Nodes whose live lists did not fit have their arcs' masks read once per snapshot
// here and once per word in the dense tier. With fewer tasks than workgroups a
// wavefront that reads a hub's arcs is what the launch waits for, and a span past
// CB_SCAN hands its task over at once (a star of 200,000 arcs, p = 0.05, R = 256:
// 46 ms here, 3.2 there; a hub of 60,000 among many tasks, 120,000 nodes, p = 0.15:
// 90 ms here, 133 there). With more, the probe decides: CB_SCANNED times as many
// arcs read by mask as nodes reached.
constexpr uint32_t CB_LONG = 1024, CB_SCAN = 16384, CB_SCANNED = 8;
constexpr uint32_t CB_PROBE = 8; // searches after which a task's snapshots are compared
constexpr uint32_t CB_SHARED = 6;    // ... that reached this many times the marks: shared
constexpr uint32_t CB_JUDGED = 32;
constexpr int CB_CS1 = 512, CB_CS2 = 4096;  // table entries per wavefront: first launch, second

struct BitsArgs {
    SnapGraph g;
    uint32_t R;
    const uint32_t *node_inst, *inst_R, *inst_off;   // batches (nullptr: one graph)
    uint32_t *gain;
    const uint32_t *in_q, *in_n;
    uint32_t *out_q, *out_n;     // tasks for the dense tier
    uint32_t *grab;
    uint32_t *judged;            // tasks judged by their probe, and those that shared (zero before)
    uint32_t *queue;             // [workgroups][wavefronts][nmax] (bitmaps) or [..][CS] (tables)
    uint32_t *any;               // tables: [workgroups][tasks][words of the largest instance], zero at rest
    uint32_t *list;              // tables: [workgroups][tasks][CB_LIST]
    uint32_t nmax;               // nodes of the largest instance
    uint32_t tasks;              // in progress per workgroup (1 .. CB_TASKS)
    unsigned long long *stats;
};

// orders a wavefront's own LDS and memory accesses for the compiler (the
// hardware keeps them in order)
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// sum over the wavefront (all lanes active), in registers: a search of a few
// nodes is shorter than the shuffles of wave_sum_u64
__device__ __forceinline__ uint32_t wave_sum_dpp(uint32_t x)
{
    auto from = [&](auto ctrl, auto rows) {
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl.value, rows.value, 0xF, false);
    };
    from(std::integral_constant<int, 0x111>(), std::integral_constant<int, 0xF>());   // row_shr:1
    from(std::integral_constant<int, 0x112>(), std::integral_constant<int, 0xF>());
    from(std::integral_constant<int, 0x114>(), std::integral_constant<int, 0xF>());
    from(std::integral_constant<int, 0x118>(), std::integral_constant<int, 0xF>());
    from(std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xA>());   // row_bcast:15
    from(std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xC>());   // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

struct WaveBig {
    uint32_t ex[64], start[64], kind[64];
};

// rev_expand for one wavefront: visit(v) for every live head of the lanes' spans
template <typename Visit>
__device__ __forceinline__ void wave_expand(WaveBig &B, const SnapGraph &a, uint32_t w, uint32_t b,
                                            const RevSpan &sp, Visit visit, uint32_t &arcs)
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

struct WaveLds {
    WaveBig B;
    uint32_t q[CB_Q];
};

// A task in progress. Its number among the workgroup's tasks is `ord`: free is
// the number that may take the place next, open that of the task in it plus one.
struct CntTask {
    uint32_t free, open, task, done, over, judge, sum, reached, words;
    unsigned long long relax, trav, arcs, scanned;
};

// The wavefronts take (task, bit) pairs in order, without a barrier: the sizes
// of a task's searches differ by two orders of magnitude, and a workgroup that
// ended each task together waited for its largest. The wavefront that finishes a
// task's last search adds up the task and opens its place. A wavefront waits
// only for an older task (a place that is still taken) or for the one that is
// reading the task in, never for a younger one, and takes one pair at a time.
template <int CS>   // table entries per wavefront (0: bitmaps)
__global__ __launch_bounds__(CB_WAVES * 64) void k_cnt_bits(BitsArgs a)
{
    constexpr bool TABLE = CS != 0;
    constexpr int LIM = CS / 4 * 3;   // most nodes in a table
    // bitmaps: [wavefronts + tasks][words of the largest instance]; tables:
    // [wavefronts][CS] nodes; then [wavefronts] of WaveLds
    extern __shared__ uint32_t maps[];
    __shared__ uint32_t cnt[CB_WAVES], s_item, s_skip;
    __shared__ CntTask T[CB_TASKS];
    __shared__ unsigned long long red[CB_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, nw = blockDim.x >> 6;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t words = (a.nmax + 31) / 32;
    const uint32_t per = TABLE ? (uint32_t)CS : words;          // words per wavefront
    uint32_t *mine = maps + (uint64_t)wv * per;
    uint32_t *any0 = TABLE ? a.any + (uint64_t)blockIdx.x * a.tasks * words : maps + (uint64_t)nw * words;
    uint32_t *queue = a.queue + ((uint64_t)blockIdx.x * nw + wv) * (TABLE ? (uint32_t)CS : a.nmax);
    const uint32_t nt = *a.in_n;
    if (blockIdx.x >= nt) return;
    const bool few = nt <= gridDim.x;
    const uint32_t nmaps = TABLE ? nw * per : (nw + a.tasks) * words;
    WaveLds &L = ((WaveLds *)(maps + nmaps))[wv];
    for (uint32_t i = tid; i < nmaps; i += blockDim.x)
        maps[i] = TABLE ? IM_EMPTY : 0u;
    if (tid == 0) { s_item = 0; s_skip = 0; }
    if (tid < CB_TASKS) {
        CntTask &t = T[tid];
        t.free = tid; t.open = 0; t.task = 0; t.done = 0; t.over = 0; t.judge = 0; t.sum = 0; t.reached = 0; t.words = 0;
        t.relax = 0; t.trav = 0; t.arcs = 0; t.scanned = 0;
    }
    // lane 0: of the tasks that this wavefront finished
    unsigned long long t_relax = 0, t_reached = 0, t_trav = 0, t_arcs = 0;
    __syncthreads();
    auto peek = [](uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto post = [](uint32_t *p, uint32_t v) {
        __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    for (;;) {
        uint32_t item = 0;
        if (lane == 0) item = atomicAdd(&s_item, 1u);
        item = __builtin_amdgcn_readfirstlane(item);   // (scalar: list and mask bases are, too)
        const uint32_t ord = item >> 6, b = item & 63u, place = ord % a.tasks;
        CntTask &tk = T[place];
        uint32_t *any = any0 + (uint64_t)place * words;
        uint32_t *list = a.list + ((uint64_t)blockIdx.x * a.tasks + place) * CB_LIST;
        if (b == 0) {
            while (peek(&tk.free) != ord) __builtin_amdgcn_s_sleep(1);
            if (lane == 0) {
                const uint32_t i = ord == 0 ? blockIdx.x : gridDim.x + atomicAdd(a.grab, 1u);
                tk.task = i < nt ? a.in_q[i] : IM_EMPTY;
                tk.judge = (i & 3u) == 0;
                if ((i & 15u) != 0 && peek(&s_skip)) { tk.judge = 0; tk.over = 1; }
                post(&tk.open, ord + 1);
            }
        }
        while (peek(&tk.open) != ord + 1) __builtin_amdgcn_s_sleep(1);
        const uint32_t task = __builtin_amdgcn_readfirstlane(tk.task);
        if (task == IM_EMPTY) break;   // (the others find it before its 64 bits are taken)
        const uint32_t w = task / a.g.n, src = task - w * a.g.n;
        const uint32_t inst = a.node_inst ? a.node_inst[src] : 0u;
        const uint32_t base = a.node_inst ? a.inst_off[inst] : 0u;
        const uint64_t valid = im_valid_bits(a.node_inst ? a.inst_R[inst] : a.R, w);
        if (((valid >> b) & 1ull) && !peek(&tk.over)) {
            // (of one search, each below 2^32: nodes, arcs, degrees of distinct nodes)
            uint32_t relax = 0, trav = 0, arcs = 0, reached = 0;
            unsigned long long scanned = 0;   // (the same in every lane)
            // queue entries are nodes (bitmaps) or table positions
            auto entry = [&](uint32_t i) { return i < (uint32_t)CB_Q ? L.q[i] : queue[i]; };
            auto push = [&](uint32_t x) {
                const uint32_t p = atomicAdd(&cnt[wv], 1u);
                if (p < (uint32_t)CB_Q) L.q[p] = x;
                else queue[p] = x;
            };
            auto visit = [&](uint32_t v) {
                if constexpr (TABLE) {
                    uint32_t h = slot_hash(v) >> (32 - __builtin_ctz(TABLE ? CS : 2));
                    // (a full table is left as it is: the task is handed over)
                    if (*(volatile uint32_t *)&cnt[wv] >= (uint32_t)LIM) { tk.over = 1; return; }
                    for (;;) {
                        const uint32_t key = atomicCAS(&mine[h], IM_EMPTY, v);
                        if (key == v) return;
                        if (key == IM_EMPTY) break;
                        h = (h + 1) & (CS - 1);
                    }
                    push(h);
                } else {
                    const uint32_t i = v - base, bit = 1u << (i & 31u);
                    if (!(atomicOr(&mine[i >> 5], bit) & bit)) push(v);
                }
            };
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
                        const uint32_t before = atomicOr(&any[i >> 5], bit);
                        if (!(before & bit)) { relax += dg; reached++; }
                        if (TABLE && before == 0) {
                            const uint32_t p = atomicAdd(&tk.words, 1u);
                            if (p < CB_LIST) list[p] = i >> 5;
                        }
                    }
                    if (__any(sp.len >= CB_LONG)) {   // (hubs alone are that long)
                        if (sp.kind == 2 && sp.len > CB_SCAN && few) { tk.over = 1; sp.len = 0; }
                        scanned += wave_sum_dpp(sp.kind == 2 ? sp.len : 0u);
                    }
                    wave_expand(L.B, a.g, w, b, sp, visit, arcs);
                }
                head = end;
                wave_order();
            }
            for (uint32_t i = lane; i < head; i += 64) {
                if (TABLE) mine[entry(i)] = IM_EMPTY;
                else mine[(entry(i) - base) >> 5] = 0;
            }
            wave_order();
            relax = wave_sum_dpp(relax); trav = wave_sum_dpp(trav);
            arcs = wave_sum_dpp(arcs); reached = wave_sum_dpp(reached);
            if (lane == 0) {
                atomicAdd(&tk.sum, head - 1);
                atomicAdd(&tk.reached, reached);
                atomicAdd(&tk.relax, (unsigned long long)relax);
                atomicAdd(&tk.trav, (unsigned long long)trav);
                atomicAdd(&tk.arcs, (unsigned long long)arcs);
                if (scanned) atomicAdd(&tk.scanned, scanned);
            }
        }
        uint32_t done = 0;
        if (TABLE) __builtin_amdgcn_s_waitcnt(0);   // the listed words are in place
        if (lane == 0)
            done = __hip_atomic_fetch_add(&tk.done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) + 1;
        done = __builtin_amdgcn_readfirstlane(done);
        // the first searches: do the snapshots share their nodes?
        if (done == CB_PROBE && lane == 0) {
            const uint32_t sum = tk.sum, reached = tk.reached;
            if (sum > 2u * reached + 64u || tk.scanned > (unsigned long long)CB_SCANNED * (sum + CB_PROBE))
                post(&tk.over, 1u);
            // (of words with few snapshots the probe is over before they can share)
            if (tk.judge && __popcll(valid) >= 32) {
                const uint32_t judged = atomicAdd(&a.judged[0], 1u) + 1;
                const uint32_t yes = sum > CB_SHARED * reached ? 1u : 0u;
                const uint32_t shared = atomicAdd(&a.judged[1], yes) + yes;
                post(&s_skip, judged >= CB_JUDGED && shared >= judged / 8 * 7 ? 1u : 0u);
            }
        }
        if (done < 64) continue;
        // (marks in memory can be far more than the task reached: clearing the
        // words that it touched, not n / 32, took the first launch on 10^6 nodes
        // from 1.48 to 1.35 ms, and keeps larger graphs from paying for n)
        if (TABLE && tk.words <= CB_LIST)
            for (uint32_t i = lane; i < tk.words; i += 64) any[list[i]] = 0;
        else
            for (uint32_t i = lane; i < words; i += 64) any[i] = 0;
        wave_order();
        if (lane == 0) {
            if (tk.over) {
                a.out_q[atomicAdd(a.out_n, 1u)] = task;
            } else {
                atomicAdd(&a.gain[src], tk.sum + (uint32_t)__popcll(valid));
                t_relax += tk.relax; t_reached += tk.reached; t_trav += tk.trav; t_arcs += tk.arcs;
            }
            tk.done = 0; tk.over = 0; tk.sum = 0; tk.reached = 0; tk.words = 0;
            tk.relax = 0; tk.trav = 0; tk.arcs = 0; tk.scanned = 0;
        }
        wave_order();
        if (TABLE) __builtin_amdgcn_s_waitcnt(0);   // the marks are gone before the place is open
        if (lane == 0) post(&tk.free, ord + a.tasks);
    }
    __syncthreads();
    auto total = [&](unsigned long long v) -> unsigned long long {
        if (lane == 0) red[wv] = v;
        __syncthreads();
        unsigned long long s = 0;
        for (uint32_t i = 0; i < nw; i++) s += red[i];
        __syncthreads();
        return s;
    };
    const unsigned long long r0 = total(t_relax), r1 = total(t_reached), r2 = total(t_trav), r3 = total(t_arcs);
    if (tid == 0 && r1) {
        stat_add(a.stats, st_tier(PASS_INIT, 2, F_RELAX), r0);
        stat_add(a.stats, st_tier(PASS_INIT, 2, F_REACHED), r1);
        stat_add(a.stats, ST_TRAV_INIT, r2);
        stat_add(a.stats, st_tier(PASS_INIT, 2, F_ARCS), r3);
    }
}
