// im_rev.h -- a round of the dynamic update by snapshot: the forward step, one
// workgroup per snapshot (k_fwd_snap), and the reverse step, 64 sources of one
// snapshot per search (k_rev_search).
//
// A round's newly covered (node, snapshot) pairs each subtract one from the
// gain of every node that reaches the node in that snapshot (the delete loop
// of Algorithm 2). The sources of one snapshot have nearly the same
// ancestors (everything that reaches a newly covered node reaches what lies
// behind it), so up to 64 of them share a search, one bit each:
//     reach[y] |= delta[x]   for every arc y -> x live in the snapshot,
// and a node's decrement is popcount(reach). Packing 64 different snapshots
// into a word instead (as the initial counts do) shares almost nothing here:
// on a weighted-cascade graph of 60,000 nodes a reached (node, word) pair held
// 1.1 snapshot bits, while 64 sources of one snapshot visit 0.13 nodes per
// decrement.
//
// Only the arcs live in the one snapshot are read, from the per-snapshot live
// lists (nodes without lists read their arcs' mask words). The searches run in LDS tables of 2,048 entries, those that outgrow them in
// tables of 4,096 entries and, past that, in a dense slot in global memory.
// The bound is the latency of a level: row bounds and list offsets, then the
// listed heads (two dependent global loads), then the table update.
// Measured against packed snapshots: see the launch code (rev_search).
#pragma once

#include "im_bfs.h"

// a graph in one direction with its masks and per-snapshot live lists
struct SnapGraph {
    const uint32_t *row;      // [n+1]
    const uint32_t *col;      // [m]
    const uint64_t *mask;     // [W][m]
    uint64_t m;
    uint32_t n, W;
    HubLists hub;
    SparseLists sp;
};

struct RevArgs {
    SnapGraph g;                // reverse arcs
    const uint32_t *node_inst;  // batches: instance of each node (nullptr: one graph)
    const uint32_t *inst_off;   // batches: first node of each instance
    // the round's sources and its tasks (rev_task)
    const uint32_t *src;
    const uint2 *tasks;
    const uint32_t *ntasks;
    // in_q / in_n: this launch's tasks (nullptr: all), out_q / out_n: tasks
    // that outgrow its tables
    const uint32_t *in_q, *in_n;
    uint32_t *out_q, *out_n;
    uint32_t *grab;             // task counter of this launch (zero before it)
    // dense slots (as the last tier of im_bfs.h): (reach, pend) records, zero
    // at rest, queues and visit list
    uint64_t *b_reach;
    uint32_t *b_qa, *b_qb, *b_vis;
    uint32_t slot_n;
    uint32_t *gain;
    unsigned long long *stats;
    int tier;
};

// a task: x = first source, y = sources (1..64) | snapshot bit << 8 | word << 16
__device__ __forceinline__ uint2 rev_task(uint32_t first, uint32_t cnt, uint32_t bit, uint32_t word)
{
    return make_uint2(first, cnt | (bit << 8) | (word << 16));
}

// where the heads of x's arcs live in snapshot 64w + b are: kind 0
// the sparse lists, 1 the hub lists, 2 the arcs themselves (heads whose mask
// word has the bit)
struct RevSpan {
    uint32_t start, len, kind;
};

__device__ __forceinline__ RevSpan rev_span(const SnapGraph &a, uint32_t w, uint32_t b, uint32_t x)
{
    const uint32_t *o = a.sp.off + sparse_at(a.sp, w * 64u + b, x);
    const uint32_t first = o[0], end = o[1];
    RevSpan s;
    if (!(first & SP_NONE)) {
        s.start = first; s.len = (end & ~SP_NONE) - first; s.kind = 0;
        return s;
    }
    const uint32_t rs = a.row[x], deg = a.row[x + 1] - rs;
    const uint32_t hs = deg >= a.hub.min_deg ? a.hub.slot[x] : IM_EMPTY;
    if (hs != IM_EMPTY) {
        const uint32_t *o = a.hub.off + ((uint64_t)hs * a.W + w) * 65 + b;
        s.start = o[0]; s.len = o[1] - s.start; s.kind = 1;
    } else {
        s.start = rs; s.len = deg; s.kind = 2;
    }
    return s;
}

// the head at position pos of a span of this kind; false: not live
__device__ __forceinline__ bool rev_head(const SnapGraph &a, uint32_t w, uint32_t b, uint32_t kind,
                                         uint32_t pos, uint32_t &v)
{
    const uint32_t *heads = kind == 0 ? a.sp.adj : kind == 1 ? a.hub.adj : a.col;
    v = heads[pos];
    return kind != 2 || ((a.mask[(uint64_t)w * a.m + pos] >> b) & 1ull);
}

constexpr int REV_SMALL = 4;   // spans up to this length are expanded by one lane

// Heads 0 .. len - 1 (at most REV_SMALL) of the lane's span, loaded together.
// A level of a thin search is mostly instructions: steps that no lane of the
// wavefront needs are skipped, and listed heads (kind 0) take a path of their
// own, without the choice of array and mask.
template <typename Visit>
__device__ __forceinline__ void rev_small(const SnapGraph &a, uint32_t w, uint32_t b, uint32_t len,
                                          const RevSpan &sp, Visit visit)
{
    uint32_t v[REV_SMALL];
    bool live[REV_SMALL];
    if (!__any(len != 0 && sp.kind != 0)) {
#pragma unroll
        for (int u = 0; u < REV_SMALL; u++) {
            v[u] = 0;
            live[u] = (uint32_t)u < len;
            if (live[u]) v[u] = a.sp.adj[sp.start + (uint32_t)u];
        }
    } else {
#pragma unroll
        for (int u = 0; u < REV_SMALL; u++) {
            v[u] = 0;
            live[u] = (uint32_t)u < len && rev_head(a, w, b, sp.kind, sp.start + (uint32_t)u, v[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < REV_SMALL; u++)
        if (live[u]) visit(v[u]);
}
constexpr int REV_U = 4;       // heads in flight per lane in the longer ones

template <int NT>
struct RevBig {                // the longer spans of one chunk of the frontier
    uint32_t ex[NT], start[NT], own[NT];   // ex: length, then exclusive prefix;
                                           // own: caller's index | kind << 30
    uint32_t wsum[NT / 64 + 1];
    uint32_t n;
};

// Expand the chunk's spans: `take` lanes hold a frontier entry `own` (below
// 2^30) with its span and delta. relax(own, v) is called for every live head.
// All threads call it; ends with a barrier.
template <int NT, typename Relax>
__device__ __forceinline__ void rev_expand(RevBig<NT> &B, const SnapGraph &a, uint32_t w, uint32_t b,
                                           bool take, uint32_t own, const RevSpan &sp, Relax relax,
                                           uint64_t &arcs)
{
    const int tid = threadIdx.x;
    const bool small = take && sp.len <= (uint32_t)REV_SMALL, big = take && !small;
    rev_small(a, w, b, small ? sp.len : 0u, sp, [&](uint32_t v) { relax(own, v); });
    if (small) arcs += sp.len;
    const uint32_t q = wave_append(big, &B.n);
    if (big) { B.start[q] = sp.start; B.ex[q] = sp.len; B.own[q] = own | (sp.kind << 30); }
    __syncthreads();
    const uint32_t nb = B.n;
    if (nb) {
        uint32_t total;
        B.ex[tid] = group_excl_scan<NT>((uint32_t)tid < nb ? B.ex[tid] : 0u, B.wsum, &total);
        if (tid == 0) { B.n = 0; arcs += total; }
        __syncthreads();
        for (uint32_t j0 = tid; j0 < total; j0 += NT * REV_U) {
            uint32_t v[REV_U], own_u[REV_U];
            bool live[REV_U];
#pragma unroll
            for (int u = 0; u < REV_U; u++) {
                const uint32_t j = j0 + (uint32_t)u * NT;
                live[u] = false; v[u] = 0; own_u[u] = 0;
                if (j < total) {
                    const int k = upper_index<NT>(B.ex, j);
                    own_u[u] = B.own[k];
                    live[u] = rev_head(a, w, b, own_u[u] >> 30, B.start[k] + (j - B.ex[k]), v[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < REV_U; u++)
                if (live[u]) relax(own_u[u] & 0x3FFFFFFFu, v[u]);
        }
    }
    __syncthreads();
}

template <int NT, int CS>
struct RevLds {
    uint32_t keys[CS];
    uint64_t reach[CS], pend[CS];
    uint16_t fr[2][CS];
    RevBig<NT> B;
    unsigned long long red[NT / 64];
    uint32_t nf, nn, cnt, ovf, task;
};

struct RevCounts {
    uint64_t relax = 0, reached = 0, arcs = 0, trav = 0, dec = 0, ovf = 0;
};

// enter `bits` at node v; an entry whose pending bits become non-zero joins list `lst`
template <int NT, int CS, int LIM>
__device__ __forceinline__ void rev_relax(RevLds<NT, CS> &L, uint32_t v, uint64_t bits, int lst,
                                          uint32_t *counter)
{
    constexpr int LOG_CS = __builtin_ctz(CS);
    if (L.ovf) return;   // abandoned: stop touching its full table
    uint32_t h = slot_hash(v) >> (32 - LOG_CS);
    int found = -1;
    for (int p = 0; p < CS; p++) {
        const uint32_t key = L.keys[h];
        if (key == v) { found = (int)h; break; }
        if (key == IM_EMPTY) {
            const uint32_t old = atomicCAS(&L.keys[h], IM_EMPTY, v);
            if (old == IM_EMPTY) {
                if (atomicAdd(&L.cnt, 1u) >= (uint32_t)LIM) L.ovf = 1;
                found = (int)h;
                break;
            }
            if (old == v) { found = (int)h; break; }
        }
        h = (h + 1) & (CS - 1);
    }
    if (found < 0) { L.ovf = 1; return; }
    const uint64_t old = atomicOr((unsigned long long *)&L.reach[found], (unsigned long long)bits);
    const uint64_t nb = bits & ~old;
    if (nb && atomicOr((unsigned long long *)&L.pend[found], (unsigned long long)nb) == 0)
        L.fr[lst][atomicAdd(counter, 1u)] = (uint16_t)found;
}

// Run task `tk` in the LDS table, which is empty on entry and on return.
// Returns false when it outgrew the table (nothing was counted then).
template <int NT, int CS, int LIM>
__device__ bool rev_run_lds(RevLds<NT, CS> &L, const RevArgs &a, uint2 tk, RevCounts &c)
{
    const int tid = threadIdx.x;
    const uint32_t cnt = tk.y & 0xFFu, b = (tk.y >> 8) & 0xFFu, w = tk.y >> 16;
    if (tid == 0) { L.nf = 0; L.nn = 0; L.cnt = 0; L.ovf = 0; L.B.n = 0; }
    __syncthreads();
    if ((uint32_t)tid < cnt) rev_relax<NT, CS, LIM>(L, a.src[tk.x + tid], 1ull << tid, 0, &L.nf);
    __syncthreads();
    uint64_t arcs = 0;
    for (int cur = 0;; cur ^= 1) {
        const uint32_t nf = L.nf;   // zero once the table has overflowed
        if (nf == 0) break;
        for (uint32_t base = 0; base < nf; base += NT) {
            const bool take = base + tid < nf;
            uint32_t idx = 0;
            uint64_t d = 0;
            RevSpan sp = {0, 0, 0};
            if (take) {
                idx = L.fr[cur][base + tid];
                // the bits gained since the last expansion; bits that arrive
                // later re-queue the entry for the next level
                d = atomicExch((unsigned long long *)&L.pend[idx], 0ull);
                sp = rev_span(a.g, w, b, L.keys[idx]);
            }
            // a longer span's delta is looked up by its owner: the bits taken
            // above are part of reach, and passing on bits of reach that are
            // still pending only brings them forward
            rev_expand<NT>(L.B, a.g, w, b, take, idx, sp,
                           [&](uint32_t own, uint32_t v) {
                               const uint64_t bits = own == idx && take ? d : L.reach[own];
                               rev_relax<NT, CS, LIM>(L, v, bits, cur ^ 1, &L.nn);
                           },
                           arcs);
        }
        if (tid == 0) { L.nf = L.ovf ? 0u : L.nn; L.nn = 0; }
        __syncthreads();
    }
    const bool ok = L.ovf == 0;
    for (uint32_t i = tid; i < CS; i += NT) {
        const uint32_t key = L.keys[i];
        if (key == IM_EMPTY) continue;
        if (ok) {
            const uint32_t pc = (uint32_t)__popcll(L.reach[i]), dg = a.g.row[key + 1] - a.g.row[key];
            atomicSub(&a.gain[key], pc);
            c.relax += dg;
            c.reached += 1;
            c.trav += (uint64_t)pc * dg;
            c.dec += pc;
        }
        L.keys[i] = IM_EMPTY; L.reach[i] = 0; L.pend[i] = 0;
    }
    c.arcs += arcs;
    __syncthreads();
    return ok;
}

// Run task `tk` in the dense slot (reach and pend zero on entry and on return).
template <int NT>
__device__ void rev_run_dense(RevBig<NT> &B, uint32_t *ctr, const RevArgs &a, uint2 tk,
                              uint32_t slot, RevCounts &c)
{
    const int tid = threadIdx.x;
    const uint32_t cnt = tk.y & 0xFFu, b = (tk.y >> 8) & 0xFFu, w = tk.y >> 16;
    // a task's sources are of one instance, and so is everything it reaches
    const uint32_t base0 = a.node_inst ? a.inst_off[a.node_inst[a.src[tk.x]]] : 0u;
    uint64_t *rec = a.b_reach + (uint64_t)slot * a.slot_n * 2;
    uint32_t *cur = a.b_qa + (uint64_t)slot * a.slot_n, *nxt = a.b_qb + (uint64_t)slot * a.slot_n;
    uint32_t *vis = a.b_vis + (uint64_t)slot * a.slot_n;
    uint32_t &nf = ctr[0], &nn = ctr[1], &nvis = ctr[2];
    if (tid == 0) { nf = 0; nn = 0; nvis = 0; B.n = 0; }
    __syncthreads();
    if ((uint32_t)tid < cnt)
        global_relax<2>(rec, rec + 1, base0, vis, cur, &nvis, &nf, a.src[tk.x + tid], 1ull << tid);
    __syncthreads();
    uint64_t arcs = 0;
    for (;;) {
        const uint32_t nfr = nf;
        if (nfr == 0) break;
        for (uint32_t base = 0; base < nfr; base += NT) {
            const bool take = base + tid < nfr;
            uint32_t x = base0;
            uint64_t d = 0;
            RevSpan sp = {0, 0, 0};
            if (take) {
                x = cur[base + tid];
                d = atomicExch((unsigned long long *)&rec[(uint64_t)(x - base0) * 2 + 1], 0ull);
                sp = rev_span(a.g, w, b, x);
            }
            rev_expand<NT>(B, a.g, w, b, take, x - base0, sp,
                           [&](uint32_t own, uint32_t v) {
                               const uint64_t bits =
                                   own == x - base0 && take
                                       ? d
                                       : (uint64_t)atomicOr((unsigned long long *)&rec[(uint64_t)own * 2], 0ull);
                               global_relax<2>(rec, rec + 1, base0, vis, nxt, &nvis, &nn, v, bits);
                           },
                           arcs);
        }
        uint32_t *t = cur; cur = nxt; nxt = t;
        if (tid == 0) { nf = nn; nn = 0; }
        __syncthreads();
    }
    const uint32_t nv = nvis;
    for (uint32_t i = tid; i < nv; i += NT) {
        const uint32_t x = vis[i];
        uint64_t *r = &rec[(uint64_t)(x - base0) * 2];
        const uint32_t pc = (uint32_t)__popcll(*r), dg = a.g.row[x + 1] - a.g.row[x];
        *r = 0;   // pend is zero at the fixpoint
        atomicSub(&a.gain[x], pc);
        c.relax += dg;
        c.reached += 1;
        c.trav += (uint64_t)pc * dg;
        c.dec += pc;
    }
    c.arcs += arcs;
    __syncthreads();
}

template <int NT>
__device__ void rev_finish(const RevArgs &a, RevCounts c, unsigned long long *red, uint32_t ran)
{
    c.relax = group_sum<NT>(c.relax, red);
    c.reached = group_sum<NT>(c.reached, red);
    c.trav = group_sum<NT>(c.trav, red);
    c.dec = group_sum<NT>(c.dec, red);
    c.arcs = group_sum<NT>(c.arcs, red);
    if (threadIdx.x == 0 && ran) {
        stat_add(a.stats, ST_DECREMENTS, c.dec);
        stat_add(a.stats, st_tier(PASS_REV, a.tier, F_RELAX), c.relax);
        stat_add(a.stats, st_tier(PASS_REV, a.tier, F_REACHED), c.reached);
        stat_add(a.stats, st_tier(PASS_REV, a.tier, F_ARCS), c.arcs);
        stat_add(a.stats, st_tier(PASS_REV, a.tier, F_OVF), c.ovf);
        stat_add(a.stats, ST_TRAV_REV, c.trav);
    }
}

// One task at a time per workgroup. DENSE: a task that outgrows the table
// runs on in the workgroup's dense slot; otherwise it is queued for the next
// launch.
template <int NT, int CS, int LIM, bool DENSE>
__global__ __launch_bounds__(NT) void k_rev_search(RevArgs a)
{
    static_assert((CS & (CS - 1)) == 0 && LIM < CS && CS <= 65536, "table");
    __shared__ RevLds<NT, CS> L;
    __shared__ uint32_t ctr[3];
    const int tid = threadIdx.x;
    const uint32_t nt = a.in_q ? *a.in_n : *a.ntasks;
    if (blockIdx.x >= nt) return;
    for (uint32_t i = tid; i < CS; i += NT) { L.keys[i] = IM_EMPTY; L.reach[i] = 0; L.pend[i] = 0; }
    RevCounts c;
    uint32_t ran = 0;
    // the first task is the workgroup's own, further ones come from a counter
    for (uint32_t t = blockIdx.x; t < nt;) {
        const uint32_t id = a.in_q ? a.in_q[t] : t;
        uint2 tk = a.tasks[id];
        // the same in every lane: snapshot, list and mask bases stay scalar
        tk.x = __builtin_amdgcn_readfirstlane(tk.x);
        tk.y = __builtin_amdgcn_readfirstlane(tk.y);
        if (!rev_run_lds<NT, CS, LIM>(L, a, tk, c)) {
            if (DENSE) {
                rev_run_dense<NT>(L.B, ctr, a, tk, blockIdx.x, c);
            } else if (tid == 0) {
                a.out_q[atomicAdd(a.out_n, 1u)] = id;
                c.ovf++;
            }
        }
        ran++;
        if (nt <= gridDim.x) break;
        if (tid == 0) L.task = gridDim.x + atomicAdd(a.grab, 1u);
        __syncthreads();
        t = L.task;
        __syncthreads();
    }
    rev_finish<NT>(a, c, L.red, ran);
}

// ---------------------------------------------------------------------------
// The forward step, one workgroup per snapshot (of every instance): commit the
// instance's argmax, search from it over the snapshot's live arcs, pruned at
// covered, and leave the newly covered nodes, which are the search's queue,
// as the reverse step's sources, 64 to a task.
// A word of 64 snapshots searched together needs many workgroups, and a grid
// barrier per level, to be as wide; the snapshots' searches are independent,
// so a level here costs list offsets, listed heads and an LDS bit per head (the
// snapshot's covered bits are taken into LDS, up to FWS_LDS_NODES nodes) and
// three workgroup barriers. Figures: rev_search.
// ---------------------------------------------------------------------------
struct FwdSnapArgs {
    SnapGraph g;                     // forward arcs
    Batch b;
    uint32_t R, Rmax, t;             // R: of one graph; Rmax workgroups per instance
    const unsigned long long *key;   // one per instance
    uint32_t *seeds_out;
    uint64_t *gains_out;
    uint8_t *sel;
    // covered nodes of each snapshot, [R][cwords] (one bit per node of the
    // graph, or of the batch); nlds: nodes of the largest instance if its bits
    // are taken into LDS for the search, else 0
    uint32_t *cov;
    uint64_t cwords;
    uint32_t nlds;
    uint32_t *src;                   // a snapshot's queue: up to n (its instance's) nodes
    uint2 *tasks;                    // nullptr: no reverse step follows
    uint32_t *ntasks;                // zero before the launch
    // the lazy path's last evaluations (one graph; kept_n = 0: none), candidate
    // j in snapshot r: kept_len[j R + r] nodes at kept_q + (j R + r) n
    uint32_t kept_n;
    const uint32_t *kept_src, *kept_len, *kept_q;
    uint32_t *stamp;                 // [W][n] last round (plus one) that newly covered the node
                                     // in any snapshot of the word, for the (node, word) counters
    unsigned long long *stats;
};

constexpr uint32_t FWS_LDS_NODES = 1u << 18;
constexpr int FWS_NT = 512, FWS_Q = 4096;   // queue entries kept in LDS as well

__global__ __launch_bounds__(FWS_NT) void k_fwd_snap(FwdSnapArgs a)
{
    extern __shared__ uint32_t fws_bits[];
    __shared__ RevBig<FWS_NT> B;
    __shared__ uint32_t q[FWS_Q], cnt, s_t0, s_kept;
    __shared__ unsigned long long red[FWS_NT / 64];
    const uint32_t tid = threadIdx.x, inst = blockIdx.x / a.Rmax, r = blockIdx.x - inst * a.Rmax;
    const unsigned long long key = a.key[inst];
    const bool single = a.b.count == 1;
    const uint32_t R = single ? a.R : a.b.R[inst];
    if (key == 0 || r >= R) return;   // the instance has its k seeds
    const uint32_t v = 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull);
    uint32_t ni = a.g.n, n0 = 0;
    uint64_t base = 0;
    if (!single) { n0 = a.b.node_off[inst]; ni = a.b.node_off[inst + 1] - n0; base = a.b.pair_off[inst]; }
    base += (uint64_t)r * ni;
    if (r == 0 && tid == 0) {
        const uint32_t out = (single ? 0u : a.b.kpre[inst]) + a.t;
        a.seeds_out[out] = v - (single ? 0u : a.b.node_off[inst]);
        a.gains_out[out] = key >> 32;
        a.sel[v] = 1;
    }
    const uint32_t w = r / 64, b = r % 64;
    uint32_t *cov = a.cov + (uint64_t)r * a.cwords, *seen = cov;
    uint32_t w0 = 0;   // first word of `seen`
    uint32_t *src = a.src + base;
    if (tid == 0) { s_kept = IM_EMPTY; cnt = 0; B.n = 0; }
    __syncthreads();
    for (uint32_t j = tid; j < a.kept_n; j += FWS_NT)
        if (a.kept_src[j] == v) s_kept = j;   // candidates are distinct: one writer
    __syncthreads();
    const bool kept = s_kept != IM_EMPTY;
    const uint32_t *list = src;   // queue entries past the first FWS_Q (kept: all)
    uint32_t N;
    if (kept) {
        // the seed's own evaluation, pruned at covered, is its newly covered set
        const uint64_t at = (uint64_t)s_kept * R + r;
        list = a.kept_q + at * ni;
        N = a.kept_len[at];
    } else {
        if (a.nlds) {
            w0 = n0 / 32;
            const uint32_t words = (n0 + ni + 31) / 32 - w0;
            for (uint32_t i = tid; i < words; i += FWS_NT) fws_bits[i] = cov[w0 + i];
            seen = fws_bits;
            __syncthreads();
        }
        auto visit = [&](uint32_t y) {
            const uint32_t bit = 1u << (y & 31u);
            if (atomicOr(&seen[(y >> 5) - w0], bit) & bit) return;
            const uint32_t p = atomicAdd(&cnt, 1u);
            if (p < (uint32_t)FWS_Q) q[p] = y;
            src[p] = y;
        };
        if (tid == 0) visit(v);
        __syncthreads();
        uint64_t arcs = 0;
        for (uint32_t head = 0;;) {
            const uint32_t end = cnt;
            __syncthreads();   // (cnt grows from here on)
            if (head == end) break;
            for (; head < end; head += FWS_NT) {
                const uint32_t i = head + tid;
                const bool take = i < end;
                RevSpan sp = {0, 0, 0};
                if (take) sp = rev_span(a.g, w, b, i < (uint32_t)FWS_Q ? q[i] : src[i]);
                rev_expand<FWS_NT>(B, a.g, w, b, take, 0u, sp, [&](uint32_t, uint32_t y) { visit(y); }, arcs);
            }
            head = end;
        }
        N = cnt;
    }
    uint64_t trav = 0, relax = 0, pairs = 0;
    for (uint32_t i = tid; i < N; i += FWS_NT) {
        const uint32_t x = !kept && i < (uint32_t)FWS_Q ? q[i] : list[i];
        const uint32_t od = a.g.row[x + 1] - a.g.row[x];
        trav += od;
        if (seen != cov || kept) atomicOr(&cov[x >> 5], 1u << (x & 31u));
        if (atomicExch(&a.stamp[(uint64_t)w * a.g.n + x], a.t + 1) != a.t + 1) { relax += od; pairs++; }
    }
    const uint32_t nt = a.tasks ? (N + 63) / 64 : 0u;
    if (tid == 0) s_t0 = nt ? atomicAdd(a.ntasks, nt) : 0u;
    trav = group_sum<FWS_NT>(trav, red);
    relax = group_sum<FWS_NT>(relax, red);
    pairs = group_sum<FWS_NT>(pairs, red);
    for (uint32_t g = tid; g < nt; g += FWS_NT)
        a.tasks[s_t0 + g] = rev_task((uint32_t)base + 64u * g, min(64u, N - 64u * g), b, w);
    if (tid == 0 && N) {
        stat_add(a.stats, ST_TRAV_FWD, trav);
        stat_add(a.stats, ST_RELAX_FWD, relax);
        stat_add(a.stats, ST_TASKS_REV, pairs);
    }
}

// ---------------------------------------------------------------------------
// Exact evaluations of the lazy path, one workgroup per (candidate, snapshot):
// the number of nodes the candidate reaches in the snapshot that are not
// covered. The queue stays where it is, for the commit of the round's seed.
// A word's 64 snapshots in eight bit groups on dense slots (the engine this
// stands in for) spend a level of about 17 us on atomics in memory; here it is
// queue, list offsets, heads and covered, and a visit bit in LDS (in memory
// past EVS_LDS_NODES nodes). Figures: select_lazy.
// ---------------------------------------------------------------------------
constexpr int EVS_NT = 256, EVS_Q = 2048;
constexpr uint32_t EVS_LDS_NODES = 1u << 18;

struct EvalSnapArgs {
    SnapGraph g;
    uint32_t R;
    const uint32_t *cand, *ncand;    // [>= ncand], device count
    const uint32_t *cov;             // as in FwdSnapArgs
    uint64_t cwords;
    uint32_t *ev;                    // [n], += per candidate (zero before)
    uint32_t *kept_src, *kept_len, *kept_q;   // as in FwdSnapArgs
    uint32_t *bits;                  // [grid][ceil(n / 32)], zero at rest; nullptr: LDS
    unsigned long long *stats;
};

__global__ __launch_bounds__(EVS_NT) void k_eval_snap(EvalSnapArgs a)
{
    extern __shared__ uint32_t evs_bits[];
    __shared__ RevBig<EVS_NT> B;
    __shared__ uint32_t q[EVS_Q], cnt;
    __shared__ unsigned long long red[EVS_NT / 64];
    const uint32_t tid = threadIdx.x, j = blockIdx.x / a.R, r = blockIdx.x - j * a.R, n = a.g.n;
    if (j >= *a.ncand) {
        if (r == 0 && tid == 0) a.kept_src[j] = IM_EMPTY;
        return;
    }
    const uint32_t v = a.cand[j], w = r / 64, b = r % 64, words = (n + 31) / 32;
    const uint32_t *cov = a.cov + (uint64_t)r * a.cwords;
    auto covered = [&](uint32_t y) { return (cov[y >> 5] >> (y & 31u)) & 1u; };
    uint32_t *list = a.kept_q + (uint64_t)blockIdx.x * n;
    uint32_t *bits = a.bits ? a.bits + (uint64_t)blockIdx.x * words : evs_bits;
    if (r == 0 && tid == 0) a.kept_src[j] = v;
    if (covered(v)) {   // uniform over the workgroup
        if (tid == 0) a.kept_len[blockIdx.x] = 0;
        return;
    }
    if (!a.bits)
        for (uint32_t i = tid; i < words; i += EVS_NT) bits[i] = cov[i];   // covered counts as seen
    if (tid == 0) { cnt = 0; B.n = 0; }
    __syncthreads();
    auto visit = [&](uint32_t y) {
        if (a.bits && covered(y)) return;
        const uint32_t m = 1u << (y & 31u);
        if (atomicOr(&bits[y >> 5], m) & m) return;
        const uint32_t p = atomicAdd(&cnt, 1u);
        if (p < (uint32_t)EVS_Q) q[p] = y;
        list[p] = y;
    };
    if (tid == 0) visit(v);
    __syncthreads();
    uint64_t arcs = 0, trav = 0;
    for (uint32_t head = 0;;) {
        const uint32_t end = cnt;
        __syncthreads();   // (cnt grows from here on)
        if (head == end) break;
        for (; head < end; head += EVS_NT) {
            const uint32_t i = head + tid;
            const bool take = i < end;
            RevSpan sp = {0, 0, 0};
            if (take) {
                const uint32_t x = i < (uint32_t)EVS_Q ? q[i] : list[i];
                sp = rev_span(a.g, w, b, x);
                trav += a.g.row[x + 1] - a.g.row[x];
            }
            rev_expand<EVS_NT>(B, a.g, w, b, take, 0u, sp, [&](uint32_t, uint32_t y) { visit(y); }, arcs);
        }
        head = end;
    }
    const uint32_t N = cnt;
    if (a.bits)
        for (uint32_t i = tid; i < N; i += EVS_NT) bits[(i < (uint32_t)EVS_Q ? q[i] : list[i]) >> 5] = 0;
    trav = group_sum<EVS_NT>(trav, red);
    arcs = group_sum<EVS_NT>(arcs, red);
    if (tid == 0) {
        a.kept_len[blockIdx.x] = N;
        atomicAdd(&a.ev[v], N);
        stat_add(a.stats, ST_TRAV_EVAL, trav);
        stat_add(a.stats, st_tier(PASS_EVAL, 2, F_RELAX), trav);
        stat_add(a.stats, st_tier(PASS_EVAL, 2, F_REACHED), N);
        stat_add(a.stats, st_tier(PASS_EVAL, 2, F_ARCS), arcs);
    }
}
