// im_rev.h -- the reverse step of the dynamic update, 64 sources of one
// snapshot per search.
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
// lists (nodes without lists read their arcs' mask words). The pairs are
// sorted by (instance, snapshot) each round (k_rev_plan, k_rev_fill); the
// searches run in LDS tables of 2,048 entries, those that outgrow them in
// tables of 4,096 entries and, past that, in a dense slot in global memory.
// The bound is the latency of a level: row bounds and list offsets, then the
// listed heads (two dependent global loads), then the table update.
// Measured against packed snapshots: see the launch code (rev_search).
#pragma once

#include "im_bfs.h"

struct RevArgs {
    // reverse graph and its per-snapshot live lists
    const uint32_t *row;      // [n+1]
    const uint32_t *col;      // [m]
    const uint64_t *mask;     // [W][m]
    uint64_t m;
    uint32_t n, W;
    HubLists hub;
    SparseLists sp;
    const uint32_t *node_inst;  // batches: instance of each node (nullptr: one graph)
    const uint32_t *inst_off;   // batches: first node of each instance
    // the round's sources, sorted by bin, and its tasks (RevTask)
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

// where the heads of x's reverse arcs live in snapshot 64w + b are: kind 0
// the sparse lists, 1 the hub lists, 2 the arcs themselves (heads whose mask
// word has the bit)
struct RevSpan {
    uint32_t start, len, kind;
};

__device__ __forceinline__ RevSpan rev_span(const RevArgs &a, uint32_t w, uint32_t b, uint32_t x)
{
    const uint64_t p = (uint64_t)w * a.n + x;
    // independent loads; the counts of a node without lists are not used
    const uint16_t *c = a.sp.cum + p * 65 + b;
    const uint32_t rs = a.row[x], re = a.row[x + 1], base = a.sp.base[p];
    const uint32_t c0 = c[0], c1 = c[1], deg = re - rs;
    RevSpan s;
    if (base != IM_EMPTY) {
        s.start = base + c0; s.len = c1 - c0; s.kind = 0;
        return s;
    }
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
__device__ __forceinline__ bool rev_head(const RevArgs &a, uint32_t w, uint32_t b, uint32_t kind,
                                         uint32_t pos, uint32_t &v)
{
    const uint32_t *heads = kind == 0 ? a.sp.adj : kind == 1 ? a.hub.adj : a.col;
    v = heads[pos];
    return kind != 2 || ((a.mask[(uint64_t)w * a.m + pos] >> b) & 1ull);
}

constexpr int REV_SMALL = 4;   // spans up to this length are expanded by one lane
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
__device__ __forceinline__ void rev_expand(RevBig<NT> &B, const RevArgs &a, uint32_t w, uint32_t b,
                                           bool take, uint32_t own, const RevSpan &sp, Relax relax,
                                           uint64_t &arcs)
{
    const int tid = threadIdx.x;
    const bool small = take && sp.len <= (uint32_t)REV_SMALL, big = take && !small;
    if (small) {
        uint32_t v[REV_SMALL];
        bool live[REV_SMALL];
#pragma unroll
        for (int u = 0; u < REV_SMALL; u++) {
            v[u] = 0;
            live[u] = (uint32_t)u < sp.len && rev_head(a, w, b, sp.kind, sp.start + (uint32_t)u, v[u]);
        }
#pragma unroll
        for (int u = 0; u < REV_SMALL; u++)
            if (live[u]) relax(own, v[u]);
        arcs += sp.len;
    }
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
                sp = rev_span(a, w, b, L.keys[idx]);
            }
            // a longer span's delta is looked up by its owner: the bits taken
            // above are part of reach, and passing on bits of reach that are
            // still pending only brings them forward
            rev_expand<NT>(L.B, a, w, b, take, idx, sp,
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
            const uint32_t pc = (uint32_t)__popcll(L.reach[i]), dg = a.row[key + 1] - a.row[key];
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
                sp = rev_span(a, w, b, x);
            }
            rev_expand<NT>(B, a, w, b, take, x - base0, sp,
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
        const uint32_t pc = (uint32_t)__popcll(*r), dg = a.row[x + 1] - a.row[x];
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
        const uint2 tk = a.tasks[id];
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
// The round's sources. A bin is one snapshot of one instance: (inst * W + w)
// * 64 + b. The forward search counts the pairs per bin (batches: k_rev_count).
// ---------------------------------------------------------------------------
constexpr int RVP_NT = 1024;

// One workgroup: bin starts (into cur, the fill's cursors), the task list and
// its length; the bin counts return to zero.
__global__ __launch_bounds__(RVP_NT) void k_rev_plan(uint32_t *cnt, uint32_t *cur, uint32_t nbins,
                                                     uint32_t W, uint2 *tasks, uint32_t *ntasks,
                                                     const unsigned long long *key, uint64_t aff_gain)
{
    __shared__ uint32_t s_w[RVP_NT / 64 + 1], s_t[RVP_NT], s_o[RVP_NT], s_c[RVP_NT];
    const int tid = threadIdx.x;
    // a round updated by the affected-set recompute has no reverse tasks
    const bool none = aff_gain && (*key >> 32) < aff_gain;
    uint32_t off0 = 0, t0 = 0;
    for (uint32_t base = 0; base < nbins; base += RVP_NT) {
        const uint32_t i = base + tid;
        const uint32_t c = i < nbins ? cnt[i] : 0u;
        if (c) cnt[i] = 0;
        uint32_t tot, tt;
        const uint32_t o = off0 + block_excl_scan<RVP_NT>(c, s_w, &tot);
        const uint32_t te = block_excl_scan<RVP_NT>((c + 63) / 64, s_w, &tt);
        if (i < nbins) cur[i] = o;
        s_t[tid] = te; s_o[tid] = o; s_c[tid] = c;
        __syncthreads();
        // the tile's tasks, spread over the threads
        for (uint32_t t = tid; t < tt && !none; t += RVP_NT) {
            const uint32_t k = (uint32_t)upper_index<RVP_NT>(s_t, t), g = t - s_t[k], bin = base + k;
            tasks[t0 + t] = rev_task(s_o[k] + 64u * g, min(64u, s_c[k] - 64u * g), bin & 63u,
                                     (bin >> 6) % W);
        }
        off0 += tot;
        t0 += tt;
        __syncthreads();
    }
    if (tid == 0) *ntasks = none ? 0u : t0;
}

// batches: the newly covered pairs per bin
__global__ __launch_bounds__(256) void k_rev_count(const uint32_t *tnodes, const uint32_t *tcounts,
                                                   const uint64_t *newly, uint32_t n, uint32_t W,
                                                   const uint32_t *node_inst, uint32_t *cnt)
{
    const uint32_t w = blockIdx.y, c = tcounts[w];
    const uint64_t off = (uint64_t)w * n;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < c; i += gridDim.x * 256u) {
        const uint32_t x = tnodes[off + i];
        uint32_t *bins = cnt + ((uint64_t)node_inst[x] * W + w) * 64;
        for (uint64_t b = newly[off + x]; b; b &= b - 1)
            atomicAdd(&bins[__ffsll((unsigned long long)b) - 1], 1u);
    }
}

// Place the sources: src[cur[bin]++] = node. One graph: each workgroup counts
// its pairs per bit in LDS and takes one range of every bin; batches: one
// atomic per pair on the bins of many instances.
__global__ __launch_bounds__(256) void k_rev_fill(const uint32_t *tnodes, const uint32_t *tcounts,
                                                  const uint64_t *newly, uint32_t n, uint32_t W,
                                                  const uint32_t *node_inst, uint32_t *cur,
                                                  uint32_t *src)
{
    __shared__ uint32_t cnt[64];
    const uint32_t w = blockIdx.y, c = tcounts[w], tid = threadIdx.x;
    const uint64_t off = (uint64_t)w * n;
    if (node_inst) {
        for (uint32_t i = blockIdx.x * 256u + tid; i < c; i += gridDim.x * 256u) {
            const uint32_t x = tnodes[off + i];
            uint32_t *bins = cur + ((uint64_t)node_inst[x] * W + w) * 64;
            for (uint64_t b = newly[off + x]; b; b &= b - 1)
                src[atomicAdd(&bins[__ffsll((unsigned long long)b) - 1], 1u)] = x;
        }
        return;
    }
    for (uint32_t base = blockIdx.x * 256u; base < c; base += gridDim.x * 256u) {
        if (tid < 64) cnt[tid] = 0;
        __syncthreads();
        const uint32_t i = base + tid;
        const uint32_t x = i < c ? tnodes[off + i] : 0u;
        const uint64_t bits = i < c ? newly[off + x] : 0ull;
        for (uint64_t b = bits; b; b &= b - 1) atomicAdd(&cnt[__ffsll((unsigned long long)b) - 1], 1u);
        __syncthreads();
        if (tid < 64 && cnt[tid]) cnt[tid] = atomicAdd(&cur[w * 64 + tid], cnt[tid]);
        __syncthreads();
        for (uint64_t b = bits; b; b &= b - 1)
            src[atomicAdd(&cnt[__ffsll((unsigned long long)b) - 1], 1u)] = x;
        __syncthreads();
    }
}
