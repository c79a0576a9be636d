// im_lt.h -- the dynamic update on linear-threshold snapshots.
//
// A linear-threshold snapshot keeps at most one in-arc per node (the tail of
// that arc is the node's parent), so its live arcs form trees and, at most one
// per component, a cycle with trees hanging from it. What a node reaches is
// its subtree (a node on a cycle reaches its whole component), so nothing has
// to be searched:
//   initial gains   subtree sizes, one walk up from every leaf in which the
//                   last child to arrive at a node goes on (k_lt_up), then
//                   the cycles (k_lt_cycle);
//   forward step    with the nodes of a snapshot in preorder a subtree is an
//                   interval (k_lt_order); its uncovered nodes are the newly
//                   covered ones;
//   reverse step    cur, |R_r(y) \ covered| of every node, falls to zero on the
//                   interval and by cur[r][v*] on the ancestors of v*
//                   (k_lt_round).
// That is O(n) per snapshot and O(newly covered + depth) per round and
// snapshot, where the general engines follow every ancestor chain (measured:
// see lt_forest). The kernels are bound by random accesses to per-snapshot
// arrays of n words.
#pragma once

#include "im_bfs.h"

constexpr uint32_t LT_NONE = 0xFFFFFFFFu;

// floor(prob[e] * 2^32): the length of arc e's draw interval
__device__ __forceinline__ uint64_t lt_len(const float *prob, uint32_t e)
{
    return (uint64_t)((double)prob[e] * 4294967296.0);
}

// ---------------------------------------------------------------------------
// In-rows by increasing arc id, with the start of every arc's interval (the
// lengths before it, added up). Rows of up to 64 in-arcs take one wavefront,
// which ranks them in registers; larger ones are listed and sorted by a
// workgroup each (k_lt_sort_big).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_lt_sort_small(const uint32_t *in_row, uint32_t *in2out,
                                                       uint32_t *in_col, const float *prob,
                                                       uint32_t n, uint64_t *start, uint32_t *big,
                                                       uint32_t *nbig)
{
    const uint32_t lane = threadIdx.x & 63;
    for (uint32_t v = blockIdx.x * 4 + (threadIdx.x >> 6); v < n; v += gridDim.x * 4) {
        const uint32_t a = in_row[v], d = in_row[v + 1] - a;
        if (d > 64) {
            if (lane == 0) big[atomicAdd(nbig, 1u)] = v;
            continue;
        }
        const bool in = lane < d;
        const uint32_t id = in ? in2out[a + lane] : LT_NONE, tail = in ? in_col[a + lane] : 0u;
        const uint64_t len = in ? lt_len(prob, id) : 0ull;
        uint32_t rank = 0;
        uint64_t acc = 0;
        for (uint32_t q = 0; q < d; q++) {
            const uint32_t o = __shfl(id, (int)q, 64);
            const uint64_t l = __shfl(len, (int)q, 64);
            if (o < id) { rank++; acc += l; }
        }
        if (in) { in2out[a + rank] = id; in_col[a + rank] = tail; start[a + rank] = acc; }
    }
}

constexpr int LTS_NT = 512;

// One workgroup per large row: least-significant-digit radix sort of (arc id,
// tail) on 8-bit digits, between the two id / tail arrays and the row's part
// of `start` (one packed word per arc), then the interval starts. Stable: a
// wavefront ranks its equal digits by ballots, wavefronts follow in order.
__global__ __launch_bounds__(LTS_NT) void k_lt_sort_big(const uint32_t *in_row, uint32_t *in2out,
                                                        uint32_t *in_col, const float *prob,
                                                        uint64_t *start, const uint32_t *big,
                                                        const uint32_t *nbig, int passes)
{
    constexpr int NW = LTS_NT / 64;
    __shared__ uint32_t base[256], wcnt[NW][256], s_w[NW + 1];
    __shared__ uint64_t s_l[NW], carry;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const uint32_t nb = *nbig;
    for (uint32_t q = blockIdx.x; q < nb; q += gridDim.x) {
        const uint32_t v = big[q], a = in_row[v], d = in_row[v + 1] - a;
        for (int pass = 0; pass < passes; pass++) {
            const bool packed = pass & 1;   // the source of this pass
            auto get = [&](uint32_t i, uint32_t &id, uint32_t &tail) {
                if (packed) {
                    const uint64_t x = start[a + i];
                    id = (uint32_t)x; tail = (uint32_t)(x >> 32);
                } else {
                    id = in2out[a + i]; tail = in_col[a + i];
                }
            };
            if (tid < 256) base[tid] = 0;
            __syncthreads();
            for (uint32_t i = tid; i < d; i += LTS_NT) {
                uint32_t id, tail;
                get(i, id, tail);
                atomicAdd(&base[(id >> (8 * pass)) & 255u], 1u);
            }
            __syncthreads();
            {
                uint32_t tot;
                const uint32_t c = tid < 256 ? base[tid] : 0u;
                const uint32_t ex = block_excl_scan<LTS_NT>(c, s_w, &tot);
                if (tid < 256) base[tid] = ex;
            }
            __syncthreads();
            for (uint32_t i0 = 0; i0 < d; i0 += LTS_NT) {
                const uint32_t i = i0 + tid;
                const bool in = i < d;
                uint32_t id = 0, tail = 0;
                if (in) get(i, id, tail);
                const uint32_t dg = (id >> (8 * pass)) & 255u;
                for (int j = tid; j < NW * 256; j += LTS_NT) (&wcnt[0][0])[j] = 0;
                uint64_t same = __ballot(in);
#pragma unroll
                for (int b = 0; b < 8; b++) {
                    const uint64_t one = __ballot((dg >> b) & 1u);
                    same &= ((dg >> b) & 1u) ? one : ~one;
                }
                const uint32_t rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
                __syncthreads();
                if (in && rank == 0) wcnt[wid][dg] = (uint32_t)__popcll(same);
                __syncthreads();
                if (tid < 256) {
                    uint32_t s = base[tid];
#pragma unroll
                    for (int w = 0; w < NW; w++) {
                        const uint32_t c = wcnt[w][tid];
                        wcnt[w][tid] = s;
                        s += c;
                    }
                    base[tid] = s;
                }
                __syncthreads();
                if (in) {
                    const uint32_t to = a + wcnt[wid][dg] + rank;
                    if (packed) { in2out[to] = id; in_col[to] = tail; }
                    else start[to] = (uint64_t)id | ((uint64_t)tail << 32);
                }
                __syncthreads();
            }
        }
        if (passes & 1)
            for (uint32_t i = tid; i < d; i += LTS_NT) {
                const uint64_t x = start[a + i];
                in2out[a + i] = (uint32_t)x;
                in_col[a + i] = (uint32_t)(x >> 32);
            }
        if (tid == 0) carry = 0;
        __syncthreads();
        for (uint32_t i0 = 0; i0 < d; i0 += LTS_NT) {
            const uint32_t i = i0 + tid;
            const uint64_t len = i < d ? lt_len(prob, in2out[a + i]) : 0ull;
            uint64_t incl = len;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint64_t y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            if (lane == 63) s_l[wid] = incl;
            __syncthreads();
            uint64_t before = carry, all = 0;
            for (int w = 0; w < NW; w++) {
                if (w < wid) before += s_l[w];
                all += s_l[w];
            }
            if (i < d) start[a + i] = before + incl - len;
            __syncthreads();
            if (tid == 0) carry += all;
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// The forest of every snapshot. Arrays [R][n] (snapshot-major):
//   par   parent of each node (LT_NONE: none; a kept self-loop is a cycle)
//   sc    children that have not arrived << 32 | subtree size so far; at the
//         end a non-zero upper half marks a node on a cycle, whose size is its
//         component's
//   cur   sum of out-degrees over each node's subtree, then |R_r(y) \ covered|
//         of the node at each position
//   pos   preorder position; on the way there, offset from an ancestor | ancestor << 32
//   ord   node at each position
// ---------------------------------------------------------------------------
struct LtForest {
    uint32_t n, R;
    uint32_t *par, *cur, *ord;
    unsigned long long *sc, *pos;
};

// A grid of lt_grid(nb, rows) workgroups walks the rows eight at a time, each on
// one XCD (consecutive workgroups go to consecutive XCDs), so that a row's
// scattered accesses meet in one L2 (k_lt_up 6.7 -> 5.7 ms, k_lt_parent 3.2 ->
// 2.8, 200,000 nodes, R = 256). False: past the last row. (64 bits: the launches'
// lanes stay below 2^32, see reserve_lt.)
constexpr uint32_t LT_XCDS = 8;

__host__ __device__ __forceinline__ uint64_t lt_grid(uint32_t nb, uint32_t rows)
{
    return (uint64_t)nb * ((rows + LT_XCDS - 1) / LT_XCDS * LT_XCDS);
}

__device__ __forceinline__ bool lt_place(uint32_t nb, uint32_t rows, uint32_t &block, uint32_t &row)
{
    const uint32_t i = blockIdx.x / LT_XCDS;
    block = i % nb;
    row = i / nb * LT_XCDS + blockIdx.x % LT_XCDS;
    return row < rows;
}

// The lanes of a wavefront with this lane's parent p (LT_NONE: none): all of them
// as a mask, itself among them; group(mask) is called by the whole wavefront for
// each of several lanes. A hub that keeps thousands of children in a snapshot has
// their additions queue at its words otherwise (R = 256, k_lt_up: a star of
// 200,000 arcs kept half the time 42.7 -> 1.4 ms, ten hubs with their leaves dealt
// in turn 11.9 -> 2.6). Parents are looked for as long as lanes share them:
// LT_SINGLE lanes that are alone end it.
constexpr int LT_SINGLE = 2;

template <typename Group>
__device__ __forceinline__ uint64_t lt_same_parent(uint32_t p, Group group)
{
    uint64_t left = __ballot(p != LT_NONE), mine = 1ull << (threadIdx.x & 63u);
    for (int single = 0; left && single < LT_SINGLE;) {
        const int lead = __ffsll((unsigned long long)left) - 1;
        const uint64_t same = __ballot(p == (uint32_t)__builtin_amdgcn_readlane((int)p, lead));
        left &= ~same;
        if (same & (same - 1)) group(same);
        else single++;
        if (same & mine) mine = same;
    }
    return mine;
}

// Each thread draws its node's kept in-arc in LTP_R snapshots: the largest j
// with start[j] <= draw (an arc of length zero shares its start with the next
// one, which comes later), if the draw lies in that arc's interval.
constexpr int LTP_R = 8;

__global__ __launch_bounds__(256) void k_lt_parent(const uint32_t *row, const uint32_t *in_row,
                                                   const uint32_t *in2out, const uint32_t *in_col,
                                                   const float *prob, const uint64_t *start,
                                                   uint64_t seed, LtForest f)
{
    uint32_t block, rows;
    if (!lt_place((f.n + 255) / 256, (f.R + LTP_R - 1) / LTP_R, block, rows)) return;
    const uint32_t v = block * 256u + threadIdx.x, r0 = rows * LTP_R;
    const bool in = v < f.n;
    const uint32_t a = in ? in_row[v] : 0u, b = in ? in_row[v + 1] : 0u;
    const uint32_t dg = in ? row[v + 1] - row[v] : 0u;
    const uint64_t key = sm64_finalise(seed + ((uint64_t)v + 1ull) * IM_GOLDEN);
    for (uint32_t r = r0; r < min(r0 + (uint32_t)LTP_R, f.R); r++) {
        uint32_t p = LT_NONE;
        if (a != b) {
            const uint64_t d = sm64_finalise(key + ((uint64_t)r + 1ull) * IM_GOLDEN) >> 32;
            uint32_t lo = a, hi = b;
            while (hi - lo > 1) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if (start[mid] <= d) lo = mid; else hi = mid;
            }
            if (d - start[lo] < lt_len(prob, in2out[lo])) p = in_col[lo];
        }
        const uint64_t at = (uint64_t)r * f.n + v;
        if (in) {
            f.par[at] = p;
            f.cur[at] = dg;
        }
        unsigned long long *sc = f.sc + (uint64_t)r * f.n;
        const uint32_t lane = threadIdx.x & 63u;
        const uint64_t same = lt_same_parent(p, [](uint64_t) {});
        if (p != LT_NONE && (uint32_t)__ffsll((unsigned long long)same) == lane + 1)
            atomicAdd(&sc[p], (unsigned long long)__popcll(same) << 32);
    }
}

// Subtree sizes and degree sums. Only a leaf's word is exactly 1 (size 1, no
// children; a node whose children have arrived holds more), so every walk
// starts once. One atomic on the parent's word adds the size, tells the
// offset of this subtree behind its parent (the size so far) and whether it
// was the last child.
__global__ __launch_bounds__(256) void k_lt_up(LtForest f)
{
    uint32_t block, r;
    if (!lt_place((f.n + 255) / 256, f.R, block, r)) return;
    const uint32_t u = block * 256u + threadIdx.x, lane = threadIdx.x & 63u;
    const uint64_t off = (uint64_t)r * f.n;
    const bool leaf = u < f.n && f.sc[off + u] == 1ull;
    uint32_t v = u, size = 1, degs = leaf ? f.cur[off + u] : 0u;
    uint32_t p = leaf ? f.par[off + u] : LT_NONE;   // (LT_NONE: the walk has ended)
    // `kids` subtrees of `nodes` nodes and degree sum `sum` in all arrive at p:
    // what was there before. The degree sum is in place before they count as
    // arrived: what it is added to comes back first, and the second addition
    // waits for that value. (Whoever counts the last child reads the sum by an
    // atomic too. A release and acquire of the whole memory instead writes the L2
    // back at every step: 5.6 -> 73 ms, 200,000 nodes, R = 256.)
    auto arrive = [&](uint32_t kids, uint32_t nodes, uint32_t sum) -> unsigned long long {
        const uint32_t before = atomicAdd(&f.cur[off + p], sum);
        asm volatile("" : "+v"(nodes) : "v"(before));
        return atomicAdd(&f.sc[off + p], (unsigned long long)nodes - ((unsigned long long)kids << 32));
    };
    // on from p if all its children have arrived with these
    auto climb = [&](unsigned long long old, uint32_t kids, uint32_t nodes) {
        if ((old >> 32) == kids) {
            size = (uint32_t)old + nodes;
            degs = atomicAdd(&f.cur[off + p], 0u);
            v = p;
            p = f.par[off + v];
        } else {
            p = LT_NONE;   // other children are still to come
        }
    };
    // leaves of one parent arrive together, the first of them for all
    uint32_t sum = degs;
    const uint64_t same = lt_same_parent(p, [&](uint64_t g) {
        const bool in = (g >> lane) & 1ull;
        const uint32_t all = (uint32_t)wave_sum_u64(in ? degs : 0u);
        if (in) sum = all;
    });
    const uint32_t kids = (uint32_t)__popcll(same), lead = (uint32_t)__ffsll((unsigned long long)same) - 1;
    const bool first = lane == lead;
    unsigned long long old = 0;
    if (p != LT_NONE && first) old = arrive(kids, kids, sum);
    old = __shfl(old, (int)lead, 64);
    if (p != LT_NONE) {
        f.pos[off + v] = ((old & 0xFFFFFFFFull) + (uint32_t)__popcll(same & ((1ull << lane) - 1ull))) |
                         ((unsigned long long)p << 32);
        if (first) climb(old, kids, kids);
        else p = LT_NONE;
    }
    while (p != LT_NONE) {
        old = arrive(1, size, degs);
        f.pos[off + v] = (old & 0xFFFFFFFFull) | ((unsigned long long)p << 32);
        climb(old, 1, size);
    }
}

// Cycles: the nodes left with one child to come. The node of the smallest
// hash is the leader (a walk stops at the first smaller one, after O(log
// length) steps on average); it is made the root of the component.
__device__ __forceinline__ uint64_t lt_order_key(uint32_t v)
{
    return ((uint64_t)(v * 0x9E3779B1u ^ (v >> 15)) << 32) | v;
}

__global__ __launch_bounds__(256) void k_lt_cycle(LtForest f)
{
    const uint32_t c = blockIdx.x * 256u + threadIdx.x;
    if (c >= f.n) return;
    const uint64_t off = (uint64_t)blockIdx.y * f.n;
    if ((f.sc[off + c] >> 32) == 0) return;
    const uint64_t mine = lt_order_key(c);
    for (uint32_t y = f.par[off + c]; y != c; y = f.par[off + y])
        if (lt_order_key(y) < mine) return;
    // the arc into the leader is cut: what hangs from each node goes to the next
    uint32_t v = f.par[off + c];
    uint32_t size = (uint32_t)f.sc[off + v], degs = f.cur[off + v];
    while (v != c) {
        const uint32_t p = f.par[off + v];
        const uint32_t sp = (uint32_t)f.sc[off + p];
        f.pos[off + v] = (unsigned long long)sp | ((unsigned long long)p << 32);
        size += sp;
        degs += f.cur[off + p];
        v = p;
    }
    // every node on the cycle reaches the component (the mark stays)
    v = c;
    do {
        f.sc[off + v] = (1ull << 32) | size;
        f.cur[off + v] = degs;
        v = f.par[off + v];
    } while (v != c);
    f.pos[off + c] = (unsigned long long)LT_NONE << 32;   // placed with the roots
}

// Positions. Roots (and cycle leaders) take consecutive ranges; a node's
// position is the sum of the offsets on its way up, found by pointer jumping
// in place: a word always holds a true (offset, ancestor) pair, whichever of
// its values a reader sees. One workgroup per snapshot.
constexpr int LTO_NT = 1024, LTO_U = 4;

__global__ __launch_bounds__(LTO_NT) void k_lt_order(LtForest f)
{
    __shared__ uint32_t s_w[LTO_NT / 64 + 1];
    const int tid = threadIdx.x;
    const uint64_t off = (uint64_t)blockIdx.x * f.n;
    unsigned long long *pos = f.pos + off;
    const uint32_t *par = f.par + off;
    uint32_t used = 0;
    for (uint32_t v0 = 0; v0 < f.n; v0 += LTO_NT) {
        const uint32_t v = v0 + tid;
        bool root = false;
        uint32_t size = 0;
        if (v < f.n) {
            const unsigned long long s = f.sc[off + v];
            // a root has no parent, a leader no ancestor
            root = par[v] == LT_NONE || ((s >> 32) && (pos[v] >> 32) == LT_NONE);
            size = root ? (uint32_t)s : 0u;
        }
        uint32_t tot;
        const uint32_t ex = block_excl_scan<LTO_NT>(size, s_w, &tot);
        if (root) pos[v] = (unsigned long long)(used + ex) | ((unsigned long long)LT_NONE << 32);
        used += tot;
    }
    __syncthreads();
    for (;;) {
        int more = 0;
        for (uint32_t v0 = tid; v0 < f.n; v0 += LTO_NT * LTO_U) {
            unsigned long long x[LTO_U], y[LTO_U];
#pragma unroll
            for (int u = 0; u < LTO_U; u++) {
                const uint32_t v = v0 + (uint32_t)u * LTO_NT;
                x[u] = v < f.n && v >= v0 ? pos[v] : ~0ull;
            }
#pragma unroll
            for (int u = 0; u < LTO_U; u++)
                y[u] = (x[u] >> 32) != LT_NONE ? pos[x[u] >> 32] : 0ull;
#pragma unroll
            for (int u = 0; u < LTO_U; u++)
                if ((x[u] >> 32) != LT_NONE) {
                    pos[v0 + (uint32_t)u * LTO_NT] =
                        ((x[u] & 0xFFFFFFFFull) + (y[u] & 0xFFFFFFFFull)) | (y[u] & 0xFFFFFFFF00000000ull);
                    if ((y[u] >> 32) != LT_NONE) more = 1;
                }
        }
        if (!__syncthreads_or(more)) break;
    }
    for (uint32_t v = tid; v < f.n; v += LTO_NT) {
        const uint32_t p = (uint32_t)pos[v];
        f.ord[off + p] = v;
        f.cur[off + p] = (uint32_t)f.sc[off + v];
    }
}

// gain[v] = sum over r of the sizes (before k_lt_order takes over cur)
constexpr int LTG_R = 16;   // snapshots per workgroup

// ... and both degrees of a node in one word pair, for the rounds
__global__ __launch_bounds__(256) void k_lt_gain(LtForest f, const uint32_t *row, const uint32_t *in_row,
                                                 uint32_t *gain, uint2 *deg, unsigned long long *stats)
{
    __shared__ unsigned long long red[4];
    const uint32_t v = blockIdx.x * 256u + threadIdx.x, r0 = blockIdx.y * LTG_R;
    uint64_t trav = 0;
    uint32_t g = 0;
    if (v < f.n) {
        if (r0 == 0) deg[v] = make_uint2(row[v + 1] - row[v], in_row[v + 1] - in_row[v]);
#pragma unroll 4
        for (uint32_t r = r0; r < min(r0 + (uint32_t)LTG_R, f.R); r++) {
            const uint64_t at = (uint64_t)r * f.n + v;
            const uint32_t s = (uint32_t)f.sc[at];
            trav += f.cur[at];
            g += s;
        }
        atomicAdd(&gain[v], g);
    }
    trav = group_sum<256>(trav, red);
    if (threadIdx.x == 0) atomicAdd(&stats[((blockIdx.x + blockIdx.y) % ST_STRIPES) * ST_COUNT + ST_TRAV_INIT],
                                    (unsigned long long)trav);
}

// One round in one snapshot per workgroup: commit the argmax, bring cur and
// the gains up to date. stamp[W][n]: the last round (plus one) that newly
// covered the node in the word, for the (node, word) counters. Bound: early
// rounds by the scattered accesses of each newly covered node (its degrees in
// one load instead of four, and four nodes' loads and exchanges in flight: 7.4 ->
// 6.4 ms for 50 rounds on 200,000 nodes), late ones by the chain of parents
// (followed beside the interval, not before it: 1.07 -> 0.79 ms for 50 rounds on
// 15,000 nodes).
constexpr int LTR_NT = 1024, LTR_U = 4;

__global__ __launch_bounds__(LTR_NT) void k_lt_round(LtForest f, const uint2 *deg,
                                                     const unsigned long long *key, uint32_t t,
                                                     uint32_t *seeds_out, uint64_t *gains_out,
                                                     uint8_t *sel, uint32_t *gain, uint32_t *stamp,
                                                     unsigned long long *stats)
{
    __shared__ unsigned long long red[LTR_NT / 64];
    __shared__ uint32_t s_first;
    const int tid = threadIdx.x;
    const unsigned long long k = *key;
    if (k == 0) return;
    const uint32_t v = 0xFFFFFFFFu - (uint32_t)(k & 0xFFFFFFFFull), r = blockIdx.x;
    if (r == 0 && tid == 0) {
        seeds_out[t] = v;
        gains_out[t] = k >> 32;
        sel[v] = 1;
    }
    const uint64_t off = (uint64_t)r * f.n;
    const uint32_t at = (uint32_t)f.pos[off + v];
    const uint32_t c = f.cur[off + at];
    if (c == 0) return;   // covered in this snapshot
    // every wavefront has read c before one of them clears it: it is the first
    // word of the interval, and a wavefront that found it cleared would leave
    // its share of the interval, or the ancestors, as they are
    __syncthreads();
    uint64_t trav_fwd = 0, relax_fwd = 0, tasks = 0, trav_rev = 0, dec = 0;
    const unsigned long long own = f.sc[off + v];
    uint32_t first = at;
    if (own >> 32) {
        // on a cycle: the whole component, whose root has the first position
        if (tid == 0) {
            for (uint32_t y = f.par[off + v]; y != v; y = f.par[off + y])
                first = min(first, (uint32_t)f.pos[off + y]);
            s_first = first;
        }
        __syncthreads();
        first = s_first;
    } else if (tid < 64) {
        // an ancestor of v reaches all that v newly covers: the first wavefront
        // follows the parents, one load after the other, and takes 64 of them at
        // a time, while the others pass over the interval (no ancestor is in it)
        uint32_t mine = 0, cnt = 0, y0 = LT_NONE;
        auto shrink = [&]() {
            if ((uint32_t)tid < cnt) {
                f.cur[off + (uint32_t)f.pos[off + mine]] -= c;
                atomicSub(&gain[mine], c);
                dec += c;
                trav_rev += (uint64_t)c * deg[mine].y;
            }
            cnt = 0;
        };
        for (uint32_t y = f.par[off + v]; y != LT_NONE;) {
            const uint32_t p = f.par[off + y];
            if (f.sc[off + y] >> 32) {   // once round the cycle
                if (y == y0) break;
                if (y0 == LT_NONE) y0 = y;
            }
            if ((uint32_t)tid == cnt) mine = y;
            if (++cnt == 64) shrink();
            y = p;
        }
        shrink();
    }
    const uint32_t len = (uint32_t)own, w = r / 64;
    // most of a later seed's interval is covered already: cur is kept by
    // position, so passing over it reads consecutive words
    constexpr uint32_t ST = LTR_NT - 64;
    for (uint32_t i0 = (uint32_t)tid - 64u; tid >= 64 && i0 < len; i0 += ST * LTR_U) {
        uint32_t cx[LTR_U], x[LTR_U];
#pragma unroll
        for (int u = 0; u < LTR_U; u++) {
            const uint32_t i = i0 + (uint32_t)u * ST;
            cx[u] = i < len && i >= i0 ? f.cur[off + first + i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < LTR_U; u++)
            x[u] = cx[u] ? f.ord[off + first + i0 + (uint32_t)u * ST] : 0u;
        uint32_t last[LTR_U];
        uint2 dg[LTR_U];
#pragma unroll
        for (int u = 0; u < LTR_U; u++) {
            last[u] = t + 1;
            dg[u] = make_uint2(0, 0);
            if (cx[u] == 0) continue;
            last[u] = atomicExch(&stamp[(uint64_t)w * f.n + x[u]], t + 1);
            dg[u] = deg[x[u]];
        }
#pragma unroll
        for (int u = 0; u < LTR_U; u++) {
            if (cx[u] == 0) continue;
            f.cur[off + first + i0 + (uint32_t)u * ST] = 0;
            atomicSub(&gain[x[u]], cx[u]);
        }
#pragma unroll
        for (int u = 0; u < LTR_U; u++) {
            trav_fwd += dg[u].x;
            dec += cx[u];
            trav_rev += (uint64_t)cx[u] * dg[u].y;
            if (last[u] != t + 1) { relax_fwd += dg[u].x; tasks++; }
        }
    }
    trav_fwd = group_sum<LTR_NT>(trav_fwd, red);
    relax_fwd = group_sum<LTR_NT>(relax_fwd, red);
    tasks = group_sum<LTR_NT>(tasks, red);
    trav_rev = group_sum<LTR_NT>(trav_rev, red);
    dec = group_sum<LTR_NT>(dec, red);
    if (tid == 0) {
        stat_add(stats, ST_TRAV_FWD, trav_fwd);
        stat_add(stats, ST_RELAX_FWD, relax_fwd);
        stat_add(stats, ST_TASKS_REV, tasks);
        stat_add(stats, ST_TRAV_REV, trav_rev);
        stat_add(stats, ST_DECREMENTS, dec);
    }
}
