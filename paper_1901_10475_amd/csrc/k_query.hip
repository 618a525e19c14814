// k_query.hip -- the n-to-n self-traversal and the canonical pair list.
//
// One lane per leaf (query box), leaves taken in sorted key order so that the
// lanes of a wave hold neighbouring boxes and walk nearly the same nodes.  A
// query visits only the part of the tree to the right of its own leaf: it
// starts at its leaf's skip link (the next node in pre-order after the leaf)
// and follows, without a stack, the left-child link into overlapping inner
// nodes and the skip link past everything else.  Every unordered pair of
// leaves is therefore tested once, from the left one.  The node test is the
// 4D overlap of Def. 4D Occupancy Region: half-open integer time tags and
// closed spatial extents; leaves of the same object are skipped, as queryObject
// excludes the queried object (Sec. 4.4).
//
// Because keys are time-major, everything right of a node whose earliest tag
// starts at t0 begins no earlier than slab(t0) * slab_ticks, so a query stops as
// soon as t0_min(node) >= t1(query) + slab_ticks - 1.
//
// Records are appended through one atomic per wave per step: the lanes with a
// hit are counted with a ballot, the lowest one reserves the range, and each
// lane writes at its prefix position.
#include "cd_internal.h"

namespace cd {

static inline unsigned nblk(uint64_t n, unsigned t) { return (unsigned)((n + t - 1) / t); }

#ifdef CD_COUNTERS
// Executed-work counters of the traversal (the diagnostic build only), in the
// order of cd_counters: box-box tests, tests of two leaves, tests of a leaf
// and an inner node, tests of two overlapping leaves of different objects
// (each one appended record), node pairs expanded, per-leaf walk steps.  Per
// object: tests with a leaf box of that object on one side (g_visits, when
// the caller bound an array).
__device__ unsigned long long g_ctr[kCounterWords];
__device__ uint32_t *g_visits;
__device__ uint32_t g_nobj;

// Wave sum, one atomic per wave; every lane of the wave must call it.
__device__ inline void ctr_wave_add(int k, uint32_t v)
{
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0 && v)
        atomicAdd(&g_ctr[k], (unsigned long long)v);
}

__device__ inline void ctr_visit(uint32_t obj)
{
    uint32_t *vis = g_visits;
    if (vis && obj < g_nobj)
        atomicAdd(&vis[obj], 1u);
}
#endif

template <int TP>
struct Q;

template <>
struct Q<CD_FP64> {
    using F = double;
    __device__ static void load(const void *tree, uint32_t N, uint32_t id, F lo[3], F hi[3],
                                uint32_t &t0, uint32_t &t1, uint32_t &link, uint32_t &esc)
    {
        const Node64 *n = (const Node64 *)tree + id;
        double4 a = *(const double4 *)&n->lo[0];   // lo0 lo1 lo2 hi0
        double2 c = *(const double2 *)&n->hi[1];   // hi1 hi2
        uint4 u = *(const uint4 *)&n->t0;          // t0 t1 link esc
        lo[0] = a.x;
        lo[1] = a.y;
        lo[2] = a.z;
        hi[0] = a.w;
        hi[1] = c.x;
        hi[2] = c.y;
        t0 = u.x;
        t1 = u.y;
        link = u.z;
        esc = u.w;
    }
    // the box and tags alone (the links share the record's last 16 bytes)
    __device__ static void load_box(const void *tree, uint32_t N, uint32_t id, F lo[3],
                                    F hi[3], uint32_t &t0, uint32_t &t1)
    {
        uint32_t link, esc;
        load(tree, N, id, lo, hi, t0, t1, link, esc);
    }
};

template <>
struct Q<CD_FP32> {
    using F = float;
    __device__ static void load(const void *tree, uint32_t N, uint32_t id, F lo[3], F hi[3],
                                uint32_t &t0, uint32_t &t1, uint32_t &link, uint32_t &esc)
    {
        const Box32 *b = (const Box32 *)tree + id;
        float4 a = *(const float4 *)&b->lo[0];     // lo0 lo1 lo2 hi0
        uint4 c = *(const uint4 *)&b->hi[1];       // hi1 hi2 t0 t1
        uint2 l = *((const uint2 *)((const Box32 *)tree + (2 * (size_t)N - 1)) + id);
        lo[0] = a.x;
        lo[1] = a.y;
        lo[2] = a.z;
        hi[0] = a.w;
        hi[1] = __uint_as_float(c.x);
        hi[2] = __uint_as_float(c.y);
        t0 = c.z;
        t1 = c.w;
        link = l.x;
        esc = l.y;
    }
    // the box and tags alone: the link array is a second cache line
    __device__ static void load_box(const void *tree, uint32_t N, uint32_t id, F lo[3],
                                    F hi[3], uint32_t &t0, uint32_t &t1)
    {
        const Box32 *b = (const Box32 *)tree + id;
        float4 a = *(const float4 *)&b->lo[0];
        uint4 c = *(const uint4 *)&b->hi[1];
        lo[0] = a.x;
        lo[1] = a.y;
        lo[2] = a.z;
        hi[0] = a.w;
        hi[1] = __uint_as_float(c.x);
        hi[2] = __uint_as_float(c.y);
        t0 = c.z;
        t1 = c.w;
    }
};

// An FP64 tree built bottom-up keeps its leaf skip links in a side array
// (*side_on set by the build).
template <int TP>
__global__ __launch_bounds__(256) void k_traverse(const void *__restrict__ tree, uint32_t N,
                                                  uint32_t slab_ticks, Rec *__restrict__ out,
                                                  unsigned long long capacity,
                                                  unsigned long long *counter,
                                                  unsigned int *err, const unsigned int *run_if,
                                                  const unsigned int *side_on,
                                                  const uint32_t *__restrict__ side)
{
    using F = typename Q<TP>::F;
    if (run_if && *run_if == 0)
        return;
    const bool use_side = TP == CD_FP64 && side_on && *side_on;
    uint32_t blk = xcd_block(blockIdx.x, gridDim.x);
    uint32_t i = blk * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    F qlo[3], qhi[3];
    uint32_t qt0, qt1, qobj, node;
    Q<TP>::load(tree, N, N - 1 + i, qlo, qhi, qt0, qt1, qobj, node);
    if (use_side)
        node = side[i];
    const uint64_t stop = (uint64_t)qt1 + slab_ticks - 1;
    const uint32_t limit = 2 * N + 2;
    const uint64_t lt = (threadIdx.x & 63) ? (~0ull >> (64 - (threadIdx.x & 63))) : 0ull;
    uint32_t steps = 0;
#ifdef CD_COUNTERS
    uint32_t c_tests = 0, c_ll = 0, c_hits = 0;
#endif
    while (node != kEnd) {
        if (++steps > limit || node >= 2 * N - 1) {
            atomicOr(err, 4u);
            break;
        }
        F lo[3], hi[3];
        uint32_t t0, t1, link, esc;
        Q<TP>::load(tree, N, node, lo, hi, t0, t1, link, esc);
        if ((uint64_t)t0 >= stop)
            break;
        bool ov = time_overlap(qt0, qt1, t0, t1) && space_overlap(qlo, qhi, lo, hi);
        bool leaf = node >= N - 1;
#ifdef CD_COUNTERS
        ++c_tests;
        c_ll += leaf ? 1u : 0u;
        c_hits += (ov && leaf && link != qobj) ? 1u : 0u;
        ctr_visit(qobj);
        if (leaf)
            ctr_visit(link);
#endif
        if (use_side && leaf)
            esc = side[node - (N - 1)];
        bool hit = ov && leaf && link != qobj;
        uint64_t m = __ballot(hit);
        if (m) {
            int leader = __ffsll((unsigned long long)m) - 1;
            unsigned long long base = 0;
            if ((int)(threadIdx.x & 63) == leader)
                base = atomicAdd(counter, (unsigned long long)__popcll(m));
            base = __shfl(base, leader, 64);
            if (hit) {
                unsigned long long pos = base + (unsigned long long)__popcll(m & lt);
                if (pos < capacity) {
                    Rec r;
                    r.i = qobj < link ? qobj : link;
                    r.j = qobj < link ? link : qobj;
                    r.tlo = qt0 > t0 ? qt0 : t0;
                    r.thi = qt1 < t1 ? qt1 : t1;
                    out[pos] = r;
                }
            }
        }
        node = (ov && !leaf) ? link : esc;
    }
#ifdef CD_COUNTERS
    if (c_tests) {
        atomicAdd(&g_ctr[0], (unsigned long long)c_tests);
        atomicAdd(&g_ctr[1], (unsigned long long)c_ll);
        atomicAdd(&g_ctr[2], (unsigned long long)(c_tests - c_ll));
        atomicAdd(&g_ctr[3], (unsigned long long)c_hits);
        atomicAdd(&g_ctr[5], (unsigned long long)c_tests);
    }
#endif
}

hipError_t launch_traverse(const void *tree, int precision, uint32_t N, uint32_t slab_ticks,
                           Rec *out, unsigned long long capacity, unsigned long long *counter,
                           unsigned int *err, const unsigned int *run_if, uint32_t threads,
                           const unsigned int *side_on, const uint32_t *side, hipStream_t s)
{
    if (N <= 1)
        return hipSuccess;
    unsigned g = nblk(N, threads);
    if (precision == CD_FP64)
        k_traverse<CD_FP64><<<g, threads, 0, s>>>(tree, N, slab_ticks, out, capacity, counter,
                                                  err, run_if, side_on, side);
    else
        k_traverse<CD_FP32><<<g, threads, 0, s>>>(tree, N, slab_ticks, out, capacity, counter,
                                                  err, run_if, nullptr, nullptr);
    return hipGetLastError();
}

// ---- node-pair self-traversal ------------------------------------------------------------------
//
// The refit records every pair of sibling nodes whose 4D boxes overlap.  Every
// overlapping pair of leaves lies under exactly one such pair (the children of
// its lowest common ancestor), and expanding an overlapping node pair into the
// overlapping pairs of their children reaches each of those leaf pairs exactly
// once.  A lane takes one pair, loads the children's boxes, tests the (up to)
// four child pairs, emits leaf pairs as records and keeps the rest to expand.

// Lanes below this one in a ballot.
__device__ inline uint32_t lanes_before(uint64_t all)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
}

// A node in a queue, by its two children instead of its id, so that expanding
// it needs no look-up of its child pair (a cache line of its own): kind N + g
// for a node split after leaf g, bit 0 of the kind set if its left child is
// leaf g (else the inner node g), bit 1 if its right child is leaf g + 1 (else
// the inner node g + 1); 4 N + j for leaf j.  An FP64 record holds what this
// takes: link is the left child, and esc, the node that follows the subtree, is
// a right child and so numbered by its first leaf, the one after the node's
// last.  FP32 records keep their links in another array; their queues (and
// those of trees of more than kCodedLeaves leaves) hold ids.
constexpr uint32_t kCodedLeaves = 0xFFFFFFFFu / 5;

__device__ inline uint32_t node_code(uint32_t N, uint32_t id, uint32_t link, uint32_t esc)
{
    const bool left = link >= N - 1;
    const uint32_t g = link - (left ? N - 1 : 0u), j = esc - (esc >= N - 1 ? N - 1 : 0u),
                   after = esc == kEnd ? N : j, kind = (left ? 1u : 0u) + (g + 2 == after ? 2u : 0u);
    return id >= N - 1 ? 4 * N + (id - (N - 1)) : kind * N + g;
}

// The pairs of one wave, the lanes' (ids, active) in, its child pairs out:
// push bit 2 ia + ic for a pair to expand, hit for a record.  IN: the pairs
// come as ids (else codes); OUT: node holds ids (else codes).
template <int TP, bool IN, bool OUT>
struct PairTest {
    using F = typename Q<TP>::F;
    uint32_t node[2][2], t0[2][2], t1[2][2], lk[2][2];
    uint32_t push, hit;

    // Side s: a leaf stays itself (twice), an inner node is its two children.
    __device__ void run(const void *__restrict__ tree, const uint2 *__restrict__ kids,
                        uint32_t N, uint2 pr, bool active, unsigned int *flags)
    {
        static_assert(OUT || TP == CD_FP64, "codes come from FP64 records");
#ifdef CD_COUNTERS
        constexpr bool kLinks = true;   // the node-visit counts need every leaf's object
#else
        constexpr bool kLinks = TP == CD_FP64;   // FP32: object ids only for overlapping leaf pairs
#endif
        const uint32_t nodes = 2 * N - 1;
        uint32_t x[2] = {pr.x, pr.y}, ids[2][2];
        F lo[2][2][3], hi[2][2][3];
        bool one[2], ok = true;
        if (IN) {
            uint2 kk[2];
            for (int side = 0; side < 2; ++side) {   // both reads asked for together
                ok &= x[side] < nodes;
                one[side] = x[side] >= N - 1;
                kk[side] = kids[one[side] ? 0u : x[side]];
            }
            for (int side = 0; side < 2; ++side) {
                ids[side][0] = one[side] ? x[side] : kk[side].x;
                ids[side][1] = one[side] ? x[side] : kk[side].y;
            }
        } else {
            for (int side = 0; side < 2; ++side) {
                one[side] = x[side] >= 4 * N;
                const uint32_t r = x[side] >= 2 * N ? 1u : 0u, y = x[side] - 2 * N * r,
                               l = y >= N ? 1u : 0u, g = y - N * l;
                ids[side][0] = one[side] ? x[side] - 4 * N + (N - 1) : g + (l ? N - 1 : 0u);
                ids[side][1] = one[side] ? ids[side][0] : g + 1 + (r ? N - 1 : 0u);
            }
        }
        for (int side = 0; side < 2; ++side)
            ok &= (ids[side][0] < nodes) & (ids[side][1] < nodes);
        if (active && !ok)
            atomicOr(flags, 2u);
        active &= ok;
        uint32_t esc[2][2];
        for (int side = 0; side < 2; ++side)
            for (int c = 0; c < 2; ++c) {
                ids[side][c] = active ? ids[side][c] : 0u;
                if (kLinks)
                    Q<TP>::load(tree, N, ids[side][c], lo[side][c], hi[side][c], t0[side][c],
                                t1[side][c], lk[side][c], esc[side][c]);
                else
                    Q<TP>::load_box(tree, N, ids[side][c], lo[side][c], hi[side][c],
                                    t0[side][c], t1[side][c]);
            }
        if (!OUT)   // the four records are asked for before any is waited for
            asm volatile("" : "+v"(esc[0][0]), "+v"(esc[0][1]), "+v"(esc[1][0]), "+v"(esc[1][1]));
        for (int side = 0; side < 2; ++side)
            for (int c = 0; c < 2; ++c)
                node[side][c] = OUT ? ids[side][c]
                                    : node_code(N, ids[side][c], lk[side][c], esc[side][c]);
        const uint32_t first_leaf = OUT ? N - 1 : 4 * N;
        push = hit = 0;
        for (int ia = 0; ia < 2; ++ia)
            for (int ic = 0; ic < 2; ++ic) {
                // every comparison made, no branches
                const bool t = (t0[0][ia] < t1[1][ic]) & (t0[1][ic] < t1[0][ia]);
                bool ov = active & !(ia & (int)one[0]) & !(ic & (int)one[1]) & t;
                for (int d = 0; d < 3; ++d)
                    ov &= (lo[0][ia][d] <= hi[1][ic][d]) & (lo[1][ic][d] <= hi[0][ia][d]);
                const bool leaves =
                    ov & (node[0][ia] >= first_leaf) & (node[1][ic] >= first_leaf);
                const uint32_t bit = 1u << (ia * 2 + ic);
                if (!kLinks && leaves) {
                    const uint2 *links = (const uint2 *)((const Box32 *)tree + (2 * (size_t)N - 1));
                    lk[0][ia] = links[node[0][ia]].x;
                    lk[1][ic] = links[node[1][ic]].x;
                }
                hit |= (leaves & (lk[0][ia] != lk[1][ic])) ? bit : 0u;
                push |= (ov & !leaves) ? bit : 0u;
            }
#ifdef CD_COUNTERS
        uint32_t c_tests = 0, c_ll = 0, c_li = 0;
        for (int ia = 0; ia < 2; ++ia)
            for (int ic = 0; ic < 2; ++ic) {
                if (!active || (ia && one[0]) || (ic && one[1]))
                    continue;
                const bool la = node[0][ia] >= first_leaf, lc = node[1][ic] >= first_leaf;
                ++c_tests;
                c_ll += (la && lc) ? 1u : 0u;
                c_li += (la != lc) ? 1u : 0u;
                if (la)
                    ctr_visit(lk[0][ia]);
                if (lc)
                    ctr_visit(lk[1][ic]);
            }
        ctr_wave_add(0, c_tests);
        ctr_wave_add(1, c_ll);
        ctr_wave_add(2, c_li);
        ctr_wave_add(3, (uint32_t)__popc(hit));
        ctr_wave_add(4, active ? 1u : 0u);
#endif
    }

    __device__ uint2 pair(int bit) const { return make_uint2(node[0][bit >> 1], node[1][bit & 1]); }

    __device__ Rec record(int bit) const
    {
        const bool a = (bit & 2) != 0, c = (bit & 1) != 0;
        const uint32_t oa = a ? lk[0][1] : lk[0][0], oc = c ? lk[1][1] : lk[1][0];
        const uint32_t a0 = a ? t0[0][1] : t0[0][0], c0 = c ? t0[1][1] : t0[1][0];
        const uint32_t a1 = a ? t1[0][1] : t1[0][0], c1 = c ? t1[1][1] : t1[1][0];
        Rec rec;
        rec.i = oa < oc ? oa : oc;
        rec.j = oa < oc ? oc : oa;
        rec.tlo = a0 > c0 ? a0 : c0;
        rec.thi = a1 < c1 ? a1 : c1;
        return rec;
    }
};

// What a wave holds in LDS: pairs (an expansion of 64 adds up to 256) and
// records.
constexpr uint32_t kExpandStack = 576, kExpandRecs = 64;
constexpr size_t kExpandLds = kExpandStack * sizeof(uint2) + kExpandRecs * sizeof(Rec);
// Pairs above which a wave sends what it holds to the queue; in deep launches
// all but 64, and sooner: a wave with that many is far behind the others.
constexpr uint32_t kExpandKeep = kExpandStack - 256, kExpandKeepDeep = 128;
// A launch over at most this many pairs goes deep; expansions a wave then makes
// after its input has run out before it hands what is left to the next launch,
// which deals it out again.  Measured on 3.2 M pairs over 60.65 M leaves and on
// 17.5 M over 79.7 M (which first shrink to 175 K a level and then grow to
// 845 K): 65 536 pairs 291 and 902 us, 131 072 279 and 903, 262 144 222 and
// 873, 524 288 249 and 1 022; without a limit of expansions 221 and 1 175.
constexpr uint32_t kExpandDeep = 262144, kExpandTail = 16, kExpandTailLast = 65536;

// One launch over the pairs of `in`, each wave by itself until its workgroup's
// last appends.
//
// Many pairs: one level.  A wave takes strips of 64 pairs and collects their
// child pairs and records in LDS.  Breadth first the pairs of a strip share
// nodes, and every level is dealt to the waves anew: depth first from the
// start, with each wave's stack in LDS, took 2.3 ms where the levels took 1.4
// (17.5 M pairs over 79.7 M leaves).
//
// Few pairs: a launch per level costs more than its work (about 8 us).  Here a
// wave goes on with its own stack, 64 pairs at a time.
//
// Appends: atomics on one address go through the memory side one after another
// (12 ns each measured: one per wave made every level of 8 192 waves 100 us),
// so a wave appends some 350 pairs at a time, a workgroup makes one last append
// of each kind, and a queue is kExpandSubs lists whose counts lie apart, taken
// in turn.
//
// Bound: many pairs by random 64-byte records, four per pair (6.5 pairs per ns:
// 2 TB/s of 64-byte pieces, each in a 128-byte line of its own half the time);
// few by the two dependent reads of an expansion (about 2 us).  Against one
// launch per level with queues of ids: 4 240 seeds over 75 000 leaves 85 -> 37
// us, 495 K over 60.65 M 478 -> 300, 1.6 M over 79.7 M 1 395 -> 1 080; FP32,
// 77 K over 11.1 M 195 -> 77, 4 M over 79.7 M 3 222 -> 2 930.
template <int TP, bool IN, bool OUT>
__global__ __launch_bounds__(1024)
__attribute__((amdgpu_waves_per_eu(TP == CD_FP64 ? 5 : 7))) void k_expand(const void *__restrict__ tree,
                                                const uint2 *__restrict__ kids, uint32_t N,
                                                const uint2 *__restrict__ in,
                                                const unsigned int *n_in, uint32_t in_cap,
                                                uint2 *__restrict__ outq, unsigned int *n_out,
                                                uint32_t sub_cap, Rec *__restrict__ out,
                                                unsigned long long capacity,
                                                unsigned long long *counter, unsigned int *flags,
                                                int first, int last)
{
    extern __shared__ uint4 held[];
    __shared__ uint32_t stop, npair[16], nrec[16], qbase;
    __shared__ unsigned long long rbase;
    // a set flag (queue overflow, bad node, the traversal handed to the
    // per-leaf walk, or an earlier launch found its queue empty) ends the
    // node-pair levels
    if (threadIdx.x == 0)
        stop = *flags;
    // the seeds are one list, a queue is kExpandSubs of them: pair k of all is
    // pair k - start[q] of the last list q that starts at or before it
    uint32_t start[kExpandSubs], n = 0;
#pragma unroll
    for (int q = 0; q < kExpandSubs; ++q) {
        start[q] = n;
        const uint32_t c = first ? (q ? 0u : *n_in) : n_in[q * kExpandSubStride];
        n += c < in_cap ? c : in_cap;
    }
    __syncthreads();
    if (stop)
        return;
    if (n == 0) {
        // every pair has been expanded: flag 8 tells the host (and the gate)
        if (blockIdx.x == 0 && threadIdx.x == 0)
            atomicOr(flags, 8u);
        return;
    }
    const bool deep = IN == OUT && !first && (last || n <= kExpandDeep);
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6, per = blockDim.x >> 6;
    Rec *const recs = reinterpret_cast<Rec *>(held) + wv * kExpandRecs;
    uint2 *const st = reinterpret_cast<uint2 *>(reinterpret_cast<Rec *>(held) + per * kExpandRecs) +
                      wv * kExpandStack;
    // input in strips of `take` pairs, dealt to the waves in turn; a short
    // input in short strips, so that more waves share its latency
    const uint32_t waves = gridDim.x * per, share = (n + waves - 1) / waves;
    const uint32_t take = !deep || share > 64 ? 64u : share < 16 ? 16u : share;
    uint64_t strip = (uint64_t)(blockIdx.x * per + wv) * take;
    uint32_t done = 0;        // pairs taken of the strip
    uint32_t cnt = 0, rc = 0, left = last ? kExpandTailLast : kExpandTail;
    const uint32_t keep = !deep || last ? kExpandKeep : kExpandKeepDeep;
    uint32_t sub = (blockIdx.x * per + wv) % kExpandSubs;   // list of the wave's next append
    auto queue = [&](uint32_t from, uint32_t list, uint32_t q) {   // the pairs held from `from` on
        uint2 *const to = outq + (size_t)list * sub_cap;
        for (uint32_t k = from + lane; k < cnt; k += 64) {
            if (q + (k - from) < sub_cap)
                to[q + (k - from)] = st[k];
            else
                atomicOr(flags, 1u);
        }
        cnt = from;
    };
    auto records = [&](unsigned long long r) {   // those held
        if (lane < rc && r + lane < capacity)
            out[r + lane] = recs[lane];
        rc = 0;
    };
    for (;;) {
        const uint32_t m = !deep ? 0u : cnt < 64 ? cnt : 64u;   // from the wave's own pairs
        uint32_t f = 0;                                         // from the input
        if (strip < n) {
            const uint32_t rest = (uint32_t)(n - strip < take ? n - strip : take) - done;
            f = rest < 64 - m ? rest : 64 - m;
        } else {
            if (!deep || cnt == 0 || left == 0)
                break;
            --left;
        }
        cnt -= m;
        uint2 pr = make_uint2(0, 0);
        if (lane < m)
            pr = st[cnt + lane];
        else if (lane < m + f) {
            const uint32_t k = (uint32_t)strip + done + (lane - m);
            size_t at = k;
#pragma unroll
            for (uint32_t q = 1; q < kExpandSubs; ++q)
                at = k >= start[q] ? k - start[q] + (size_t)q * in_cap : at;
            pr = in[at];
        }
        asm volatile("" ::: "memory");
        if (strip < n) {
            done += f;
            if (done == take || strip + done == n) {
                strip += (uint64_t)waves * take;
                done = 0;
            }
        }
        PairTest<TP, IN, OUT> P;
        P.run(tree, kids, N, pr, lane < m + f, flags);
        // records, one a lane at a time
        for (;;) {
            const uint64_t some = __ballot(P.hit != 0);
            if (some == 0)
                break;
            const uint32_t total = (uint32_t)__popcll(some);
            if (rc + total > kExpandRecs) {   // those held, at once
                uint32_t r0 = 0, r1 = 0;
                if (lane == 0) {
                    const unsigned long long r = atomicAdd(
                        counter, (unsigned long long)__builtin_amdgcn_readfirstlane(rc));
                    r0 = (uint32_t)r;
                    r1 = (uint32_t)(r >> 32);
                }
                records(((unsigned long long)__builtin_amdgcn_readfirstlane(r1) << 32) |
                        __builtin_amdgcn_readfirstlane(r0));
            }
            if (P.hit != 0) {
                recs[rc + lanes_before(some)] = P.record(__ffs(P.hit) - 1);
                P.hit &= P.hit - 1;
            }
            rc += total;
        }
        // a lane's child pairs side by side: they share children, and so records
        uint32_t at = cnt;
#pragma unroll
        for (int bit = 0; bit < 4; ++bit) {
            const uint64_t all = __ballot((P.push & (1u << bit)) != 0);
            at += lanes_before(all);
            cnt += (uint32_t)__popcll(all);
        }
#pragma unroll
        for (int bit = 0; bit < 4; ++bit)
            if (P.push & (1u << bit))
                st[at++] = P.pair(bit);
        asm volatile("" ::: "memory");
        if (cnt > keep) {
            const uint32_t from = deep ? 64u : 0u;
            uint32_t q = 0;
            if (lane == 0)
                q = atomicAdd(n_out + sub * kExpandSubStride,
                              __builtin_amdgcn_readfirstlane(cnt - from));
            queue(from, sub, __builtin_amdgcn_readfirstlane(q));
            sub = (sub + 1) % kExpandSubs;
        }
    }
    if (lane == 0) {
        npair[wv] = cnt;
        nrec[wv] = rc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t p = 0, r = 0;
        for (uint32_t k = 0; k < per; ++k) {
            p += npair[k];
            r += nrec[k];
        }
        qbase = p ? atomicAdd(n_out + blockIdx.x % kExpandSubs * kExpandSubStride, p) : 0u;
        rbase = r ? atomicAdd(counter, (unsigned long long)r) : 0ull;
    }
    __syncthreads();
    uint32_t q = qbase;
    unsigned long long r = rbase;
    for (uint32_t k = 0; k < wv; ++k) {
        q += npair[k];
        r += nrec[k];
    }
    queue(0, blockIdx.x % kExpandSubs, q);
    records(r);
}

hipError_t launch_expand(const void *tree, const uint2 *kids, int precision, uint32_t N,
                         const uint2 *in, const unsigned int *n_in, uint32_t in_cap, uint2 *outq,
                         unsigned int *n_out, uint32_t sub_cap, Rec *out,
                         unsigned long long capacity, unsigned long long *counter,
                         unsigned int *flags, bool first, bool last, uint32_t blocks,
                         uint32_t threads, hipStream_t s)
{
    if (N <= 1)
        return hipSuccess;
    const size_t lds = threads / 64 * kExpandLds;
    auto run = [&](auto kernel) {
        kernel<<<blocks, threads, lds, s>>>(tree, kids, N, in, n_in, in_cap, outq, n_out, sub_cap,
                                            out, capacity, counter, flags, first ? 1 : 0, last ? 1 : 0);
        return hipGetLastError();
    };
    if (precision == CD_FP32)
        return run(k_expand<CD_FP32, true, true>);
    if (N > kCodedLeaves)
        return run(k_expand<CD_FP64, true, true>);
    // the seeds are ids, every later queue codes
    return first ? run(k_expand<CD_FP64, true, false>) : run(k_expand<CD_FP64, false, false>);
}

// ---- every level in one launch ----------------------------------------------------------------
//
// The same levels, run by one grid that the device holds at once: the
// workgroups take a level's pairs in turn, then wait for each other at a
// counter, so the next level reads a complete queue and count.  What one
// level hands to the next -- queue entries, counts, flags -- is written and
// read as device-scope atomics, each coherent by itself across the XCDs'
// separate L2 caches, and every wave waits for its own writes to complete
// before its workgroup arrives; no fence has to write back or invalidate the
// L2s (measured: with a release/acquire arrival per workgroup the traversal
// of the 16 848-object hour took 0.91 ms, with this one 0.79 ms; one launch
// per level takes 0.53 ms, so this form is not the default).
// The grid is sized on the host to the resident capacity, so every workgroup
// being waited for is running.  The wait ends in any case: a workgroup that
// sees an overflow or bad-node flag, or waits past kGridWaitTicks of the
// 100 MHz real-time clock, sets the handover flag and leaves; the query then
// runs the per-leaf walk from a cleared count, and every other workgroup sees
// the flag at its next wait.  A level with an empty input ends the kernel in
// every workgroup alike (the count is complete when it is read).
constexpr long long kGridWaitTicks = 200000000ll;   // 2 s

__device__ inline unsigned int load_dev(const unsigned int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One level over the n pairs of `in`, by every workgroup of the grid in turn
// (block-uniform loop: the block scan needs every thread).  The queue entries
// are written and read as device-scope atomics, each coherent across the XCDs'
// separate L2 caches by itself, for a reader in the same launch.
template <int TP>
__device__ inline void expand_level(const void *__restrict__ tree, const uint2 *__restrict__ kids,
                                    uint32_t N, const uint2 *__restrict__ in, uint32_t n,
                                    uint2 *__restrict__ outq, unsigned int *n_out,
                                    uint32_t out_cap, Rec *__restrict__ out,
                                    unsigned long long capacity, unsigned long long *counter,
                                    unsigned int *flags, uint32_t *wsum, unsigned int &qbase,
                                    unsigned long long &rbase)
{
    for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
        const uint32_t k = base + threadIdx.x;
        uint2 pr = make_uint2(0, 0);
        if (k < n) {
            const unsigned long long v =
                __hip_atomic_load(reinterpret_cast<const unsigned long long *>(in + k),
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pr = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
        }
        PairTest<TP, true, true> P;
        P.run(tree, kids, N, pr, k < n, flags);
        // one scan packs both counts: pushes in the low 16 bits, hits above
        uint32_t mine = (uint32_t)__popc(P.push) | ((uint32_t)__popc(P.hit) << 16);
        uint32_t total;
        uint32_t pre = block_exclusive_scan(mine, wsum, &total);
        if (threadIdx.x == 0) {
            qbase = (total & 0xFFFFu) ? atomicAdd(n_out, total & 0xFFFFu) : 0u;
            rbase = (total >> 16) ? atomicAdd(counter, (unsigned long long)(total >> 16)) : 0ull;
        }
        __syncthreads();
        uint32_t q = qbase + (pre & 0xFFFFu);
        unsigned long long r = rbase + (pre >> 16);
#pragma unroll
        for (int bit = 0; bit < 4; ++bit) {
            if (P.push & (1u << bit)) {
                if (q < out_cap)
                    __hip_atomic_store(reinterpret_cast<unsigned long long *>(outq + q),
                                       (unsigned long long)P.pair(bit).x |
                                           ((unsigned long long)P.pair(bit).y << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else
                    atomicOr(flags, 1u);
                ++q;
            }
            if (P.hit & (1u << bit)) {
                if (r < capacity)
                    out[r] = P.record(bit);
                ++r;
            }
        }
        __syncthreads();
    }
}

template <int TP>
__global__ __launch_bounds__(1024) void k_expand_all(const void *__restrict__ tree,
                                                    const uint2 *__restrict__ kids, uint32_t N,
                                                    const uint2 *seeds, const unsigned int *nseeds,
                                                    uint32_t seed_cap, uint2 *qa, uint2 *qb,
                                                    unsigned int *qcount, uint32_t qcap,
                                                    uint32_t max_levels, Rec *__restrict__ out,
                                                    unsigned long long capacity,
                                                    unsigned long long *counter,
                                                    unsigned int *flags, unsigned int *bar)
{
    __shared__ uint32_t wsum[64];
    __shared__ unsigned int qbase, go;
    __shared__ unsigned long long rbase;
    // handed over before the launch, or while this workgroup was not yet running:
    // read once, because a workgroup's waves must leave together
    if (threadIdx.x == 0)
        go = (load_dev(flags) & 7u) == 0;
    __syncthreads();
    if (!go)
        return;
    const uint2 *in = seeds;
    const unsigned int *n_in = nseeds;
    uint32_t in_cap = seed_cap;
    for (uint32_t lev = 0; lev < max_levels; ++lev) {
        uint32_t n = load_dev(n_in);
        n = n < in_cap ? n : in_cap;
        if (n == 0) {
            if (blockIdx.x == 0 && threadIdx.x == 0)
                atomicOr(flags, 8u);
            return;
        }
        uint2 *outq = (lev & 1) ? qb : qa;
        expand_level<TP>(tree, kids, N, in, n, outq, qcount + lev + 1, qcap, out,
                               capacity, counter, flags, wsum, qbase, rbase);
        // every wave's queue stores and count updates have completed (each
        // is coherent by itself) before its workgroup arrives
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) {
            __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned int target = (lev + 1) * gridDim.x;
            const long long start = wall_clock64();
            unsigned int ok = 1;
            while (load_dev(bar) < target) {
                if ((load_dev(flags) & 7u) || wall_clock64() - start > kGridWaitTicks) {
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
            if (!ok)
                atomicOr(flags, 4u);
            go = ok;
        }
        __syncthreads();
        if (!go)
            return;
        in = outq;
        n_in = qcount + lev + 1;
        in_cap = qcap;
    }
    // levels exhausted with pairs left: the walk finishes the query
    if (blockIdx.x == 0 && threadIdx.x == 0 && load_dev(n_in) != 0)
        atomicOr(flags, 4u);
}

// Workgroups of k_expand_all<TP> (1 024 lanes) the device holds at once.
static uint32_t resident_expand_all(int precision)
{
    static uint32_t cached[2] = {0, 0};
    const int t = precision == CD_FP64 ? 0 : 1;
    if (cached[t])
        return cached[t];
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    hipError_t e = precision == CD_FP64
                       ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                             &per_cu, reinterpret_cast<const void *>(&k_expand_all<CD_FP64>),
                             1024, 0)
                       : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                             &per_cu, reinterpret_cast<const void *>(&k_expand_all<CD_FP32>),
                             1024, 0);
    if (e != hipSuccess || per_cu <= 0 || cus <= 0)
        return 0;
    cached[t] = (uint32_t)(per_cu * cus);
    return cached[t];
}

hipError_t launch_expand_all(const void *tree, const uint2 *kids, int precision, uint32_t N,
                             const uint2 *seeds, const unsigned int *nseeds, uint32_t seed_cap,
                             uint2 *qa, uint2 *qb, unsigned int *qcount, uint32_t qcap,
                             uint32_t max_levels, Rec *out, unsigned long long capacity,
                             unsigned long long *counter, unsigned int *flags, unsigned int *bar,
                             uint32_t blocks, hipStream_t s)
{
    if (N <= 1)
        return hipSuccess;
    uint32_t res = resident_expand_all(precision);
    if (res == 0)
        return hipErrorInvalidDeviceFunction;
    uint32_t g = blocks < res ? blocks : res;
    g = g ? g : 1;
    if (precision == CD_FP64)
        k_expand_all<CD_FP64><<<g, 1024, 0, s>>>(tree, kids, N, seeds, nseeds, seed_cap, qa, qb,
                                                  qcount, qcap, max_levels, out, capacity,
                                                  counter, flags, bar);
    else
        k_expand_all<CD_FP32><<<g, 1024, 0, s>>>(tree, kids, N, seeds, nseeds, seed_cap, qa, qb,
                                                  qcount, qcap, max_levels, out, capacity,
                                                  counter, flags, bar);
    return hipGetLastError();
}

// ---- device-side control of the query (no host reads) -----------------------------------------

// Before the node-pair levels: the control words, the flags (init, or the whole
// traversal handed to the per-leaf walk after a build error or lost seeds) and
// the record count.
__global__ __launch_bounds__(1024) void k_query_begin(const TreeHeader *hdr, unsigned int *ctl,
                                                      uint32_t words, uint32_t flags_at,
                                                      unsigned int init,
                                                      unsigned long long *counter)
{
    const unsigned int f = init | (hdr->err || hdr->seed_overflow ? 4u : 0u);
    for (uint32_t k = threadIdx.x; k < words; k += blockDim.x)
        ctl[k] = k == flags_at ? f : 0u;
    if (threadIdx.x == 0)
        *counter = 0ull;
}

// After the last level: the per-leaf walk runs (from a cleared counter) if
// an overflow, bad-node or handover flag is set (bits 1, 2, 4; bit 8 only
// marks a drained queue) or one of the last queue's `lists` lists is not empty.
__global__ void k_query_decide(const unsigned int *last_count, uint32_t lists,
                               const unsigned int *qflags, unsigned long long *counter,
                               unsigned int *walk)
{
    unsigned int w = (*qflags & 7u) != 0 ? 1u : 0u;
    for (uint32_t q = 0; q < lists; ++q)
        w |= last_count[q * kExpandSubStride] != 0 ? 1u : 0u;
    if (w)
        *counter = 0ull;
    *walk = w;
}

// Slots [min(count, cap), cap) get a record that sorts after every real one
// and is the same in every slot, so the sort and the repeat removal can run
// over a fixed number of slots.
__global__ void k_pad_records(Rec *raw, const unsigned long long *counter, uint32_t cap)
{
    uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long c = *counter;
    if (r >= cap || (unsigned long long)r < c)
        return;
    Rec pad;
    pad.i = pad.j = pad.tlo = pad.thi = 0xFFFFFFFFu;
    raw[r] = pad;
}

// Result words: count (records written, or records found when they exceed the
// capacity) and status bits (1 capacity exceeded, 2 tree inconsistent).
// padded: the list was formed over all cap slots, the unused ones one filler.
__device__ inline void report_finish(unsigned long long c, unsigned int tree_err, uint32_t uniq,
                                     uint32_t cap, bool padded, unsigned long long *count_out,
                                     unsigned int *status_out)
{
    unsigned int st = 0;
    if (c > cap)
        st |= 1u;
    if (tree_err)
        st |= 2u;
    unsigned long long n = 0;
    if (c > cap)
        n = c;
    else if (c > 0)
        n = (unsigned long long)uniq - (padded && c < cap ? 1ull : 0ull);
    *count_out = n;
    *status_out = st;
}

__global__ void k_query_finish(const unsigned long long *counter, const unsigned int *tree_err,
                               const uint32_t *uniq, uint32_t cap,
                               unsigned long long *count_out, unsigned int *status_out)
{
    report_finish(*counter, *tree_err, *uniq, cap, true, count_out, status_out);
}

// Side by side, for one read: the record count, the tree's error word and the
// last of the queues 1 .. levels that held pairs (0: none did).  At least
// `levels` lanes of one workgroup, all of them; last: a word of LDS.
__device__ inline void report_status(const unsigned long long *counter,
                                     const unsigned int *tree_err, const unsigned int *qcount,
                                     uint32_t levels, unsigned int *out, unsigned int *last)
{
    if (threadIdx.x == 0)
        *last = 0;
    __syncthreads();
    const uint32_t l = threadIdx.x + 1;
    unsigned int any = 0;
    for (uint32_t q = 0; q < kExpandSubs && l <= levels; ++q)
        any |= qcount[q * kExpandSubStride + l];
    if (any)
        atomicMax(last, l);
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long c = *counter;
        out[0] = (unsigned int)c;
        out[1] = (unsigned int)(c >> 32);
        out[2] = *tree_err;
        out[3] = *last;
    }
}

__global__ __launch_bounds__(512) void k_query_status(const unsigned long long *counter,
                                                      const unsigned int *tree_err,
                                                      const unsigned int *qcount, uint32_t levels,
                                                      unsigned int *out)
{
    __shared__ unsigned int last;
    report_status(counter, tree_err, qcount, levels, out, &last);
}

hipError_t launch_query_status(const unsigned long long *counter, const unsigned int *tree_err,
                               const unsigned int *qcount, uint32_t levels, unsigned int *out,
                               hipStream_t s)
{
    static_assert(kExpandMaxLevels <= 512, "one lane per level");
    k_query_status<<<1, 512, 0, s>>>(counter, tree_err, qcount, levels, out);
    return hipGetLastError();
}

hipError_t launch_query_begin(const TreeHeader *hdr, unsigned int *ctl, uint32_t words,
                              uint32_t flags_at, unsigned int init, unsigned long long *counter,
                              hipStream_t s)
{
    k_query_begin<<<1, 1024, 0, s>>>(hdr, ctl, words, flags_at, init, counter);
    return hipGetLastError();
}

hipError_t launch_query_decide(const unsigned int *last_count, uint32_t lists,
                               const unsigned int *qflags, unsigned long long *counter,
                               unsigned int *walk, hipStream_t s)
{
    k_query_decide<<<1, 1, 0, s>>>(last_count, lists, qflags, counter, walk);
    return hipGetLastError();
}

hipError_t launch_pad_records(Rec *raw, const unsigned long long *counter, uint32_t cap,
                              hipStream_t s)
{
    if (cap == 0)
        return hipSuccess;
    k_pad_records<<<nblk(cap, 256), 256, 0, s>>>(raw, counter, cap);
    return hipGetLastError();
}

hipError_t launch_query_finish(const unsigned long long *counter, const unsigned int *tree_err,
                               const uint32_t *uniq, uint32_t cap,
                               unsigned long long *count_out, unsigned int *status_out,
                               hipStream_t s)
{
    k_query_finish<<<1, 1, 0, s>>>(counter, tree_err, uniq, cap, count_out, status_out);
    return hipGetLastError();
}

__device__ inline bool rec_eq(const Rec &a, const Rec &b)
{
    return a.i == b.i && a.j == b.j && a.tlo == b.tlo && a.thi == b.thi;
}

constexpr int kRecPer = kSmallCanon / 1024;   // records per lane of a 1 024-lane workgroup

// A record as two words in canonical order.
__device__ inline ulonglong2 rec_key(const Rec &r)
{
    return make_ulonglong2((unsigned long long)r.i << 32 | r.j,
                           (unsigned long long)r.tlo << 32 | r.thi);
}

// Short runs of records are sorted by brute force over the chip: a record's
// place is the number of records of its run before it (equal ones in input
// order).  kRankPer records per workgroup, each compared by kRankSlices lanes
// with the run's records in turn, a tile of them in LDS at a time; the lanes of
// a wave read 128 consecutive bytes (no bank conflicts).  A list of up to
// kSmallCanon records is one run, and one workgroup then drops its repeats.
// Bound: latency (the 10 M comparisons of 3 258 records take 3 us of 12).
// Against one workgroup's LDS radix sort, 8 to 10 digit passes of 4 to 6 us
// each: a few hundred records 41 -> 7 us, 3 258 66 -> 19, both with the repeats.
constexpr uint32_t kRankThreads = 256, kRankPer = 8, kRankSlices = kRankThreads / kRankPer,
                   kRankTile = 1024;

// Run blockIdx.y: the records [y width, (y + 1) width) of the list.
template <class Count>
__global__ __launch_bounds__(kRankThreads) void k_rank_runs(const Rec *__restrict__ list,
                                                            uint32_t host, Count g,
                                                            uint32_t width,
                                                            Rec *__restrict__ runs)
{
    __shared__ ulonglong2 tile[kRankTile];
    __shared__ uint32_t before[kRankPer];
    uint32_t m;
    const uint32_t first = blockIdx.y * width + blockIdx.x * kRankPer;
    if (!g.get(host, m) || first >= m)
        return;   // (the whole workgroup)
    const Rec *in = list + blockIdx.y * width;
    Rec *const sorted = runs + blockIdx.y * width;
    m -= blockIdx.y * width;
    m = m < width ? m : width;
    const uint32_t k = blockIdx.x * kRankPer + threadIdx.x % kRankPer;
    const uint32_t slice = threadIdx.x / kRankPer;
    const Rec me = in[k < m ? k : m - 1];
    const ulonglong2 x = rec_key(me);
    if (threadIdx.x < kRankPer)
        before[threadIdx.x] = 0;
    uint32_t rank = 0;
    for (uint32_t base = 0; base < m; base += kRankTile) {
        const uint32_t n = m - base < kRankTile ? m - base : kRankTile;
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < n; q += kRankThreads)
            tile[q] = rec_key(in[base + q]);
        __syncthreads();
#pragma unroll 4
        for (uint32_t q = slice; q < n; q += kRankSlices) {
            const ulonglong2 y = tile[q];
            const bool tie = (y.y < x.y) | ((y.y == x.y) & (base + q < k));
            rank += (y.x < x.x) | ((y.x == x.x) & tie) ? 1u : 0u;
        }
    }
    for (int o = kRankPer; o < 64; o <<= 1)
        rank += __shfl_xor(rank, o, 64);
    if ((threadIdx.x & 63u) < kRankPer)
        atomicAdd(&before[threadIdx.x % kRankPer], rank);
    __syncthreads();
    if (threadIdx.x < kRankPer && k < m)
        sorted[before[threadIdx.x]] = me;
}

// The sorted list without its repeats; *total = its length + bias.  Being the
// query's last kernel it also makes its report (a launch of its own is 4.5 us).
__global__ __launch_bounds__(1024) void k_small_unique(const Rec *__restrict__ sorted,
                                                       uint32_t host, SmallCount g,
                                                       Rec *__restrict__ out,
                                                       unsigned int *total, uint32_t bias,
                                                       QueryReport report)
{
    __shared__ uint32_t wsum[33];
    __shared__ unsigned int last;
    if (report.status)
        report_status(report.counter, report.tree_err, report.qcount, report.levels,
                      report.status, &last);
    uint32_t m;
    if (!g.get(host, m))
        return;
    const uint32_t k0 = threadIdx.x * kRecPer;   // each lane owns kRecPer consecutive records
    Rec r[kRecPer + 1];
    uint32_t mine = 0, keep = 0;
    if (k0 < m) {
        r[0] = sorted[k0 ? k0 - 1 : 0];
#pragma unroll
        for (int q = 0; q < kRecPer; ++q)
            r[q + 1] = sorted[k0 + q < m ? k0 + q : m - 1];
#pragma unroll
        for (int q = 0; q < kRecPer; ++q) {
            const bool on = k0 + q < m && (k0 + q == 0 || !rec_eq(r[q + 1], r[q]));
            keep |= on ? 1u << q : 0u;
            mine += on ? 1u : 0u;
        }
    }
    uint32_t all;
    uint32_t pos = block_exclusive_scan(mine, wsum, &all);
#pragma unroll
    for (int q = 0; q < kRecPer; ++q)
        if (keep & (1u << q))
            out[pos++] = r[q + 1];
    if (threadIdx.x == 0) {
        *total = all + bias;
        if (report.count_out)
            report_finish(*report.counter, *report.tree_err, all, report.cap, false,
                          report.count_out, report.status_out);
    }
}

// Medium lists: runs of kRunWidth records, sorted as above, then merged
// kMergeRuns at a time: a record's place in the merged run is its place in its
// own plus the records before it in the others (equal ones of earlier runs
// first), found by binary searches that advance together.  Bound: the chain of
// dependent reads of a pass (11 to 17), so few wide passes; in long lists their
// number.  A pass that has only two or four runs left is compiled for those:
// every other run costs each step of the search a read of nothing.
// Whole calls against 4 096-record tiles sorted by one workgroup each and merged
// pairwise: 5 000 records 165 -> 113 us, 16 000 170 -> 120, 100 000 195 -> 161,
// 180 000 215 -> 198, 262 000 222 -> 218 (with eight runs in every pass: 117, 139,
// 192, 229, 253).  Those calls copied the list before its tiles, which a query's
// list never was: there the list alone of 11 000 records 72 -> 55 us, of 36 000 88 ->
// 83, but of 136 000 119 -> 139 and of 204 000 132 -> 161.
constexpr uint32_t kRunWidth = 1024, kMergeRuns = 8;

template <uint32_t RUNS>
__global__ __launch_bounds__(256) void k_merge_runs(const Rec *__restrict__ in, uint32_t bound,
                                                    uint32_t width, Rec *__restrict__ out,
                                                    DevCount g)
{
    uint32_t count;
    if (!g.get(bound, count))
        return;
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count)
        return;
    const uint32_t run = k / width, group = run / RUNS * RUNS;
    const Rec me = in[k];
    const ulonglong2 x = rec_key(me);
    uint32_t len[RUNS], pos[RUNS];   // of the other runs; those before me
#pragma unroll
    for (uint32_t q = 0; q < RUNS; ++q) {
        const uint64_t b = (uint64_t)(group + q) * width;
        len[q] = group + q == run || b >= count ? 0u : (uint32_t)(count - b < width ? count - b : width);
        pos[q] = 0;
    }
    for (uint32_t step = width; step; step >>= 1) {
#pragma unroll
        for (uint32_t q = 0; q < RUNS; ++q) {
            const bool in_run = pos[q] + step <= len[q];
            const uint64_t at = (uint64_t)(group + q) * width + pos[q] + step - 1;
            const ulonglong2 y = rec_key(in[in_run ? at : k]);
            const bool tie = (y.y < x.y) | ((y.y == x.y) & (group + q < run));
            const bool before = (y.x < x.x) | ((y.x == x.x) & tie);
            pos[q] += (in_run & before) ? step : 0u;
        }
    }
    uint64_t place = (uint64_t)group * width + (k - run * width);
#pragma unroll
    for (uint32_t q = 0; q < RUNS; ++q)
        place += pos[q];
    out[place] = me;
}

hipError_t launch_small_canon(const Rec *in, uint32_t count, Rec *tmp, Rec *out,
                              unsigned int *total, hipStream_t s, const SmallCount &g,
                              uint32_t bias, const QueryReport &report)
{
    if (count == 0 || count > (uint32_t)kSmallCanon || (g.counter && g.limit != count))
        return hipErrorInvalidValue;
    k_rank_runs<<<(count + kRankPer - 1) / kRankPer, kRankThreads, 0, s>>>(in, count, g, count,
                                                                           tmp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    k_small_unique<<<1, 1024, 0, s>>>(tmp, count, g, out, total, bias, report);
    return hipGetLastError();
}

hipError_t launch_medium_canon(const Rec *in, Rec *a, Rec *b, uint32_t count, uint32_t *flags, uint32_t *pos,
                               void *scan_ws, Rec *out, hipStream_t s, const DevCount &g,
                               unsigned int *total, uint32_t bias)
{
    if (count <= (uint32_t)kSmallCanon || count > (uint32_t)kMediumCanon ||
        (g.counter && (!total || g.hi != count || !g.qflags || !g.tree_err)))
        return hipErrorInvalidValue;
    // Ranking a run costs its square: past the 65 536 records that two passes
    // merge a third one runs anyway and takes twice the runs, so they are half as
    // long (100 000 records 172 -> 161 us a call, 262 000 228 -> 218; a third pass
    // for fewer records would cost more than that).
    const uint32_t width = count > kMergeRuns * kMergeRuns * kRunWidth ? kRunWidth / 2 : kRunWidth;
    k_rank_runs<<<dim3(width / kRankPer, nblk(count, width)), kRankThreads, 0, s>>>(in, count, g,
                                                                                  width, b);
    hipError_t e = hipGetLastError();
    Rec *src = b, *dst = a;
    // passes for the bound; with a smaller device count the last ones copy
    for (uint32_t w = width; e == hipSuccess && w < count; w *= kMergeRuns) {
        const uint32_t left = nblk(count, w), blocks = nblk(count, 256);
        if (left <= 2)
            k_merge_runs<2><<<blocks, 256, 0, s>>>(src, count, w, dst, g);
        else if (left <= 4)
            k_merge_runs<4><<<blocks, 256, 0, s>>>(src, count, w, dst, g);
        else
            k_merge_runs<kMergeRuns><<<blocks, 256, 0, s>>>(src, count, w, dst, g);
        e = hipGetLastError();
        Rec *t = src;
        src = dst;
        dst = t;
    }
    if (e != hipSuccess)
        return e;
    return launch_unique(src, count, flags, pos, scan_ws, out, s, g, total, bias);
}

// ---- canonical list: sorted records, repeats dropped -----------------------------------------

__global__ void k_unique_flags(const Rec *in, uint32_t bound, uint32_t *flags, DevCount g)
{
    uint32_t count;
    if (!g.get(bound, count))
        return;
    uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= bound)
        return;
    if (r >= count) {   // past a device count: nothing to keep
        flags[r] = 0u;
        return;
    }
    bool f = true;
    if (r > 0) {
        Rec a = in[r - 1], b = in[r];
        f = a.i != b.i || a.j != b.j || a.tlo != b.tlo || a.thi != b.thi;
    }
    flags[r] = f ? 1u : 0u;
}

__global__ void k_unique_scatter(const Rec *in, uint32_t bound, const uint32_t *flags,
                                 const uint32_t *pos, Rec *out, uint32_t *total, uint32_t bias,
                                 DevCount g)
{
    uint32_t count;
    if (!g.get(bound, count))
        return;
    uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= count)
        return;
    if (flags[r])
        out[pos[r]] = in[r];
    if (r == count - 1)
        *total = pos[r] + flags[r] + bias;
}

hipError_t launch_unique(const Rec *in, uint32_t count, uint32_t *flags, uint32_t *pos,
                         void *scan_ws, Rec *out, hipStream_t s, const DevCount &g,
                         unsigned int *total, uint32_t bias)
{
    // total is written to pos[count] (pos holds count + 1 entries), or with a
    // device count to *total
    if (count == 0)
        return launch_fill_u32(pos, 0u, 1, s);
    k_unique_flags<<<nblk(count, 256), 256, 0, s>>>(in, count, flags, g);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        e = scan_exclusive_u32(flags, pos, count, scan_ws, s);
    if (e != hipSuccess)
        return e;
    k_unique_scatter<<<nblk(count, 256), 256, 0, s>>>(in, count, flags, pos, out,
                                                      g.counter ? total : pos + count, bias, g);
    return hipGetLastError();
}

#ifdef CD_COUNTERS
hipError_t counters_reset(uint32_t *visits, uint32_t nobj, hipStream_t s)
{
    static const unsigned long long zero[kCounterWords] = {};
    hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess)
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_ctr), zero, sizeof zero, 0, hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_visits), &visits, sizeof visits, 0,
                              hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_nobj), &nobj, sizeof nobj, 0, hipMemcpyHostToDevice);
    return e;
}

hipError_t counters_read(unsigned long long *out, hipStream_t s)
{
    hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess)
        e = hipMemcpyFromSymbol(out, HIP_SYMBOL(g_ctr), kCounterWords * sizeof(unsigned long long),
                                0, hipMemcpyDeviceToHost);
    return e;
}
#endif

} // namespace cd
