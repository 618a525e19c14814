// k_agglo.hip -- hierarchy, inner boxes and skip links, bottom-up, over leaves
// in key order.
//
// The tree is the AABB tree of Sec. 3.2 over 4D boxes: the binary radix tree
// over the leaves' keys (time slab above the 30-bit Morton code), the same
// tree as the top-down build's (k_tree.hip), found from the prefixes that
// neighbouring keys share (cd_logic.h, "bottom-up construction"): the node
// split after leaf g covers the leaves between the nearest shorter prefixes on
// either side, and its children sit at the positions g and g + 1.
//
// Pass 1 takes chunks of up to 1 024 leaves, one workgroup each.  A chunk's
// nodes are found first, from bytes alone: every lane looks up the two nearest
// smaller prefixes of its splits (at most five 8-byte LDS reads each way), so
// each node's range, side, id and slot are known before any box is touched.
// The nodes are then put in an order by height and the boxes are united level
// by level: slot g and slot g + 1 into the slot of the node's id, full lanes,
// one barrier a level, no atomics.  The position a node is written to held a
// leaf (or the item) whose own parent is already formed, because only an
// ancestor of a leaf can end at it.  The last levels hold a few nodes each:
// one wave runs them without barriers while the others write what does not
// need the boxes (child pairs, leaf links).  Sibling pairs whose boxes overlap
// are recorded (seeds of the node-pair traversal).  A chunk's nodes and leaves
// whose parents reach outside it are its roots; they are handed up, in position
// order.
//
// Uniform steps in the sorted layout: the codes of a slab are those of the
// seven other slabs of its block, so a workgroup takes one range of ranks in 8
// consecutive slabs, finds the nodes once and only unites boxes in the other
// seven, with the next slab's leaves already on the way into registers.  The
// codes are compared in every slab; a slab whose codes differ (boxes the caller
// built), or runs of three and more equal codes (whose order follows the
// positions), get nodes of their own.
//
// Later passes: one workgroup per 48 lists of roots builds everything above
// them (pass after pass inside the workgroup when they exceed 768 items) and
// hands its own roots up, so 60 M leaves take three of them, and no scan or
// compaction of the lists runs between the passes.
//
// Bound: pass 1 by the chain of levels (about 15 a chunk, five of them wide,
// 6 us of the 15 us of a chunk with shared nodes) with two workgroups of FP64
// slots on a CU, then by HBM.  Against the form before it, whose lanes climbed
// the hierarchy by LDS atomics, rebuilt it in every slab and scanned and
// compacted the roots between up to nine passes: 60.65 M FP64 leaves in place
// 2.55 -> 1.76 ms (8.5 GB at 4.8 TB/s), the passes above 317 -> 215 us; 79.7 M
// FP64 boxes gathered into an FP32 tree 4.33 -> 3.98 and 440 -> 231 us (FP64
// tree: 3.86 -> 4.0 ms, 385 -> 245 us: the gather of 64-byte pieces of six
// arrays bounds it either way).
//
// Leaves come in place (FP64 records the sorted-layout box build wrote in key
// order), from box arrays in key order, or from the general key sort: pass 1
// then reads each leaf's box through the sorted (key, box index) items and
// writes its leaf record.  An FP32 tree holds the outward-rounded boxes; its
// slots hold floats, so unions and sibling tests are those of its records.
#include <type_traits>

#include "cd_internal.h"

namespace cd {

namespace {

inline unsigned nblk(uint64_t n, unsigned t) { return (unsigned)((n + t - 1) / t); }

constexpr int kAggChunk = 1024;    // items of one chunk
constexpr int kAggThreads = 512;
constexpr int kAggOut = 256;       // roots one chunk may hand up
constexpr int kAggItems = 768;     // items of one chunk of a later pass (two workgroups a CU)
constexpr int kAggGroup = 48;      // lists one later workgroup takes
constexpr int kAggSlabs = 8;       // units (slabs, chunks) one workgroup of pass 1 takes
// Slabs of at least this many boxes are cut into chunks of their own (at least
// half full); smaller ones share chunks of 1 024 consecutive leaves.
constexpr uint32_t kAggSlabMin = 512;
constexpr int kPer = kAggChunk / kAggThreads;
constexpr uint32_t kMaxHeight = 126;   // above the 97 a chunk of ordered keys can reach

// A node handed to the next pass: leaf range, id, and four prefixes (prefix7):
// after its first leaf, after its last, before its first, after the leaf that
// follows it; one byte each, lowest first.
struct AggItem {
    uint32_t f, l, id, a;
};
static_assert(sizeof(AggItem) == 16, "AggItem layout");

// Keys of boxes already in key order: leaf j is box j, its key (j / ms) << 32 |
// code[j].  raw is what is read for a key, the rest is arithmetic (so that
// reads can be asked for early).
struct CodeItems {
    using Raw = uint32_t;
    const uint32_t *code;
    uint32_t ms, N;
    __device__ Raw raw(uint32_t j) const { return code[j]; }
    __device__ uint64_t key(Raw r, uint32_t j) const { return (uint64_t)(j / ms) << 32 | r; }
    __device__ uint32_t box(Raw, uint32_t j) const { return j; }
};

// The key sort's output.  PACKED: words slab << (cb + ib) | code << ib | box;
// else (slab << 32 | code, box) items of 16 bytes.
template <bool PACKED>
struct SortedItems {
    using Raw = typename std::conditional<PACKED, uint64_t, uint4>::type;
    const Raw *items;
    uint32_t N, ib, cb;
    __device__ Raw raw(uint32_t j) const { return items[j]; }
    __device__ uint64_t key(Raw w, uint32_t) const
    {
        if constexpr (PACKED)
            return ((w >> (cb + ib)) << 32) | ((uint32_t)(w >> ib) & ((1u << cb) - 1));
        else
            return (uint64_t)w.y << 32 | w.x;
    }
    __device__ uint32_t box(Raw w, uint32_t) const
    {
        if constexpr (PACKED)
            return (uint32_t)(w & ((1ull << ib) - 1));
        else
            return w.z;
    }
};
static_assert(sizeof(KV) == 16 && offsetof(KV, val) == 8, "KV read as four words");

// Slots of boxes in LDS.  FP64: four 16-byte words laid out as a tree record
// (lo0 lo1 | lo2 hi0 | hi1 hi2 | t0 t1 link esc); FP32: two (lo0 lo1 lo2 hi0 |
// hi1 hi2 t0 t1).  Word q of slot s is at w[q][s]: random slots spread over all
// banks, two neighbouring slots share one address register (constant
// offsets), and the four words of padding per row keep the words of one slot
// in different banks for copies by W lanes per slot.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <int TP, int CAP>
struct Slots {
    static constexpr int W = TP == CD_FP64 ? 4 : 2;
    u32x4 w[W][CAP + 4];
};

// min and max of numbers, one instruction each (fmin and fmax of the language
// first quiet both operands).
__device__ inline double min_of(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline double max_of(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float min_of(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float max_of(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ inline u32x4 two_doubles(double a, double b)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    return u32x4{(uint32_t)x, (uint32_t)(x >> 32), (uint32_t)y, (uint32_t)(y >> 32)};
}
__device__ inline double first_double(u32x4 v)
{
    return __builtin_bit_cast(double, (uint64_t)v.x | ((uint64_t)v.y << 32));
}
__device__ inline double second_double(u32x4 v)
{
    return __builtin_bit_cast(double, (uint64_t)v.z | ((uint64_t)v.w << 32));
}

template <int TP>
struct SlotBox;

template <>
struct SlotBox<CD_FP64> {
    double lo[3], hi[3];
    uint32_t t0, t1;
    template <int CAP>
    __device__ void get(const Slots<CD_FP64, CAP> &R, uint32_t s)
    {
        const u32x4 a = R.w[0][s], b = R.w[1][s], c = R.w[2][s];
        const uint2 d = *(const uint2 *)&R.w[3][s];
        lo[0] = first_double(a);
        lo[1] = second_double(a);
        lo[2] = first_double(b);
        hi[0] = second_double(b);
        hi[1] = first_double(c);
        hi[2] = second_double(c);
        t0 = d.x;
        t1 = d.y;
    }
    // the box and tags (link and esc, the last word's upper half, stay)
    template <int CAP>
    __device__ void put(Slots<CD_FP64, CAP> &R, uint32_t s) const
    {
        R.w[0][s] = two_doubles(lo[0], lo[1]);
        R.w[1][s] = two_doubles(lo[2], hi[0]);
        R.w[2][s] = two_doubles(hi[1], hi[2]);
        *(uint2 *)&R.w[3][s] = make_uint2(t0, t1);
    }
    // a node's record from the tree
    __device__ void load(const void *nodes, uint32_t N, uint32_t id)
    {
        NodeIO<CD_FP64>::get_box(nodes, N, id, lo, hi, t0, t1);
    }
    __device__ void from(const double l[3], const double h[3])
    {
        for (int d = 0; d < 3; ++d) {
            lo[d] = l[d];
            hi[d] = h[d];
        }
    }
};

template <>
struct SlotBox<CD_FP32> {
    float lo[3], hi[3];
    uint32_t t0, t1;
    template <int CAP>
    __device__ void get(const Slots<CD_FP32, CAP> &R, uint32_t s)
    {
        const u32x4 a = R.w[0][s], b = R.w[1][s];
        lo[0] = __uint_as_float(a.x);
        lo[1] = __uint_as_float(a.y);
        lo[2] = __uint_as_float(a.z);
        hi[0] = __uint_as_float(a.w);
        hi[1] = __uint_as_float(b.x);
        hi[2] = __uint_as_float(b.y);
        t0 = b.z;
        t1 = b.w;
    }
    template <int CAP>
    __device__ void put(Slots<CD_FP32, CAP> &R, uint32_t s) const
    {
        R.w[0][s] = u32x4{__float_as_uint(lo[0]), __float_as_uint(lo[1]), __float_as_uint(lo[2]),
                          __float_as_uint(hi[0])};
        R.w[1][s] = u32x4{__float_as_uint(hi[1]), __float_as_uint(hi[2]), t0, t1};
    }
    __device__ void load(const void *nodes, uint32_t N, uint32_t id)
    {
        const Box32 *b = (const Box32 *)nodes + id;
        const float4 a = *(const float4 *)&b->lo[0];
        const uint4 c = *(const uint4 *)&b->hi[1];
        lo[0] = a.x;
        lo[1] = a.y;
        lo[2] = a.z;
        hi[0] = a.w;
        hi[1] = __uint_as_float(c.x);
        hi[2] = __uint_as_float(c.y);
        t0 = c.z;
        t1 = c.w;
    }
    __device__ void from(const double l[3], const double h[3])
    {
        for (int d = 0; d < 3; ++d) {   // outward; floats held as doubles stay
            lo[d] = __double2float_rd(l[d]);
            hi[d] = __double2float_ru(h[d]);
        }
    }
};

template <int TP>
__device__ inline SlotBox<TP> united(const SlotBox<TP> &a, const SlotBox<TP> &b)
{
    SlotBox<TP> u;
    for (int d = 0; d < 3; ++d) {
        u.lo[d] = min_of(a.lo[d], b.lo[d]);
        u.hi[d] = max_of(a.hi[d], b.hi[d]);
    }
    u.t0 = a.t0 < b.t0 ? a.t0 : b.t0;
    u.t1 = a.t1 > b.t1 ? a.t1 : b.t1;
    return u;
}

// The 4D overlap of two boxes, every comparison made (no branches).
template <int TP>
__device__ inline bool slots_overlap(const SlotBox<TP> &a, const SlotBox<TP> &b)
{
    const bool t = (a.t0 < b.t1) & (b.t0 < a.t1);
    const bool x = (a.lo[0] <= b.hi[0]) & (b.lo[0] <= a.hi[0]);
    const bool y = (a.lo[1] <= b.hi[1]) & (b.lo[1] <= a.hi[1]);
    const bool z = (a.lo[2] <= b.hi[2]) & (b.lo[2] <= a.hi[2]);
    return (t & x) & (y & z);
}

// What a chunk knows of the node in a slot (meta) and of a node's turn (sched):
// split | (last item, or slot) << 10 | flags.
constexpr uint32_t kBits10 = 1023u, kLeftItem = 1u << 20, kRightItem = 1u << 21,
                   kFormed = 1u << 22, kWhole = 1u << 23;
constexpr uint32_t kSeed = 1u << 31;   // sched: the node's children overlap
// A root: first item | last item << 10 | flags.
constexpr uint32_t kRootSingle = 1u << 20, kRootLeft = 1u << 21, kRootWhole = 1u << 22;

// This lane, opaque to the compiler: what is computed from it stays inside the
// loop over slabs instead of being kept (and spilled) across it.
__device__ inline uint32_t lane_in_chunk()
{
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// LDS of one chunk.
template <int TP, bool LEAVES>
struct AggShared {
    static constexpr int kCap = LEAVES ? kAggChunk : kAggItems;
    Slots<TP, kCap> rec;
    uint64_t b[128], m8[16], m64[2];   // ByteMins
    uint64_t formed[16];               // a bit per split
    uint32_t sched[kCap], meta[kCap];
    uint8_t height[1024 + 4];              // of the node in a slot
    uint32_t hist[128];
    uint32_t lev[128];
    uint32_t roots[kAggOut];
    uint2 sbuf[kSeedStage];
    unsigned int nlev, nwide, nroots, sn, sbase, over, taken;
    // items: leaf ranges, ids, prefixes after the first leaf (one more: after
    // the leaf that follows the chunk)
    uint32_t itf[LEAVES ? 1 : kCap], itl[LEAVES ? 1 : kCap], iti[LEAVES ? 1 : kCap];
    uint8_t af[LEAVES ? 8 : kCap + 8];
    uint32_t pre[LEAVES ? 1 : kAggGroup + 1];
    __device__ ByteMins mins() const { return ByteMins{b, m8, m64}; }
    __device__ uint32_t value(uint32_t k) const { return ((const uint8_t *)b)[k]; }
};

// The chunk's place in the tree: item K's leaves and id, and the prefixes at
// its edges (vL before item 0, vR after item m - 1 -- also S's byte m - 1 --,
// vN after the leaf that follows).
template <int TP, bool LEAVES>
struct Chunk {
    AggShared<TP, LEAVES> &S;
    uint32_t N, base, m;   // base: leaf of item 0 (LEAVES)
    uint32_t vL, vR, vN;
    __device__ uint32_t first(uint32_t K) const { return LEAVES ? base + K : S.itf[K]; }
    __device__ uint32_t last(uint32_t K) const { return LEAVES ? base + K : S.itl[K]; }
    __device__ uint32_t item(uint32_t K) const { return LEAVES ? N - 1 + base + K : S.iti[K]; }
    // prefix after the first leaf of item K (K == m: of the item that follows)
    __device__ uint32_t after_first(uint32_t K) const
    {
        return LEAVES ? (K < m ? S.value(K) : vN) : S.af[K];
    }
    // nodes formed here (after find_nodes)
    __device__ uint32_t nodes() const { return S.lev[S.nlev]; }
    __device__ bool root_here() const { return vL == 0 && vR == 0; }   // covers every leaf
    // id of the node that covers the whole chunk
    __device__ uint32_t whole_id() const { return root_here() ? 0u : vR >= vL ? last(m - 1) : first(0); }
    // skip link of a node or leaf whose last item is L
    __device__ uint32_t escape(uint32_t L) const
    {
        const uint32_t r = last(L);
        return r + 1 >= N ? kEnd : after_first(L + 1) >= S.value(L) ? r + 1 : N + r;
    }
};

// Finds the nodes of the chunk whose m prefixes are in S.b (kPrefixPad from m
// on): S.sched in level order with the level starts S.lev (a node's level is
// its height, so levels shrink; the first nwide hold more than 64 nodes),
// S.meta by slot, S.roots.  Starts and ends with a barrier.  False if the
// heights did not settle (cannot happen: the nodes form a tree).
template <int TP, bool LEAVES>
__device__ __forceinline__ bool find_nodes(AggShared<TP, LEAVES> &S, uint32_t m, uint32_t vL, bool tree_root)
{
    const uint32_t t = lane_in_chunk();
    __syncthreads();
    if (t < 128) {
        uint32_t v = byte_min(S.b[t]);
        ((uint8_t *)S.m8)[t] = (uint8_t)v;
        for (int o = 1; o < 8; o <<= 1) {
            const uint32_t u = __shfl_xor(v, o, 64);
            v = u < v ? u : v;
        }
        if ((t & 7) == 0)
            ((uint8_t *)S.m64)[t >> 3] = (uint8_t)v;
        S.hist[t] = 0;
    }
    if (t == 0)
        S.nroots = 0;
    for (int j = 0; j < kPer; ++j)
        if (t + j * kAggThreads < AggShared<TP, LEAVES>::kCap)
            S.meta[t + j * kAggThreads] = 0;
    if (t < 1024 / 4)
        ((uint32_t *)S.height)[t] = 0;
    __syncthreads();
    const ByteMins B = S.mins();
    ChunkNode nd[kPer];
    uint32_t turn[kPer], rank[kPer], h[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t g = t + j * kAggThreads;
        nd[j].formed = false;
        rank[j] = h[j] = turn[j] = 0;
        if (g + 1 < m) {
            nd[j] = chunk_node(B, m, g, vL);
            const uint32_t dst = nd[j].whole ? 0u : nd[j].left ? nd[j].n : nd[j].p + 1;
            turn[j] = g | dst << 10 | (nd[j].p + 1 == g ? kLeftItem : 0u) |
                      (nd[j].n == g + 1 ? kRightItem : 0u);
        }
        const uint64_t f = __ballot(nd[j].formed);
        if ((t & 63) == 0)
            S.formed[g >> 6] = f;
    }
    // heights: a node is one above its children, whose heights appear at the
    // slots g and g + 1; every wave looks until all of its nodes have theirs
    // (leaf pairs have theirs at once, and the waves of a workgroup run
    // together, so each look settles at least the lowest nodes left)
    uint8_t *const H = S.height;
    bool open = true;
    for (uint32_t look = 0; open && look < 100000; ++look) {
        asm volatile("" ::: "memory");   // read anew: other waves write too
        uint32_t a[kPer], c[kPer];       // every read in flight before the first test
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t g = turn[j] & kBits10;   // 0 for lanes without a node
            a[j] = H[g];
            c[j] = H[g + 1];
        }
        bool left = false;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t ha = turn[j] & kLeftItem ? 0u : a[j];
            const uint32_t hc = turn[j] & kRightItem ? 0u : c[j];
            const bool wait = (!(turn[j] & kLeftItem) & (a[j] == 0)) |
                              (!(turn[j] & kRightItem) & (c[j] == 0));
            if (nd[j].formed & (h[j] == 0) & !wait) {
                // at most 97; more only for keys out of order
                const uint32_t up = 1 + (ha > hc ? ha : hc);
                h[j] = up < kMaxHeight ? up : kMaxHeight;
                H[(turn[j] >> 10) & kBits10] = (uint8_t)h[j];
            }
            left |= nd[j].formed & (h[j] == 0);
        }
        open = __any(left);
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (h[j])
            rank[j] = atomicAdd(&S.hist[h[j]], 1u);
    __syncthreads();
    if (t < 64) {   // level starts: heights 2 t + 1 and 2 t + 2 (none above 97)
        const uint32_t c0 = 2 * t + 1 < 128 ? S.hist[2 * t + 1] : 0u;
        const uint32_t c1 = 2 * t + 2 < 128 ? S.hist[2 * t + 2] : 0u;
        const uint32_t e0 = wave_inclusive_scan(c0 + c1) - c0 - c1, e1 = e0 + c0;
        S.lev[2 * t] = e0;
        S.lev[2 * t + 1] = e1;
        const uint64_t n0 = __ballot(c0 > 0), n1 = __ballot(c1 > 0);
        const uint64_t w0 = __ballot(c0 > 64), w1 = __ballot(c1 > 64);
        if (t == 0) {
            S.nlev = (uint32_t)(__popcll(n0) + __popcll(n1));
            S.nwide = (uint32_t)(__popcll(w0) + __popcll(w1));
        }
    }
    // roots: nodes and single items whose parent is not formed here
    auto outside = [&](uint32_t split) {
        return split >= m - 1 || !((S.formed[split >> 6] >> (split & 63)) & 1);
    };
    auto root = [&](uint32_t e) {
        const unsigned int k = atomicAdd(&S.nroots, 1u);
        if (k < (unsigned)kAggOut)
            S.roots[k] = e;
    };
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t g = t + j * kAggThreads;
        if (g < m && !(m == 1 && tree_root) && outside(chunk_item_parent(B, g, vL)))
            root(g | g << 10 | kRootSingle);
        const ChunkNode &c = nd[j];
        if (c.formed && !(c.whole && tree_root) && outside(c.left ? c.n : c.p))
            root((c.p + 1) | c.n << 10 | (c.left ? kRootLeft : 0u) | (c.whole ? kRootWhole : 0u));
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const ChunkNode &c = nd[j];
        if (!h[j])
            continue;
        S.sched[S.lev[h[j] - 1] + rank[j]] = turn[j];
        S.meta[(turn[j] >> 10) & kBits10] =
            (turn[j] & ~(kBits10 << 10)) | c.n << 10 | kFormed | (c.whole ? kWhole : 0u);
    }
    __syncthreads();
    return !open;
}

// Unites the boxes level by level (slots complete before the call, after a
// barrier); ends with a barrier.  Wide levels take every wave and a barrier
// each; the narrow ones above them are wave 0's alone, which needs none, while
// the other waves run `meanwhile` (lane, lanes).
// Nodes whose children overlap are marked in S.sched and counted in S.over.
template <int TP, bool LEAVES, class Meanwhile>
__device__ __forceinline__ void unite_levels(AggShared<TP, LEAVES> &S, Meanwhile meanwhile)
{
    const uint32_t t = lane_in_chunk(), lane = t & 63u;
    const uint32_t nlev = __builtin_amdgcn_readfirstlane(S.nlev);
    const uint32_t nwide = __builtin_amdgcn_readfirstlane(S.nwide);
    // level starts in the wave's registers (kMaxHeight levels at most)
    const uint32_t la = S.lev[lane], lb = S.lev[64 + lane];
    auto start = [&](uint32_t k) {
        return k < 64 ? __builtin_amdgcn_readlane(la, k) : __builtin_amdgcn_readlane(lb, k - 64);
    };
    // the lane's next node is read a level ahead
    uint32_t from = 0, to = start(1), w, i;
    auto turn = [&]() {
        i = from + t;
        w = S.sched[i < to ? i : 0u];
    };
    auto meet = [&](uint32_t now, uint32_t at) {
        const uint32_t g = now & kBits10;
        SlotBox<TP> a, o;
        a.get(S.rec, g);
        o.get(S.rec, g + 1);
        united(a, o).put(S.rec, (now >> 10) & kBits10);
        if (slots_overlap(a, o)) {
            S.sched[at] = now | kSeed;
            atomicAdd(&S.over, 1u);
        }
    };
    turn();
#pragma unroll 1
    for (uint32_t k = 0; k < nwide; ++k) {
        const uint32_t now = w, at = i;
        const bool on = at < to;
        from = to;
        to = start(k + 2);
        turn();
        if (on)
            meet(now, at);
        __syncthreads();
    }
    if (t < 64) {
        __builtin_amdgcn_s_setprio(3);
#pragma unroll 1
        for (uint32_t k = nwide; k < nlev; ++k) {
            const uint32_t now = w, at = i;
            const bool on = at < to;
            from = to;
            to = start(k + 2);
            turn();
            if (on)
                meet(now, at);
            wave_lds_sync();
        }
        __builtin_amdgcn_s_setprio(0);
    } else {
        meanwhile(t - 64, (uint32_t)kAggThreads - 64);
    }
    __syncthreads();
}

// The chunk's roots to out[0 .. kAggOut) in position order, their number to
// *count (S.roots after find_nodes).
template <int TP, bool LEAVES>
__device__ __forceinline__ void hand_up(const Chunk<TP, LEAVES> &C, AggItem *__restrict__ out,
                        uint32_t *__restrict__ count, bool &bad)
{
    AggShared<TP, LEAVES> &S = C.S;
    const uint32_t np = S.nroots < (unsigned)kAggOut ? S.nroots : (unsigned)kAggOut;
    if (threadIdx.x == 0) {
        *count = np;
        bad |= S.nroots > (unsigned)kAggOut;
    }
    for (uint32_t k = threadIdx.x; k < np; k += kAggThreads) {
        const uint32_t e = S.roots[k], F = e & kBits10, L = (e >> 10) & kBits10;
        uint32_t rank = 0;
        for (uint32_t q = 0; q < np; ++q)
            rank += (S.roots[q] & kBits10) < F;
        AggItem it;
        it.f = C.first(F);
        it.l = C.last(L);
        it.id = e & kRootSingle ? C.item(F)
                : e & kRootWhole ? C.whole_id()
                : e & kRootLeft  ? it.l
                                 : it.f;
        it.a = C.after_first(F) | S.value(L) << 8 | (F ? S.value(F - 1) : C.vL) << 16 |
               C.after_first(L + 1) << 24;
        out[rank] = it;
    }
}

// The staged seeds to the seed list; S.sn is clear afterwards.  Every lane
// calls it; starts and ends with a barrier.
template <int TP, bool LEAVES>
__device__ __forceinline__ void flush_seeds(AggShared<TP, LEAVES> &S, const SeedSink &seeds)
{
    __syncthreads();
    const uint32_t ms = S.sn;
    if (threadIdx.x == 0)
        S.sbase = ms ? seeds.reserve(ms) : 0u;
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < ms; k += kAggThreads)
        if (S.sbase + k < seeds.cap)
            seeds.items[S.sbase + k] = S.sbuf[k];
    __syncthreads();
    if (threadIdx.x == 0)
        S.sn = 0;
    __syncthreads();
}

// The children pairs that unite_levels marked, to the stage (one reservation in
// the seed list serves many chunks), or straight to the list when one chunk
// has more than the stage holds.  Called after a barrier; seeds_taken follows
// after the next one.
template <int TP, bool LEAVES>
__device__ __forceinline__ void take_seeds(const Chunk<TP, LEAVES> &C, const SeedSink &seeds)
{
    AggShared<TP, LEAVES> &S = C.S;
    const uint32_t n = __builtin_amdgcn_readfirstlane(S.over), t = lane_in_chunk();
    if (n == 0)
        return;
    const bool direct = n > (uint32_t)kSeedStage;
    if (__builtin_amdgcn_readfirstlane(S.sn) + n > (uint32_t)kSeedStage)
        flush_seeds(S, seeds);
    if (direct) {
        if (t == 0)
            S.sbase = seeds.reserve(n);
        __syncthreads();
    }
    const uint32_t staged = S.sn, nodes = C.nodes();
#pragma unroll 1
    for (uint32_t i = t; i < nodes; i += kAggThreads) {
        const uint32_t w = S.sched[i], g = w & kBits10;
        if (!(w & kSeed))
            continue;
        S.sched[i] = w & ~kSeed;
        const uint2 pair = make_uint2(w & kLeftItem ? C.item(g) : C.last(g),
                                      w & kRightItem ? C.item(g + 1) : C.first(g + 1));
        const uint32_t k = atomicAdd(&S.taken, 1u);
        if (!direct)
            S.sbuf[staged + k] = pair;
        else if (S.sbase + k < seeds.cap)
            seeds.items[S.sbase + k] = pair;
    }
}
// After the barrier that follows take_seeds; a barrier comes before the next
// chunk's seeds.
template <int TP, bool LEAVES>
__device__ __forceinline__ void seeds_taken(AggShared<TP, LEAVES> &S)
{
    if (threadIdx.x == 0) {
        if (S.over <= (unsigned)kSeedStage)
            S.sn += S.over;
        S.over = S.taken = 0;
    }
}

// Is a leaf's slab (t0 / ticks) the one of its position?  ONE: the chunk lies
// in one slab, of the times that slab_times gives (beyond: past every 32-bit tick);
// else slabs of ms leaves, item K of the chunk being leaf base + K (ms == 0: no
// slabs).
template <bool ONE>
struct SlabCheck {
    uint32_t ticks, start, base, ms;
    bool beyond;
    __device__ __forceinline__ bool off(uint32_t t0, uint32_t K) const
    {
        if (ONE)
            return beyond | (t0 - start >= ticks);
        return ms && t0 / ticks != (base + K) / ms;
    }
};

// One chunk's leaves in registers, on their way to the slots.  In place
// (GATHER < 0): four lanes per 64-byte record.  Otherwise kPer leaves a lane.
// Lanes past the chunk take its last leaf along (no branches, so that nothing
// waits for a load before its value is needed).
template <int TP, int GATHER>
struct LeafRegs {
    using F = typename std::conditional<GATHER == CD_FP32, float, double>::type;
    F lo[kPer][3], hi[kPer][3];
    uint32_t t0[kPer], t1[kPer], obj[kPer];
    __device__ __forceinline__ void load(const BoxView &bv, const void *, uint32_t,
                                         const uint32_t (&src)[kPer], uint32_t, uint32_t)
    {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            for (int d = 0; d < 3; ++d) {
                lo[j][d] = ((const F *)bv.lo[d])[src[j]];
                hi[j][d] = ((const F *)bv.hi[d])[src[j]];
            }
            t0[j] = bv.t0[src[j]];
            t1[j] = bv.t1[src[j]];
            obj[j] = bv.obj[src[j]];
        }
    }
    template <bool ONE>
    __device__ __forceinline__ void store(AggShared<TP, true> &S, uint32_t m,
                                          const SlabCheck<ONE> &in_slab, bool &misplaced) const
    {
        const uint32_t t = lane_in_chunk();
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t K = t + j * kAggThreads;
            double l[3], h[3];
            for (int d = 0; d < 3; ++d) {
                l[d] = (double)lo[j][d];
                h[d] = (double)hi[j][d];
            }
            SlotBox<TP> x;
            x.from(l, h);
            x.t0 = t0[j];
            x.t1 = t1[j];
            x.put(S.rec, K);
            if constexpr (TP == CD_FP64)   // the leaf record's object id
                *((uint2 *)&S.rec.w[3][K] + 1) = make_uint2(obj[j], 0u);
            misplaced |= (K < m) & in_slab.off(t0[j], K);
        }
    }
};

template <int TP>
struct LeafRegs<TP, -1> {
    static constexpr int kLoads = kAggChunk * 4 / kAggThreads;
    u32x4 v[kLoads];
    __device__ __forceinline__ void load(const BoxView &, const void *nodes, uint32_t N,
                                         const uint32_t (&)[kPer], uint32_t base, uint32_t m)
    {
        const u32x4 *r = (const u32x4 *)((const Node64 *)nodes + (size_t)(N - 1) + base);
        const uint32_t t = lane_in_chunk();
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const uint32_t x = t + j * kAggThreads;
            v[j] = r[x < 4 * m ? x : 4 * m - 4 + (x & 3u)];
        }
    }
    template <bool ONE>
    __device__ __forceinline__ void store(AggShared<TP, true> &S, uint32_t m,
                                          const SlabCheck<ONE> &in_slab, bool &misplaced) const
    {
        const uint32_t t = lane_in_chunk();
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const uint32_t x = t + j * kAggThreads, r = x >> 2, q = x & 3u;
            S.rec.w[q][r] = v[j];
        }
        if ((t & 3u) != 3)   // the lane's records' last words hold their t0
            return;
        if (ONE) {   // the latest after the slab's start decides
            uint32_t late = 0;
#pragma unroll
            for (int j = 0; j < kLoads; ++j) {
                const uint32_t d = v[j].x - in_slab.start;
                late = d > late ? d : late;
            }
            misplaced |= in_slab.beyond | (late >= in_slab.ticks);
        } else {
#pragma unroll 1
            for (uint32_t r = t >> 2; r < m; r += kAggThreads / 4)
                misplaced |= in_slab.off(S.rec.w[3][r].x, r);
        }
    }
};

// Records [0, m) of the slots that `which` selects, W lanes of 16 bytes per
// record, to record id(r): whole lines a wave, non-temporal.
template <int TP, class Which, class Id>
__device__ __forceinline__ void copy_slots(const Slots<TP, kAggChunk> &S, uint32_t m, u32x4 *nodes,
                                  Which which, Id id)
{
    constexpr uint32_t W = Slots<TP, kAggChunk>::W;
    const uint32_t t = lane_in_chunk();
#pragma unroll 2   // (the next chunk's leaves hold many registers meanwhile)
    for (uint32_t j = 0; j < (uint32_t)kAggChunk * W / kAggThreads; ++j) {
        const uint32_t x = t + j * kAggThreads, r = x / W, q = x % W;
        if (r < m && which(r))
            __builtin_nontemporal_store(S.w[q][r], nodes + (size_t)id(r) * W + q);
    }
}

}  // namespace

// One chunk's keys on their way (raw): the lane's own leaves', and in lanes 0 ..
// 4 of every wave those around the chunk's edges (leaf base - 1, base, base + m
// - 1, base + m, base + m + 1), in lanes 5 .. the successors of the wave's last
// own leaves.
template <class Items>
struct KeyRegs {
    typename Items::Raw own[kPer], edge;
    uint32_t edge_at;
    __device__ __forceinline__ void load(const Items &G, uint32_t base, uint32_t m)
    {
        const uint32_t t = lane_in_chunk(), l = t & 63u;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            // lanes past the chunk read its last key (no branches)
            const uint32_t k = t + j * kAggThreads;
            own[j] = G.raw(base + (k < m ? k : m - 1));
        }
        uint32_t at = l == 0 ? base - 1 : l == 1 ? base : base + m - 3 + l;
        at = l >= 5 ? base + (t - l) + 64 + (l - 5) * kAggThreads : at;
        edge_at = ((l < 5 + kPer) & (at < G.N)) != 0 ? at : base;   // others: unused
        edge = G.raw(edge_at);
    }
};

// What a chunk needs of its keys: the prefixes after the lane's leaves (one
// byte each), those at the edges, and the order check.
struct Prefixes {
    uint32_t own, vL, vR, vN;
    bool disorder;
    template <class Items>
    __device__ __forceinline__ void edges(const KeyRegs<Items> &raw, const Items &G,
                                          uint32_t base, uint32_t m)
    {
        const uint64_t e = G.key(raw.edge, raw.edge_at);
        auto at = [&](uint32_t k) {
            return (uint64_t)__builtin_amdgcn_readlane((uint32_t)e, k) |
                   (uint64_t)__builtin_amdgcn_readlane((uint32_t)(e >> 32), k) << 32;
        };
        const uint64_t k0 = at(0), k1 = at(1), k2 = at(2), k3 = at(3), k4 = at(4);
        vL = base ? prefix7(k0, k1, base - 1, base) : 0u;
        vR = base + m < G.N ? prefix7(k2, k3, base + m - 1, base + m) : 0u;
        vN = base + m + 1 < G.N ? prefix7(k3, k4, base + m, base + m + 1) : 0u;
        disorder = base + m < G.N && k2 > k3;
    }
    // after edges
    template <class Items>
    __device__ __forceinline__ void leaves(const KeyRegs<Items> &raw, const Items &G,
                                           uint32_t base, uint32_t m)
    {
        own = 0;
        const uint32_t t = lane_in_chunk();
        const uint64_t e = G.key(raw.edge, raw.edge_at);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t K = t + j * kAggThreads;
            const uint64_t x = G.key(raw.own[j], base + (K < m ? K : m - 1));
            const uint64_t after = __shfl_down((unsigned long long)x, 1, 64);
            const uint64_t over = (uint64_t)__builtin_amdgcn_readlane((uint32_t)e, 5 + j) |
                                  (uint64_t)__builtin_amdgcn_readlane((uint32_t)(e >> 32), 5 + j) << 32;
            const uint64_t y = (t & 63u) == 63 ? over : after;
            uint32_t v = kPrefixPad;
            if (K + 1 < m) {
                v = prefix7(x, y, base + K, base + K + 1);
                disorder |= x > y;
            } else if (K < m) {
                v = vR;
            }
            own |= v << (8 * j);
        }
    }
};

// Pass 1.  SHARED: workgroup (block of `units` slabs, chunk c of nc) takes ranks
// [c size, (c + 1) size) of each of the block's slabs of n leaves; else
// workgroup b takes the `units` chunks of `size` leaves from b units on (n ==
// N).  Roots of chunk k (slab nc + c, or k-th) go to out[k][0 .. kAggOut), their
// number to out_count[k].  TP: tree precision (FP32 only with GATHER >= 0).  The
// leaf skip links go to leaf_esc (FP64 trees) or into the FP32 tree's link
// records.  The next chunk's keys are read before this one's nodes are found
// and its leaves while this one's boxes are united.
template <int TP, int GATHER, class Items, bool SHARED>
__global__ __launch_bounds__(kAggThreads)
    __attribute__((amdgpu_waves_per_eu(TP == CD_FP64 || GATHER == CD_FP64 ? 4 : 6))) void k_agglo_leaves(
        Items G, BoxView bv, uint32_t slab_ticks, uint32_t n, uint32_t nc,
        uint32_t size, uint32_t units, void *__restrict__ nodes, uint2 *__restrict__ kids,
        uint32_t *__restrict__ leaf_esc, AggItem *__restrict__ out,
        uint32_t *__restrict__ out_count, SeedSink seeds, unsigned int *err)
{
    static_assert(TP == CD_FP64 || GATHER >= 0, "FP32 trees take their leaves by gather");
    constexpr bool LEAVES = true, kCode = std::is_same<Items, CodeItems>::value;
    static_assert(kCode || (!SHARED && GATHER >= 0), "slabs and records in place go by code");
    __shared__ AggShared<TP, LEAVES> S;
    const uint32_t N = G.N, blk = xcd_block(blockIdx.x, gridDim.x);
    const uint32_t c = SHARED ? blk % nc : 0u, all = SHARED ? N / n : nc;
    const uint32_t u0 = (SHARED ? blk / nc : blk) * units;
    const uint32_t u1 = u0 + units < all ? u0 + units : all;
    if (u0 >= u1)
        return;
    // first leaf and leaf count of unit u
    auto base_of = [&](uint32_t u) { return SHARED ? u * n + c * size : u * size; };
    auto count_of = [&](uint32_t u) {
        const uint32_t room = SHARED ? n - c * size : N - u * size;
        return room < size ? room : size;
    };
    bool bad = false, misplaced = false;
    KeyRegs<Items> key;            // of the next chunk
    LeafRegs<TP, GATHER> R;        // of this one
    Prefixes P;                    // of this one
    uint32_t mine[kPer];           // SHARED: this chunk's codes
    bool redo = true;
    key.load(G, base_of(u0), count_of(u0));
    auto boxes = [&](uint32_t (&src)[kPer], uint32_t base, uint32_t m) {
        const uint32_t t = lane_in_chunk();
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t k = t + j * kAggThreads;
            src[j] = G.box(key.own[j], base + (k < m ? k : m - 1));
        }
    };
    uint32_t src[kPer];
    boxes(src, base_of(u0), count_of(u0));
    R.load(bv, nodes, N, src, base_of(u0), count_of(u0));
    P.edges(key, G, base_of(u0), count_of(u0));
    P.leaves(key, G, base_of(u0), count_of(u0));
    if constexpr (SHARED)
        for (int j = 0; j < kPer; ++j)
            mine[j] = key.own[j];
    if (u0 + 1 < u1)
        key.load(G, base_of(u0 + 1), count_of(u0 + 1));
    if (threadIdx.x == 0)
        S.sn = S.over = S.taken = 0;
    for (uint32_t u = u0; u < u1; ++u) {
        const uint32_t base = base_of(u), m = count_of(u), t = lane_in_chunk();
        const bool more = u + 1 < u1;
        const Chunk<TP, LEAVES> C{S, N, base, m, P.vL, P.vR, P.vN};
        SlabCheck<SHARED> in_slab{slab_ticks, 0u, base, 0u, false};
        if constexpr (SHARED) {
            in_slab.beyond = !slab_times(u, slab_ticks, &in_slab.start, &in_slab.ticks);
        } else if constexpr (kCode) {
            in_slab.ms = G.ms;
        }
        R.store(S, m, in_slab, misplaced);
        // the next chunk's keys are here too: they were asked for before R
        Prefixes Q;
        bool differ = false;
        if (more) {
            const uint32_t nb = base_of(u + 1), nm = count_of(u + 1);
            Q.edges(key, G, nb, nm);
            if constexpr (SHARED) {
                // the nodes found serve the next slab if its codes are the same
                // (and those around it, unless the slab ends there)
                differ = (c > 0 && Q.vL != P.vL) || (c + 1 < nc && Q.vR != P.vR);
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    differ |= key.own[j] != mine[j];
                    mine[j] = key.own[j];
                }
            } else {
                Q.leaves(key, G, nb, nm);
            }
            boxes(src, nb, nm);
        }
        // (what the last chunk leaves undefined below is not used)
        KeyRegs<Items> key_ahead;
        if (u + 2 < u1)
            key_ahead.load(G, base_of(u + 2), count_of(u + 2));
        bool redo_next = true;
        if (redo) {
            if constexpr (SHARED) {
                if (u > u0) {   // (rare: codes read again)
                    KeyRegs<Items> again;
                    again.load(G, base, m);
                    P.leaves(again, G, base, m);
                }
            }
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                ((uint8_t *)S.b)[t + j * kAggThreads] = (uint8_t)(P.own >> (8 * j));
            bad |= !find_nodes(S, m, C.vL, C.root_here());
            if constexpr (SHARED) {   // runs of three or more equal codes
                for (int j = 0; j < kPer; ++j) {
                    const uint32_t K = t + j * kAggThreads;
                    differ |= K < m && S.value(K) >= kPrefixTie &&
                              (K ? S.value(K - 1) : C.vL) >= kPrefixTie;
                }
            }
        } else if (t == 0) {
            ((uint8_t *)S.b)[m - 1] = (uint8_t)C.vR;
        }
        misplaced |= P.disorder;
        if constexpr (SHARED)
            redo_next = __syncthreads_or(differ);
        if constexpr (GATHER >= 0) {   // leaf records
            copy_slots<TP>(S.rec, m, (u32x4 *)nodes, [](uint32_t) { return true; },
                           [&](uint32_t r) { return N - 1 + base + r; });
            if constexpr (TP == CD_FP32) {
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    const uint32_t r = t + j * kAggThreads;
                    if (r < m) {
                        Link l;
                        l.link = R.obj[j];
                        l.esc = C.escape(r);
                        ((Link *)((Box32 *)nodes + (2 * (size_t)N - 1)))[N - 1 + base + r] = l;
                    }
                }
            }
            __syncthreads();
        }
        LeafRegs<TP, GATHER> R_ahead;
        if (more)
            R_ahead.load(bv, nodes, N, src, base_of(u + 1), count_of(u + 1));
        // links of the nodes formed here and of the leaves
        unite_levels(S, [&](uint32_t l, uint32_t lanes) {
            for (uint32_t r = l; r < m; r += lanes) {
                if constexpr (TP == CD_FP64)
                    __builtin_nontemporal_store(C.escape(r), &leaf_esc[base + r]);
                const uint32_t w = S.meta[r], g = w & kBits10;
                if (!(w & kFormed))
                    continue;
                const uint32_t id = w & kWhole ? C.whole_id() : base + r;
                const uint32_t lid = w & kLeftItem ? C.item(g) : base + g;
                const uint32_t rid = w & kRightItem ? C.item(g + 1) : base + g + 1;
                const uint32_t ie = C.escape((w >> 10) & kBits10);
                kids[id] = make_uint2(lid, rid);
                if constexpr (TP == CD_FP32) {
                    Link x;
                    x.link = lid;
                    x.esc = ie;
                    ((Link *)((Box32 *)nodes + (2 * (size_t)N - 1)))[id] = x;
                } else {
                    *((uint2 *)&S.rec.w[3][r] + 1) = make_uint2(lid, ie);
                }
            }
        });
        const uint32_t wid = C.whole_id();
        copy_slots<TP>(S.rec, m, (u32x4 *)nodes, [&](uint32_t r) { return (S.meta[r] & kFormed) != 0; },
                       [&](uint32_t r) { return S.meta[r] & kWhole ? wid : base + r; });
        const uint32_t k = SHARED ? u * nc + c : u;
        hand_up(C, out + (size_t)k * kAggOut, &out_count[k], bad);
        take_seeds(C, seeds);
        key = key_ahead;
        P = Q;
        R = R_ahead;
        redo = redo_next;
        __syncthreads();
        seeds_taken(S);
    }
    flush_seeds(S, seeds);
    if (misplaced)
        atomicOr(err, 1u);
    if (bad)
        atomicOr(err, 2u);
}

// Scratch items of one group of `lists` lists: a pass that does not take all
// its items at once leaves at most kAggOut for each chunk of kAggItems of them
// (the passes after it write over the items they have read).
__host__ __device__ constexpr uint32_t group_scratch(uint32_t lists)
{
    const uint32_t items = lists * kAggOut;
    return items > (uint32_t)kAggItems ? (items + kAggItems - 1) / kAggItems * kAggOut : 0u;
}
static_assert(kAggOut <= kAggItems, "a chunk's roots fit where its items were");
static_assert(kAggGroup * kAggOut / 27 <= kAggItems, "three scratch passes suffice");

// Later passes: workgroup q builds the tree above the lists [q kAggGroup,
// (q + 1) kAggGroup) of in (kAggOut places each, in_count items) and hands its
// own roots up as list q of out.  More than kAggItems items run pass after
// pass through this group's scratch (at most a third of them is left by each).
template <int TP>
__global__ __launch_bounds__(kAggThreads) void k_agglo_items(
    uint32_t N, const AggItem *in, const uint32_t *__restrict__ in_count,
    uint32_t lists, AggItem *scratch, void *nodes, uint2 *__restrict__ kids,
    AggItem *out, uint32_t *__restrict__ out_count, SeedSink seeds, unsigned int *err)
{
    constexpr bool LEAVES = false;
    __shared__ AggShared<TP, LEAVES> S;
    __shared__ uint32_t sub_count;
    const uint32_t t = threadIdx.x, q = blockIdx.x, l0 = q * kAggGroup;
    const uint32_t nl = lists - l0 < (uint32_t)kAggGroup ? lists - l0 : (uint32_t)kAggGroup;
    if (t < 64) {
        const uint32_t v = t < nl ? in_count[l0 + t] : 0u;
        const uint32_t inc = wave_inclusive_scan(v < (uint32_t)kAggOut ? v : (uint32_t)kAggOut);
        if (t < (uint32_t)kAggGroup)
            S.pre[t + 1] = inc;
        if (t == 0) {
            S.pre[0] = 0;
            S.sn = S.over = S.taken = 0;
        }
    }
    __syncthreads();
    uint32_t total = S.pre[kAggGroup];
    if (total == 0) {
        if (t == 0)
            out_count[q] = 0;
        return;
    }
    bool bad = false;
    // this group's items: its input lists, then its scratch list
    AggItem *const buf = scratch + (size_t)q * group_scratch(kAggGroup);
    const AggItem *src = nullptr;
    auto item = [&](uint32_t i) {
        if (src)
            return src[i];
        uint32_t lo = 0, hi = kAggGroup;   // last list with pre[list] <= i
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (S.pre[mid] <= i)
                lo = mid;
            else
                hi = mid;
        }
        return in[(size_t)(l0 + lo) * kAggOut + (i - S.pre[lo])];
    };
    for (uint32_t round = 0;; ++round) {
        const bool final = total <= (uint32_t)kAggItems;
        AggItem *dst = final ? out + (size_t)q * kAggOut : buf;
        uint32_t made = 0;
        for (uint32_t c0 = 0; c0 < total; c0 += kAggItems) {
            const uint32_t m = total - c0 < (uint32_t)kAggItems ? total - c0 : (uint32_t)kAggItems;
            Chunk<TP, LEAVES> C{S, N, 0, m, item(c0).a >> 16 & 0xFFu, item(c0 + m - 1).a >> 8 & 0xFFu,
                                item(c0 + m - 1).a >> 24};
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const uint32_t K = t + j * kAggThreads;
                uint32_t v = kPrefixPad;
                if (K < m) {
                    const AggItem it = item(c0 + K);
                    S.itf[K] = it.f;
                    S.itl[K] = it.l;
                    S.iti[K] = it.id;
                    S.af[K] = (uint8_t)it.a;
                    v = it.a >> 8 & 0xFFu;
                    SlotBox<TP> x;
                    x.load(nodes, N, it.id);
                    x.put(S.rec, K);
                }
                ((uint8_t *)S.b)[K] = (uint8_t)v;   // 1 024 of them
            }
            if (t == 0)
                S.af[m] = (uint8_t)C.vN;
            bad |= !find_nodes(S, m, C.vL, C.root_here());
            unite_levels(S, [](uint32_t, uint32_t) {});
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const uint32_t r = t + j * kAggThreads;
                const uint32_t w = r < m ? S.meta[r] : 0u, g = w & kBits10;
                if (!(w & kFormed))
                    continue;
                const uint32_t nlast = (w >> 10) & kBits10;
                const uint32_t id = w & kWhole ? C.whole_id() : r == nlast ? C.last(r) : C.first(r);
                const uint32_t lid = w & kLeftItem ? C.item(g) : C.last(g);
                const uint32_t rid = w & kRightItem ? C.item(g + 1) : C.first(g + 1);
                SlotBox<TP> x;
                x.get(S.rec, r);
                double lo[3], hi[3];
                for (int d = 0; d < 3; ++d) {
                    lo[d] = (double)x.lo[d];
                    hi[d] = (double)x.hi[d];
                }
                NodeIO<TP>::put(nodes, N, id, lo, hi, x.t0, x.t1, lid, C.escape(nlast));
                kids[id] = make_uint2(lid, rid);
            }
            hand_up(C, dst + made, final ? &out_count[q] : &sub_count, bad);
            take_seeds(C, seeds);
            __syncthreads();
            seeds_taken(S);
            if (!final)
                made += sub_count;
            // the records and scratch items written by this workgroup, before
            // it reads them again
            __threadfence_block();
            __syncthreads();
        }
        if (final)
            break;
        src = buf;
        total = made;
        if (total == 0 || round > 3) {   // cannot happen: every pass leaves a third
            if (t == 0)
                out_count[q] = 0;
            bad = true;
            break;
        }
    }
    flush_seeds(S, seeds);
    if (bad)
        atomicOr(err, 2u);
}

namespace {

// Chunks of pass 1, at most: all but the last are full, or (slabs of ms >=
// kAggSlabMin boxes) a slab has ceil(ms / 1024) of them, which is at most
// floor(ms / 512).
size_t agglo_chunks(uint32_t N) { return N < 2 * kAggSlabMin ? 1 : N / kAggSlabMin; }

// The workspace: pass 1's roots per chunk, the lists of every other pass
// after it, the groups' scratch, the lists' lengths.
struct AggPlan {
    AggItem *stage[2], *scratch;
    uint32_t *counts[2];
    size_t bytes;
};

AggPlan agglo_plan(void *ws, uint32_t N)
{
    const size_t chunks = agglo_chunks(N), groups = (chunks + kAggGroup - 1) / kAggGroup;
    Carve cv(ws, ~(size_t)0);
    AggPlan P;
    P.stage[0] = cv.take<AggItem>(chunks * kAggOut);
    P.counts[0] = cv.take<uint32_t>(chunks);
    P.stage[1] = P.scratch = nullptr;
    P.counts[1] = nullptr;
    if (chunks > 1) {
        if (groups > 1)
            P.stage[1] = cv.take<AggItem>(groups * kAggOut);
        P.scratch = cv.take<AggItem>(chunks / kAggGroup * group_scratch(kAggGroup) +
                                     group_scratch((uint32_t)(chunks % kAggGroup)));
        P.counts[1] = cv.take<uint32_t>(groups);
    }
    P.bytes = cv.off;
    return P;
}

// Passes 2, 3, ... over the roots that pass 1's chunks left.
template <int TP>
hipError_t agglo_item_passes(uint32_t N, uint32_t lists, void *nodes, uint2 *kids,
                             const AggPlan &P, const SeedSink &seeds, unsigned int *err,
                             hipStream_t s)
{
    hipError_t e = hipSuccess;
    for (int cur = 0; e == hipSuccess && lists > 1; cur ^= 1) {
        const uint32_t groups = nblk(lists, kAggGroup);
        // (one group hands up nothing, or, after a key order error, roots that
        // nobody reads: over the items it has read)
        k_agglo_items<TP><<<groups, kAggThreads, 0, s>>>(
            N, P.stage[cur], P.counts[cur], lists, P.scratch, nodes, kids,
            P.stage[groups > 1 ? cur ^ 1 : cur], P.counts[cur ^ 1], seeds, err);
        e = hipGetLastError();
        lists = groups;
    }
    return e;
}

// Pass 1 and the passes above it.
template <int TP, int GATHER, class Items>
hipError_t agglo_build(const Items &G, const BoxView &bv, uint32_t slab_ticks, void *nodes,
                       uint2 *kids, uint32_t *leaf_esc, void *ws, const SeedSink &seeds,
                       unsigned int *err, hipStream_t s)
{
    const uint32_t N = G.N;
    const AggPlan P = agglo_plan(ws, N);
    uint32_t lists = 0;
    // A workgroup takes fewer units as long as that leaves less than a few times
    // the workgroups the chip holds at once: on a full chip eight units are the
    // faster choice (the next unit's leaves are read while this one is built),
    // below it they run one after another beside idle CUs or in a long last
    // round.  75 slabs of 1 000: 90 us in 10 workgroups, 22 in 75; 7 780 FP32
    // chunks: 457 us in 1 945 workgroups, 443 in 3 890.  Where slabs share
    // nodes, fewer units find them more often: 1 200 slabs of 5 000 take 213 us
    // by four units and 230 by two.
    constexpr uint32_t kResident = TP == CD_FP64 ? 512u : 768u;
    // Slabs that fill half a chunk or more: cut into equal chunks, whose nodes
    // are found once per block of kAggSlabs slabs.  Smaller slabs (and keys
    // without slabs): chunks of consecutive leaves, nodes found in each.
    if constexpr (std::is_same<Items, CodeItems>::value) {
        if (G.ms >= kAggSlabMin) {
            const uint32_t nc = nblk(G.ms, kAggChunk), size = nblk(G.ms, nc), slabs = N / G.ms;
            lists = slabs * nc;
            uint32_t units = kAggSlabs;
            while (units > 1 && nblk(slabs, units) * nc < 2 * kResident)
                units /= 2;
            k_agglo_leaves<TP, GATHER, Items, true>
                <<<nblk(slabs, units) * nc, kAggThreads, 0, s>>>(
                    G, bv, slab_ticks, G.ms, nc, size, units, nodes, kids, leaf_esc,
                    P.stage[0], P.counts[0], seeds, err);
        }
    }
    if (lists == 0) {
        lists = nblk(N, kAggChunk);
        uint32_t units = kAggSlabs;
        while (units > 1 && nblk(lists, units) < 3 * kResident)
            units /= 2;
        k_agglo_leaves<TP, GATHER, Items, false><<<nblk(lists, units), kAggThreads, 0, s>>>(
            G, bv, slab_ticks, N, lists, kAggChunk, units, nodes, kids, leaf_esc, P.stage[0],
            P.counts[0], seeds, err);
    }
    hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : agglo_item_passes<TP>(N, lists, nodes, kids, P, seeds, err, s);
}

}  // namespace

size_t agglo_ws_bytes(uint32_t N) { return agglo_plan(nullptr, N).bytes; }

hipError_t launch_agglo(const uint32_t *code, uint32_t slab_size, uint32_t slab_ticks,
                        uint32_t N, void *nodes, uint2 *kids, uint32_t *leaf_esc, void *ws,
                        const SeedSink &seeds, unsigned int *err, hipStream_t s)
{
    if (N == 0)
        return hipSuccess;
    if (!code || slab_size == 0 || slab_ticks == 0 || !ws || N % slab_size != 0)
        return hipErrorInvalidValue;
    return agglo_build<CD_FP64, -1>(CodeItems{code, slab_size, N}, BoxView{}, slab_ticks, nodes,
                                    kids, leaf_esc, ws, seeds, err, s);
}

hipError_t launch_agglo_gather(const AggLeafSource &src, const BoxView &bv, int box_precision,
                               int tree_precision, uint32_t N, void *nodes, uint2 *kids,
                               uint32_t *leaf_esc, void *ws, const SeedSink &seeds,
                               unsigned int *err, hipStream_t s)
{
    if (N == 0)
        return hipSuccess;
    const bool by_code = src.code && src.slab_size > 0 && src.slab_ticks > 0;
    const bool by_packed = src.packed && src.ib >= 1 && src.ib <= 32 &&
                           (uint64_t)N <= (1ull << src.ib) && src.cb >= 1 &&
                           src.cb <= kKeyCodeBits;
    if (!(by_code || by_packed || src.kv) || !ws || (by_code && N % src.slab_size != 0) ||
        (tree_precision == CD_FP64 && (!leaf_esc || box_precision != CD_FP64)))
        return hipErrorInvalidValue;
    auto build = [&](const auto &G) {
        using Items = typename std::decay<decltype(G)>::type;
        const uint32_t w = by_code ? src.slab_ticks : 1u;
        if (tree_precision == CD_FP64)
            return agglo_build<CD_FP64, CD_FP64, Items>(G, bv, w, nodes, kids, leaf_esc, ws,
                                                        seeds, err, s);
        if (box_precision == CD_FP64)
            return agglo_build<CD_FP32, CD_FP64, Items>(G, bv, w, nodes, kids, nullptr, ws, seeds,
                                                        err, s);
        return agglo_build<CD_FP32, CD_FP32, Items>(G, bv, w, nodes, kids, nullptr, ws, seeds,
                                                    err, s);
    };
    if (by_code)
        return build(CodeItems{src.code, src.slab_size, N});
    if (by_packed)
        return build(SortedItems<true>{src.packed, N, src.ib, src.cb});
    return build(SortedItems<false>{(const uint4 *)src.kv, N, 0, 0});
}

} // namespace cd
