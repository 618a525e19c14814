// cd_hostcheck.cpp -- the LBVH index arithmetic of cd_logic.h and the Kepler
// solver of orbit.h run on the CPU.
//
// Pre-flight only: the tests use it to check, without a GPU, that the Karras
// topology is a proper binary tree, that the skip links follow pre-order, that
// the stackless walk the traversal kernel performs terminates and finds
// the same pairs as the oracle, and that every Kepler solve ends at its root.
// It is not a fallback for any library call.
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <random>
#include <vector>

#include "cd_logic.h"
#include "orbit.h"

using namespace cd;

extern "C" {

// Topology of the tree over N sorted keys: for inner node i, its children,
// leaf range and skip link; for leaf i, its skip link.
int hc_karras(const uint64_t *keys, int64_t N, uint32_t *left, uint32_t *right, int64_t *first,
              int64_t *last, uint32_t *esc_inner, uint32_t *esc_leaf)
{
    if (N < 1)
        return 0;
    KeyArray K{keys};
    for (int64_t i = 0; i + 1 < N; ++i) {
        KarrasNode nd = karras_node(K, N, i);
        left[i] = nd.left;
        right[i] = nd.right;
        first[i] = nd.first;
        last[i] = nd.last;
        esc_inner[i] = karras_escape(K, N, nd.last);
    }
    for (int64_t i = 0; i < N; ++i)
        esc_leaf[i] = karras_escape(K, N, i);
    return 0;
}

// The same topology through the 32-bit views the kernels use: over the 64-bit
// keys (slab_size == 0), or over time-major slabs of slab_size keys whose
// upper 32 bits are the slab index (codes = the low 32 bits).
int hc_karras32(const uint64_t *keys, int64_t N, uint32_t slab_size, uint32_t *left,
                uint32_t *right, int64_t *first, int64_t *last, uint32_t *esc_inner,
                uint32_t *esc_leaf)
{
    if (N < 1 || N >= (int64_t)1 << 31)
        return -1;
    const uint32_t n = (uint32_t)N;
    std::vector<uint32_t> codes;
    if (slab_size) {
        if (n % slab_size)
            return -1;
        codes.resize(n);
        for (uint32_t i = 0; i < n; ++i)
            codes[i] = (uint32_t)keys[i];
    }
    for (uint32_t i = 0; i < n; ++i) {
        uint32_t s = slab_size ? i / slab_size : 0;
        SlabKeys32 V{slab_size ? codes.data() + (size_t)s * slab_size : nullptr,
                     s * slab_size, slab_size, s};
        if (i + 1 < n) {
            KarrasNode nd = slab_size ? karras_node_u32(V, n, i)
                                      : karras_node_u32(KeysFrom32{keys, keys[i]}, n, i);
            left[i] = nd.left;
            right[i] = nd.right;
            first[i] = nd.first;
            last[i] = nd.last;
            esc_inner[i] = slab_size ? slab_escape32(V, n, (uint32_t)nd.last)
                                     : keys_escape32(keys, n, (uint32_t)nd.last);
        }
        esc_leaf[i] = slab_size ? slab_escape32(V, n, i) : keys_escape32(keys, n, i);
    }
    return 0;
}

// Solves of the box kernels: (E, sin E, cos E) of Kepler's equation at M[k] from
// the cold start to cold[3 k ..], and at M[k] + dM[k] from the warm start there
// to warm[3 k ..].
void hc_kepler(int64_t n, const double *M, const double *dM, const double *e, double *cold,
               double *warm)
{
    for (int64_t k = 0; k < n; ++k) {
        double E = kepler_start(M[k], e[k]), sE, cE, q;
        kepler(M[k], e[k], E, sE, cE, q);
        cold[3 * k] = E;
        cold[3 * k + 1] = sE;
        cold[3 * k + 2] = cE;
        E = kepler_next(E, sE, q, e[k], dM[k]);
        kepler(M[k] + dM[k], e[k], E, sE, cE, q);
        warm[3 * k] = E;
        warm[3 * k + 1] = sE;
        warm[3 * k + 2] = cE;
    }
}

// 1 if the hierarchy's check takes time t to be one of slab u.
int hc_in_slab(uint32_t u, uint32_t ticks, uint32_t t)
{
    uint32_t start, width;
    return slab_times(u, ticks, &start, &width) && t - start < width ? 1 : 0;
}

int hc_packed_code_bits(int sb, int ib) { return packed_code_bits(sb, ib); }

uint32_t hc_morton30(double x, double y, double z, const double *mn, const double *inv_ext)
{
    return morton30(x, y, z, mn, inv_ext);
}

// The traversal kernel's walk for every leaf, over node arrays in the same
// numbering (inner 0..N-2, leaves N-1..2N-2): lo/hi [2N-1][3], t0/t1 [2N-1],
// link [2N-1] (left child or object id), esc [2N-1].  Writes up to cap records
// (i, j, t_lo, t_hi) and returns the number found, or -1 if a walk exceeded
// 2N + 2 steps.
int64_t hc_traverse(int64_t N, const double *lo, const double *hi, const uint32_t *t0,
                    const uint32_t *t1, const uint32_t *link, const uint32_t *esc,
                    uint32_t slab_ticks, uint32_t *out, int64_t cap)
{
    int64_t count = 0;
    for (int64_t i = 0; i < N; ++i) {
        int64_t q = N - 1 + i;
        uint64_t stop = (uint64_t)t1[q] + slab_ticks - 1;
        uint32_t node = esc[q];
        int64_t steps = 0;
        while (node != kEnd) {
            if (++steps > 2 * N + 2)
                return -1;
            if ((uint64_t)t0[node] >= stop)
                break;
            bool ov = time_overlap(t0[q], t1[q], t0[node], t1[node]) &&
                      space_overlap(lo + 3 * q, hi + 3 * q, lo + 3 * (int64_t)node,
                                    hi + 3 * (int64_t)node);
            bool leaf = node >= N - 1;
            if (ov && leaf && link[node] != link[q]) {
                if (count < cap) {
                    uint32_t a = link[q], b = link[node];
                    out[4 * count + 0] = a < b ? a : b;
                    out[4 * count + 1] = a < b ? b : a;
                    out[4 * count + 2] = t0[q] > t0[node] ? t0[q] : t0[node];
                    out[4 * count + 3] = t1[q] < t1[node] ? t1[q] : t1[node];
                }
                ++count;
            }
            node = (ov && !leaf) ? link[node] : esc[node];
        }
    }
    return count;
}

// The bottom-up build of k_agglo.hip replayed on the CPU: pass 1 over chunks
// of C leaves, later passes over the lists that groups of chunks handed up (in
// position order; a group with more than C items runs pass after pass over
// its own list until one chunk is left).  A chunk's nodes are found and run in
// the kernel's order: levels of equal prefix, longest first, each level's
// nodes in a shuffled order (every order is one the GPU may take), all of a
// level's reads before its writes.  Every meeting is checked to find both
// children where the kernel reads them, and each chunk's hand-ups to stay
// within the kernel's limit.  Writes each inner node's children and skip link
// and each leaf's skip link, as hc_karras32 does.  Returns 0, or a negative
// code naming the first violated check.
namespace {
struct HcItem {
    uint32_t f, l, id;
    uint32_t af, al, ab, an;   // prefixes after f, after l, before f, after l + 1
};
struct HcTree {
    uint32_t N;
    uint32_t *left, *right, *esc_inner;
    std::vector<uint8_t> formed;
    std::mt19937_64 rng;
};

// One chunk of at most 1 024 items; its roots are appended to out.
int hc_chunk(HcTree &T, const HcItem *it, uint32_t m, std::vector<HcItem> &out)
{
    uint64_t b[128], m8[16], m64[2];
    uint8_t bytes[1024], k8[128], k64[16];
    for (uint32_t k = 0; k < 1024; ++k)
        bytes[k] = k < m ? (uint8_t)it[k].al : (uint8_t)kPrefixPad;
    memcpy(b, bytes, sizeof b);
    for (int w = 0; w < 128; ++w)
        k8[w] = (uint8_t)byte_min(b[w]);
    memcpy(m8, k8, sizeof m8);
    for (int w = 0; w < 16; ++w)
        k64[w] = (uint8_t)byte_min(m8[w]);
    memcpy(m64, k64, sizeof m64);
    const ByteMins B{b, m8, m64};
    const uint32_t vL = it[0].ab, vR = it[m - 1].al, N = T.N;
    std::vector<ChunkNode> nd(m);
    std::vector<std::pair<uint32_t, uint32_t>> order;   // (prefix, split)
    for (uint32_t g = 0; g + 1 < m; ++g) {
        nd[g] = chunk_node(B, m, g, vL);
        // against a plain search
        uint32_t p = kNone, n = kNone;
        for (uint32_t k = g; k-- > 0;)
            if (bytes[k] <= bytes[g]) {
                p = k;
                break;
            }
        for (uint32_t k = g + 1; k < m; ++k)
            if (bytes[k] < bytes[g]) {
                n = k;
                break;
            }
        if (p != nd[g].p || n != (nd[g].n < m ? nd[g].n : kNone))
            return -1;
        if (nd[g].formed)
            order.push_back({bytes[g], g});
    }
    std::shuffle(order.begin(), order.end(), T.rng);
    std::stable_sort(order.begin(), order.end(),
                     [](const auto &x, const auto &y) { return x.first > y.first; });
    std::vector<uint32_t> slot(m);
    for (uint32_t k = 0; k < m; ++k)
        slot[k] = it[k].id;
    auto node_id = [&](const ChunkNode &c) {
        if (c.whole && vL == 0 && vR == 0)
            return 0u;   // the root
        return c.left ? it[c.n].l : it[c.p + 1].f;
    };
    std::vector<uint32_t> wrote(m, kNone);
    for (size_t s = 0; s < order.size();) {
        size_t e = s;
        while (e < order.size() && order[e].first == order[s].first)
            ++e;
        for (size_t k = s; k < e; ++k) {   // a level's reads ...
            const uint32_t g = order[k].second;
            const ChunkNode c = nd[g];
            const uint32_t l = c.p + 1 == g ? it[g].id : it[g].l;
            const uint32_t r = c.n == g + 1 ? it[g + 1].id : it[g + 1].f;
            if (slot[g] != l || slot[g + 1] != r)
                return -6;   // a slot does not hold the child
            const uint32_t id = node_id(c);
            if (id >= N - 1 || T.formed[id])
                return -2;
            T.formed[id] = 1;
            T.left[id] = l;
            T.right[id] = r;
            const uint32_t last = it[c.n].l, an = c.n + 1 < m ? it[c.n + 1].af : it[m - 1].an;
            T.esc_inner[id] = last + 1 >= N ? kEnd : an >= it[c.n].al ? last + 1 : N + last;
        }
        for (size_t k = s; k < e; ++k) {   // ... before its writes
            const ChunkNode c = nd[order[k].second];
            const uint32_t dst = c.whole ? 0 : c.left ? c.n : c.p + 1;
            slot[dst] = node_id(c);
            wrote[dst] = order[k].second;
        }
        s = e;
    }
    // roots: nodes and single items whose parent is not formed here
    auto outside = [&](uint32_t split) { return split == kNone || split == m - 1 || !nd[split].formed; };
    std::vector<HcItem> roots;
    for (uint32_t k = 0; k < m; ++k) {
        if (m == 1 && vL == 0 && vR == 0)
            break;
        if (outside(chunk_item_parent(B, k, vL)))
            roots.push_back(it[k]);
        if (k + 1 >= m || !nd[k].formed)
            continue;
        const ChunkNode c = nd[k];
        if (c.whole && vL == 0 && vR == 0)
            continue;
        if (outside(c.left ? c.n : c.p)) {
            const HcItem &F = it[c.p + 1], &L = it[c.n];
            roots.push_back(HcItem{F.f, L.l, node_id(c), F.af, L.al, F.ab,
                                   c.n + 1 < m ? it[c.n + 1].af : L.an});
        }
    }
    if (roots.size() > 256)
        return -5;
    std::sort(roots.begin(), roots.end(),
              [](const HcItem &x, const HcItem &y) { return x.f < y.f; });
    out.insert(out.end(), roots.begin(), roots.end());
    return 0;
}
}  // namespace

int hc_agglo(const uint32_t *codes, int64_t N64, uint32_t ms, uint32_t C, uint64_t seed,
             uint32_t *left, uint32_t *right, uint32_t *esc_inner, uint32_t *esc_leaf)
{
    if (N64 < 1 || N64 >= ((int64_t)1 << 31) || ms == 0 || C < 4 || C > 1024 || (C & (C - 1)))
        return -20;
    const uint32_t N = (uint32_t)N64, group = C / 16 < 2 ? 2 : C / 16;
    const CodeKeys G{codes, ms, N};
    HcTree T{N, left, right, esc_inner, std::vector<uint8_t>(N, 0), std::mt19937_64(seed)};
    auto after = [&](uint32_t j) {   // prefix after leaf j
        return j + 1 < N ? prefix7(G.key(j), G.key(j + 1), j, j + 1) : 0u;
    };
    std::vector<HcItem> leaves(N);
    for (uint32_t j = 0; j < N; ++j) {
        leaves[j] = HcItem{j, j, N - 1 + j, after(j), after(j), j ? after(j - 1) : 0u, after(j + 1)};
        esc_leaf[j] = j + 1 >= N ? kEnd : after(j + 1) >= after(j) ? j + 1 : N + j;
    }
    std::vector<std::vector<HcItem>> lists;
    for (uint32_t c0 = 0; c0 < N; c0 += C) {
        std::vector<HcItem> out;
        int rc = hc_chunk(T, &leaves[c0], std::min(C, N - c0), out);
        if (rc)
            return rc;
        lists.push_back(out);
    }
    while (lists.size() > 1) {
        std::vector<std::vector<HcItem>> next;
        for (size_t q = 0; q < lists.size(); q += group) {
            std::vector<HcItem> in, out;
            for (size_t k = q; k < std::min(lists.size(), q + group); ++k)
                in.insert(in.end(), lists[k].begin(), lists[k].end());
            for (int round = 0;; ++round) {
                if (round > 20)
                    return -8;   // no progress
                out.clear();
                for (size_t c0 = 0; c0 < in.size(); c0 += C) {
                    int rc = hc_chunk(T, &in[c0], (uint32_t)std::min((size_t)C, in.size() - c0), out);
                    if (rc)
                        return rc;
                }
                if (in.size() <= C)
                    break;
                in = out;
            }
            next.push_back(out);
        }
        lists.swap(next);
    }
    if (!lists.empty() && !lists[0].empty())
        return -9;
    for (uint32_t i = 0; i + 1 < N; ++i)
        if (!T.formed[i])
            return -10;   // an inner node never formed
    return 0;
}

} // extern "C"
