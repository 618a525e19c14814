// k_sort.hip -- fills, device-wide exclusive scan, stable LSD radix sorts.
//
// Radix sorts:
//   * radix_sort_words / _keyed / _records: device-wide, stable, over 8-byte
//     items (a key and its box index packed in one word), (key, index) pairs or
//     pair records in 9-bit digits, one histogram + scan + scatter per digit.
//     They sort tree keys when boxes are not grouped in slabs and put pair
//     records in canonical order.
//   * radix_sort16: the same in 8-bit digits and less scratch, for the small
//     (key, index) lists of the band graph.
//   * k_slab_build: one 1024-thread workgroup per time slab; keys stay in
//     registers and move through LDS between digit passes, so a slab of up to
//     kSegCap boxes is sorted with one read and one write of global memory.
// All rank digits stably with the same wave-level scheme: the lanes holding
// equal digits are found with a ballot for each bit of the digit, the lowest of
// them bumps a per-(digit, wave) counter in LDS, and a digit-major scan of those
// counters turns per-wave ranks into positions.
#include "cd_internal.h"

namespace cd {

static inline unsigned nblk(uint64_t n, unsigned t) { return (unsigned)((n + t - 1) / t); }

// ---- fills ---------------------------------------------------------------------

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t count)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < count; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u64(unsigned long long *p, unsigned long long v, size_t count)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < count; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t count, hipStream_t s)
{
    if (count == 0)
        return hipSuccess;
    unsigned g = nblk(count, 256);
    k_fill_u32<<<g > 4096 ? 4096 : g, 256, 0, s>>>(p, v, count);
    return hipGetLastError();
}
hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, size_t count,
                           hipStream_t s)
{
    if (count == 0)
        return hipSuccess;
    unsigned g = nblk(count, 256);
    k_fill_u64<<<g > 4096 ? 4096 : g, 256, 0, s>>>(p, v, count);
    return hipGetLastError();
}

// ---- device-wide exclusive scan of uint32 ---------------------------------------

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const uint32_t *in, uint32_t *out,
                                                             size_t count, uint32_t *tile_sums)
{
    __shared__ uint32_t tile[kScanTile];
    __shared__ uint32_t wsum[64];
    size_t base = (size_t)blockIdx.x * kScanTile;
    for (int k = 0; k < kScanItems; ++k) {
        size_t g = base + (size_t)k * kScanThreads + threadIdx.x;
        tile[k * kScanThreads + threadIdx.x] = g < count ? in[g] : 0u;
    }
    __syncthreads();
    uint32_t v[kScanItems];
    uint32_t sum = 0;
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = tile[threadIdx.x * kScanItems + k];
        sum += v[k];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(sum, wsum, &total);
    for (int k = 0; k < kScanItems; ++k) {
        uint32_t x = v[k];
        tile[threadIdx.x * kScanItems + k] = run;
        run += x;
    }
    __syncthreads();
    for (int k = 0; k < kScanItems; ++k) {
        size_t g = base + (size_t)k * kScanThreads + threadIdx.x;
        if (g < count)
            out[g] = tile[k * kScanThreads + threadIdx.x];
    }
    if (threadIdx.x == 0 && tile_sums)
        tile_sums[blockIdx.x] = total;
}

__global__ void k_scan_add(uint32_t *out, size_t count, const uint32_t *tile_off)
{
    size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < count)
        out[g] += tile_off[g / kScanTile];
}

size_t scan_ws_bytes(size_t count)
{
    size_t bytes = 0;
    while (count > (size_t)kScanTile) {
        count = (count + kScanTile - 1) / kScanTile;
        bytes += align_up(count * sizeof(uint32_t), 256);
    }
    return bytes + 256;
}

hipError_t scan_exclusive_u32(const uint32_t *in, uint32_t *out, size_t count, void *ws,
                              hipStream_t s)
{
    if (count == 0)
        return hipSuccess;
    size_t tiles = (count + kScanTile - 1) / kScanTile;
    uint32_t *sums = tiles > 1 ? (uint32_t *)ws : nullptr;
    k_scan_tiles<<<(unsigned)tiles, kScanThreads, 0, s>>>(in, out, count, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || tiles == 1)
        return e;
    void *rest = (char *)ws + align_up(tiles * sizeof(uint32_t), 256);
    e = scan_exclusive_u32(sums, sums, tiles, rest, s);
    if (e != hipSuccess)
        return e;
    k_scan_add<<<nblk(count, 256), 256, 0, s>>>(out, count, sums);
    return hipGetLastError();
}

// ---- device-wide LSD radix sort of 16-byte items ------------------------------------------

constexpr int kRadThreads = 256;
constexpr int kRadItems = 16;
constexpr int kRadTile = kRadThreads * kRadItems;  // 4096
constexpr int kRadWaves = kRadThreads / 64;

struct DigitKV {
    uint32_t shift;
    __device__ uint32_t operator()(const uint4 &it) const
    {
        uint64_t key = ((uint64_t)it.y << 32) | it.x;
        return (uint32_t)(key >> shift) & 0xFFu;
    }
};
// Digit counts of one tile.  Lanes count into one of 16 copies of the
// histogram (by lane mod 16, rows of 257 words so that the copies of one
// digit sit in different banks): a tile whose items share a digit (a slab
// digit, say) then contends 4 lanes deep instead of 4 096.
template <typename Item, typename Digit>
__global__ __launch_bounds__(kRadThreads) void k_radix_upsweep(const Item *in, size_t count,
                                                               Digit dig, uint32_t *hist,
                                                               uint32_t nblocks)
{
    constexpr int kCopies = 16;
    __shared__ uint32_t h[kCopies * 257];
    for (int k = threadIdx.x; k < kCopies * 257; k += kRadThreads)
        h[k] = 0;
    __syncthreads();
    size_t base = (size_t)blockIdx.x * kRadTile;
    uint32_t dg[kRadItems];   // every load in flight before the first count
#pragma unroll
    for (int k = 0; k < kRadItems; ++k) {
        size_t g = base + (size_t)k * kRadThreads + threadIdx.x;
        dg[k] = g < count ? dig(in[g]) : 256u;
    }
    uint32_t *mine = h + (threadIdx.x % kCopies) * 257;
#pragma unroll
    for (int k = 0; k < kRadItems; ++k)
        if (dg[k] < 256u)
            atomicAdd(&mine[dg[k]], 1u);
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kCopies; ++q)
        sum += h[q * 257 + threadIdx.x];
    hist[(size_t)threadIdx.x * nblocks + blockIdx.x] = sum;
}

template <typename Item, typename Digit>
__global__ __launch_bounds__(kRadThreads) void k_radix_downsweep(const Item *in, Item *out,
                                                                 size_t count, Digit dig,
                                                                 const uint32_t *hist_scan,
                                                                 uint32_t nblocks)
{
    // per-(wave, digit) counters, wave-major with a 257-word row: lanes of a
    // wave (same w, random d) and the per-digit prefix (same d, all w) both
    // spread over the banks
    __shared__ uint32_t cnt[kRadWaves * 257];
    __shared__ uint32_t dbase[256];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = threadIdx.x; k < kRadWaves * 257; k += kRadThreads)
        cnt[k] = 0;
    dbase[threadIdx.x] = hist_scan[(size_t)threadIdx.x * nblocks + blockIdx.x];
    __syncthreads();
    size_t wbase = (size_t)blockIdx.x * kRadTile + (size_t)w * (64 * kRadItems);
    Item item[kRadItems];
    uint32_t dg[kRadItems], rk[kRadItems];
    uint64_t lt = lanemask_lt();
#pragma unroll
    for (int j = 0; j < kRadItems; ++j) {   // every load in flight before the ranking
        size_t g = wbase + (size_t)j * 64 + lane;
        item[j] = g < count ? in[g] : Item{};
    }
    for (int j = 0; j < kRadItems; ++j) {
        size_t g = wbase + (size_t)j * 64 + lane;
        bool valid = g < count;
        uint32_t d = valid ? dig(item[j]) : 0u;
        uint64_t act = __ballot(valid);
        uint64_t peers = match_digit(d, act);
        uint32_t c = valid ? cnt[w * 257 + d] : 0u;
        uint32_t mine = (uint32_t)__popcll(peers & lt);
        if (valid && mine == 0)
            cnt[w * 257 + d] = c + (uint32_t)__popcll(peers);
        dg[j] = d;
        rk[j] = c + mine;
    }
    __syncthreads();
    {   // per digit: exclusive prefix over waves
        uint32_t d = threadIdx.x, run = 0;
        for (int ww = 0; ww < kRadWaves; ++ww) {
            uint32_t t = cnt[ww * 257 + d];
            cnt[ww * 257 + d] = run;
            run += t;
        }
    }
    __syncthreads();
    for (int j = 0; j < kRadItems; ++j) {
        size_t g = wbase + (size_t)j * 64 + lane;
        if (g < count) {
            size_t pos = (size_t)dbase[dg[j]] + cnt[w * 257 + dg[j]] + rk[j];
            if (pos < count)
                out[pos] = item[j];
        }
    }
}

size_t radix_ws_bytes(size_t count)
{
    size_t nb = (count + kRadTile - 1) / kRadTile;
    size_t h = nb * 256;
    return align_up(h * sizeof(uint32_t), 256) + scan_ws_bytes(h);
}

hipError_t radix_sort16(void *a, void *b, size_t count, const DigitPlan &plan,
                        void *ws, void **result, hipStream_t s)
{
    *result = a;
    if (count <= 1 || plan.npass == 0)
        return hipSuccess;
    uint32_t nb = (uint32_t)((count + kRadTile - 1) / kRadTile);
    size_t h = (size_t)nb * 256;
    uint32_t *hist = (uint32_t *)ws;
    void *sws = (char *)ws + align_up(h * sizeof(uint32_t), 256);
    uint4 *src = (uint4 *)a, *dst = (uint4 *)b;
    for (int p = 0; p < plan.npass; ++p) {
        const DigitKV dg{plan.shift[p]};
        k_radix_upsweep<<<nb, kRadThreads, 0, s>>>(src, count, dg, hist, nb);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess)
            e = scan_exclusive_u32(hist, hist, h, sws, s);
        if (e != hipSuccess)
            return e;
        k_radix_downsweep<<<nb, kRadThreads, 0, s>>>(src, dst, count, dg, hist, nb);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        uint4 *t = src;
        src = dst;
        dst = t;
    }
    *result = src;
    return hipSuccess;
}

// ---- device-wide LSD radix sort of words, keyed items and records ------------------------
//
// Items of 8 or 16 bytes, digits of 9 bits, so that 36 key bits take four
// passes.  Per pass: k_digits_up counts each tile's digits into a row,
// k_digits_rows turns every kDigitChunk rows into prefixes and their sum,
// k_digits_chunks the sums into prefixes over the chunks and digit totals, and
// k_digits_down ranks a tile's items, stages them in LDS in digit order and
// writes each digit's run in consecutive lanes (128 bytes on average).  The
// first pass takes its items from a source of its own: the tree's key words are
// formed from the boxes' codes and tags as they are read, and its counts read
// the codes alone.
// Bound: HBM, three times the item's size a pass, and in the scatter the ranking
// (some 40 instructions an item).
// 36 bits of 79.7 M tree words: counts 3.9 TB/s (the first, of codes alone, 2.8:
// neighbours are one object's, with equal digits), scatter 4.1, 1.98 ms in all;
// as 37 bits with a digit of 10 and the words written by a kernel of their own
// 2.36 (keys 0.28, 10-bit scatter at 3.0 TB/s).  88 M words of 100 000 objects:
// 2.92 -> 2.42 ms.
constexpr int kDigitThreads = 512, kDigitWaves = kDigitThreads / 64, kDigitChunk = 64;
constexpr int kDigitBits = 9, kDigitBins = 1 << kDigitBits, kDigitCopies = 8;   // of the counters
static_assert(kDigitBins == kDigitThreads, "a lane per digit");
template <class Item>
struct Digits {
    // two workgroups' LDS on a CU
    static constexpr int kItems = 128 / (int)sizeof(Item);
    static constexpr int kTile = kDigitThreads * kItems;
};

// Where a pass takes its items from.  raw: what is read (for the scatter,
// low_raw for the counts of the first digit); item: the item.
template <class T>
struct ItemArray {
    using Item = T;
    using Raw = T;
    using LowRaw = T;
    const T *__restrict__ in;
    __device__ Raw raw(uint32_t g) const { return in[g]; }
    __device__ Item item(const Raw &v, uint32_t, bool *) const { return v; }
    __device__ LowRaw low_raw(uint32_t g) const { return in[g]; }
    __device__ Item low_item(const LowRaw &v) const { return v; }
    __device__ void report(bool) const {}
};
// The tree's key words, formed as launch_keys forms them.
struct KeyWords {
    using Item = uint64_t;
    using Raw = uint2;
    using LowRaw = uint32_t;
    KeySource k;
    __device__ Raw raw(uint32_t g) const { return make_uint2(k.code[g], k.t0[g]); }
    __device__ Item item(const Raw &v, uint32_t g, bool *bad) const
    {
        return key_word(k, v.x, v.y, g, bad);
    }
    // the code's bits alone: a first digit never reaches the slab
    __device__ LowRaw low_raw(uint32_t g) const { return k.code[g]; }
    __device__ Item low_item(uint32_t c) const { return key_code(k, c); }
    __device__ void report(bool bad) const
    {
        if (bad)
            atomicOr(k.err, 1u);
    }
};

// Digits of `mask`'s width.  A word's bits from `shift` on.
struct DigitWord {
    uint32_t shift, mask;
    __device__ uint32_t operator()(uint64_t v) const { return (uint32_t)(v >> shift) & mask; }
};
// A (64-bit key, index) item's key bits from `shift` on.
struct DigitKey {
    uint32_t shift, mask;
    __device__ uint32_t operator()(const uint4 &v) const
    {
        return (uint32_t)(((uint64_t)v.y << 32 | v.x) >> shift) & mask;
    }
};
// A record as one number, from the lowest field: t_hi (as the duration t_hi -
// t_lo, which keeps the order and takes fewer bits, or itself), t_lo, j, i, in
// `dur`, low - dur, j and whatever bits (t_lo and j cut to theirs: the filler of
// unused slots has every bit set); its bits from `shift` on.
struct DigitRec {
    uint32_t dur, low, j, tlo_mask, j_mask, as_end, shift, mask;
    __device__ uint32_t operator()(const uint4 &v) const
    {
        const uint64_t t = (uint64_t)(v.z & tlo_mask) << dur | (as_end ? v.w : v.w - v.z);
        const uint64_t ids = (uint64_t)v.x << j | (v.y & j_mask);
        // a digit that straddles the two words takes its upper bits from ids
        const uint64_t at = shift >= low ? ids >> (shift - low)
                            : shift + kDigitBits > low ? t >> shift | ids << (low - shift)
                                               : t >> shift;
        return (uint32_t)at & mask;
    }
};

// Digit counts of one tile (kCopies histograms by lane, rows of
// kDigitBins + 1 words so that the copies of one digit sit in different banks).
template <class Source, class Digit>
__global__ __launch_bounds__(kDigitThreads) void k_digits_up(Source src, uint32_t count,
                                                             Digit digit,
                                                             uint32_t *__restrict__ rows)
{
    using W = Digits<typename Source::Item>;
    constexpr int kRow = kDigitBins + 1;
    __shared__ uint32_t h[kDigitCopies * kRow];
    const uint32_t base = blockIdx.x * (uint32_t)W::kTile + threadIdx.x;
    typename Source::LowRaw v[W::kItems];
#pragma unroll
    for (int k = 0; k < W::kItems; ++k) {   // every load in flight before the first count
        const uint32_t g = base + k * kDigitThreads;
        v[k] = src.low_raw(g < count ? g : count - 1);
    }
    for (int k = threadIdx.x; k < kDigitCopies * kRow; k += kDigitThreads)
        h[k] = 0;
    __syncthreads();
    uint32_t *const mine = h + (threadIdx.x % kDigitCopies) * kRow;
#pragma unroll
    for (int k = 0; k < W::kItems; ++k)
        if (base + k * kDigitThreads < count)
            atomicAdd(&mine[digit(src.low_item(v[k]))], 1u);
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int c = 0; c < kDigitCopies; ++c)
        sum += h[c * kRow + threadIdx.x];
    rows[(size_t)blockIdx.x * kDigitBins + threadIdx.x] = sum;
}

// Rows [c kDigitChunk, ...) of one chunk: each count becomes the sum of those of
// the chunk's earlier rows, the chunk's total goes to sums[c].
__global__ __launch_bounds__(256) void k_digits_rows(uint32_t *__restrict__ rows, uint32_t tiles,
                                                    uint32_t *__restrict__ sums)
{
    constexpr int kBins = kDigitBins, kBatch = 16;
    const uint32_t d = blockIdx.y * 256 + threadIdx.x, r0 = blockIdx.x * kDigitChunk;
    const uint32_t n = tiles - r0 < (uint32_t)kDigitChunk ? tiles - r0 : (uint32_t)kDigitChunk;
    uint32_t run = 0;
    for (uint32_t k = 0; k < n; k += kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (uint32_t q = 0; q < kBatch; ++q)
            v[q] = k + q < n ? rows[(size_t)(r0 + k + q) * kBins + d] : 0u;
#pragma unroll
        for (uint32_t q = 0; q < kBatch; ++q) {
            if (k + q < n)
                rows[(size_t)(r0 + k + q) * kBins + d] = run;
            run += v[q];
        }
    }
    sums[(size_t)blockIdx.x * kBins + d] = run;
}

// One wave per digit: its sums over the chunks become prefixes, the total goes
// to the row after the last chunk's.
__global__ __launch_bounds__(256) void k_digits_chunks(uint32_t *__restrict__ sums, uint32_t chunks)
{
    constexpr int kBins = kDigitBins;
    const uint32_t d = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint32_t run = 0;
    for (uint32_t c0 = 0; c0 < chunks; c0 += 64) {
        const uint32_t c = c0 + lane;
        const uint32_t v = c < chunks ? sums[(size_t)c * kBins + d] : 0u;
        const uint32_t inc = wave_inclusive_scan(v);
        if (c < chunks)
            sums[(size_t)c * kBins + d] = run + inc - v;
        run += (uint32_t)__builtin_amdgcn_readlane(inc, 63);
    }
    if (lane == 0)
        sums[(size_t)chunks * kBins + d] = run;
}

template <class Source, class Digit>
__global__ __launch_bounds__(kDigitThreads) void k_digits_down(
    Source src, typename Source::Item *__restrict__ out, uint32_t count, Digit digit,
    const uint32_t *__restrict__ rows, const uint32_t *__restrict__ sums, uint32_t chunks)
{
    using Item = typename Source::Item;
    using W = Digits<Item>;
    __shared__ Item stage[W::kTile];
    __shared__ uint16_t cnt[kDigitWaves][kDigitBins + 2];   // per wave and digit
    __shared__ uint32_t to[kDigitBins];                     // place of staged item 0 by digit
    __shared__ uint32_t wsum[33];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t base = blockIdx.x * (uint32_t)W::kTile;
    const uint32_t m = count - base < (uint32_t)W::kTile ? count - base : (uint32_t)W::kTile;
    const uint32_t k0 = w * 64 * W::kItems + lane;
    Item item[W::kItems];
    uint32_t rank[W::kItems];
    {
        typename Source::Raw raw[W::kItems];
        bool bad = false;
#pragma unroll
        for (int j = 0; j < W::kItems; ++j) {   // every load in flight before the ranking
            const uint32_t k = k0 + j * 64;
            raw[j] = src.raw(base + (k < m ? k : m - 1));
        }
#pragma unroll
        for (int j = 0; j < W::kItems; ++j) {
            const uint32_t k = k0 + j * 64;
            item[j] = src.item(raw[j], base + (k < m ? k : m - 1), &bad);
        }
        src.report(bad);
    }
    const uint32_t d0 = threadIdx.x;   // this lane's digit
    uint32_t place = rows[(size_t)blockIdx.x * kDigitBins + d0];
    if (chunks > 1)
        place += sums[(size_t)(blockIdx.x / kDigitChunk) * kDigitBins + d0];
    const uint32_t all = sums[(chunks > 1 ? (size_t)chunks * kDigitBins : 0) + d0];
    for (uint32_t k = threadIdx.x; k < (uint32_t)(kDigitWaves * (kDigitBins + 2) / 2);
         k += kDigitThreads)
        reinterpret_cast<uint32_t *>(&cnt[0][0])[k] = 0;
    __syncthreads();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int j = 0; j < W::kItems; ++j) {
        const bool valid = k0 + j * 64 < m;
        const uint32_t d = digit(item[j]);
        const uint64_t peers = match_digit<kDigitBits>(d, __ballot(valid));
        const uint32_t c = cnt[w][d], mine = (uint32_t)__popcll(peers & lt);
        if (valid && mine == 0)
            cnt[w][d] = (uint16_t)(c + (uint32_t)__popcll(peers));
        rank[j] = c + mine;
    }
    __syncthreads();
    {   // the digit: where its words start in the tile and in the output
        uint32_t words = 0;
        for (int ww = 0; ww < kDigitWaves; ++ww)
            words += cnt[ww][d0];
        uint32_t total;
        uint32_t run = block_exclusive_scan(words, wsum, &total);
        to[d0] = block_exclusive_scan(all, wsum, &total) + place - run;
        for (int ww = 0; ww < kDigitWaves; ++ww) {
            const uint32_t t = cnt[ww][d0];
            cnt[ww][d0] = (uint16_t)run;
            run += t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < W::kItems; ++j)
        if (k0 + j * 64 < m)
            stage[cnt[w][digit(item[j])] + rank[j]] = item[j];
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < m; k += kDigitThreads) {
        const Item v = stage[k];
        const uint32_t at = to[digit(v)] + k;
        if (at < count)
            out[at] = v;
    }
}

namespace {
uint32_t digit_chunks(uint32_t tiles) { return (tiles + kDigitChunk - 1) / kDigitChunk; }
// Rows, chunk sums and totals of one pass (one chunk's sums are the totals).
template <class Item>
size_t digit_bytes(size_t count)
{
    const uint32_t tiles = nblk(count, Digits<Item>::kTile), chunks = digit_chunks(tiles);
    return ((size_t)tiles + chunks + (chunks > 1 ? 1 : 0)) * (4u << kDigitBits);
}
}  // namespace

size_t radix_digits_ws_bytes(size_t count)
{
    return digit_bytes<uint4>(count);   // (more than 8-byte items' half as many tiles)
}

template <class Source, class Digit>
static hipError_t digit_pass(const Source &src, typename Source::Item *dst, uint32_t count,
                             const Digit &digit, uint32_t *rows, hipStream_t s)
{
    const uint32_t tiles = nblk(count, Digits<typename Source::Item>::kTile);
    const uint32_t chunks = digit_chunks(tiles);
    uint32_t *const sums = rows + (size_t)tiles * kDigitBins;
    k_digits_up<<<tiles, kDigitThreads, 0, s>>>(src, count, digit, rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    k_digits_rows<<<dim3(chunks, kDigitBins / 256), 256, 0, s>>>(rows, tiles, sums);
    e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if (chunks > 1) {
        k_digits_chunks<<<kDigitBins / 4, 256, 0, s>>>(sums, chunks);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    k_digits_down<<<tiles, kDigitThreads, 0, s>>>(src, dst, count, digit, rows, sums, chunks);
    return hipGetLastError();
}

hipError_t radix_sort_words(uint64_t *a, uint64_t *b, uint32_t count, uint32_t low, uint32_t bits,
                            const KeySource *keys, void *ws, uint64_t **result, hipStream_t s)
{
    *result = a;
    if (keys && (count <= 1 || low != keys->ib || keys->cb < (uint32_t)kDigitBits))
        return hipErrorInvalidValue;
    if (count <= 1 || bits == 0)
        return hipSuccess;
    if (low + bits > 64)
        return hipErrorInvalidValue;
    uint64_t *src = a, *dst = b;
    for (bool first = true; bits > 0; first = false) {
        const uint32_t left = (bits + kDigitBits - 1) / kDigitBits;
        const uint32_t take = (bits + left - 1) / left;
        const DigitWord d{low, (1u << take) - 1};
        hipError_t e = first && keys
                           ? digit_pass(KeyWords{*keys}, dst, count, d, (uint32_t *)ws, s)
                           : digit_pass(ItemArray<uint64_t>{src}, dst, count, d, (uint32_t *)ws, s);
        if (e != hipSuccess)
            return e;
        low += take;
        bits -= take;
        uint64_t *t = src;
        src = dst;
        dst = t;
    }
    *result = src;
    return hipSuccess;
}

// Passes of 9-bit digits over `bits` bits of 16-byte items, from `in` (kept) to
// a, b, a, ...
template <class Make>
static hipError_t sort_items16(const void *in, void *a, void *b, uint32_t count, uint32_t bits,
                               void *ws, const void **result, hipStream_t s, Make &&make)
{
    *result = in;
    if (count <= 1)
        return hipSuccess;
    const uint4 *src = (const uint4 *)in;
    uint4 *dst = (uint4 *)a, *next = (uint4 *)b;
    for (uint32_t low = 0; low < bits;) {
        const uint32_t left = (bits - low + 8) / 9, take = (bits - low + left - 1) / left;
        hipError_t e = digit_pass(ItemArray<uint4>{src}, dst, count,
                                  make(low, (1u << take) - 1), (uint32_t *)ws, s);
        if (e != hipSuccess)
            return e;
        low += take;
        src = dst;
        uint4 *t = dst;
        dst = next;
        next = t;
    }
    *result = src;
    return hipSuccess;
}

hipError_t radix_sort_keyed(KV *a, KV *b, uint32_t count, uint32_t bits, void *ws,
                            const KV **result, hipStream_t s)
{
    const void *res = nullptr;
    hipError_t e = sort_items16(a, b, a, count, bits, ws, &res, s, [](uint32_t low, uint32_t mask) {
        return DigitKey{low, mask};
    });
    *result = (const KV *)res;
    return e;
}

hipError_t radix_sort_records(const Rec *in, Rec *a, Rec *b, uint32_t count,
                              const RecWidths &w, void *ws, const Rec **result, hipStream_t s)
{
    if (w.dur > 32 || w.tlo > 32 || w.j > 32 || w.i > 32)
        return hipErrorInvalidValue;
    const void *res = nullptr;
    hipError_t e = sort_items16(
        in, a, b, count, w.dur + w.tlo + w.j + w.i, ws, &res, s,
        [&](uint32_t low, uint32_t mask) {
            return DigitRec{w.dur, w.dur + w.tlo, w.j, (uint32_t)((1ull << w.tlo) - 1),
                            (uint32_t)((1ull << w.j) - 1), w.as_end ? 1u : 0u, low, mask};
        });
    *result = (const Rec *)res;
    return e;
}

// Per workgroup, the OR of every field of its records: i, j, t_lo, the duration
// t_hi - t_lo, and 1 if one is negative.
__global__ __launch_bounds__(256) void k_rec_widths(const Rec *__restrict__ in, uint32_t count,
                                                    uint32_t *__restrict__ part)
{
    __shared__ uint32_t red[4][kRecFields];
    uint32_t v[kRecFields] = {0, 0, 0, 0, 0};
    for (uint64_t k = (uint64_t)blockIdx.x * 256 + threadIdx.x; k < count;
         k += (uint64_t)gridDim.x * 256) {
        const Rec r = in[k];
        v[0] |= r.i;
        v[1] |= r.j;
        v[2] |= r.tlo;
        v[3] |= r.thi - r.tlo;
        v[4] |= r.thi < r.tlo ? 1u : 0u;
    }
    for (int f = 0; f < kRecFields; ++f) {
        for (int o = 32; o >= 1; o >>= 1)
            v[f] |= __shfl_xor(v[f], o, 64);
        if ((threadIdx.x & 63) == 0)
            red[threadIdx.x >> 6][f] = v[f];
    }
    __syncthreads();
    if (threadIdx.x < (uint32_t)kRecFields)
        part[blockIdx.x * kRecFields + threadIdx.x] = red[0][threadIdx.x] | red[1][threadIdx.x] |
                                                      red[2][threadIdx.x] | red[3][threadIdx.x];
}

hipError_t launch_rec_widths(const Rec *in, uint32_t count, uint32_t *part, hipStream_t s)
{
    k_rec_widths<<<kRecParts, 256, 0, s>>>(in, count, part);
    return hipGetLastError();
}

// ---- per-slab LDS radix sort ---------------------------------------------------------
//
// Block = kSegThreads (16 waves).  Wave w holds the keys with local index
// w * 64 * ITEMS + j * 64 + lane (item j) in registers.  Per 8-bit digit:
// rank inside the wave per item, scan the (digit, wave) counters, scatter keys
// and values as pairs through one LDS exchange buffer, read back.

constexpr int kSegWaves = kSegThreads / 64;
static_assert(kSegCap <= 65536, "a local index in 16 bits");

// Sorts the m <= kSegThreads * ITEMS keys of one workgroup by 32-bit key,
// stably, in four 8-bit digit passes; item j of lane `lane` of wave w is local
// index w * 64 * ITEMS + j * 64 + lane, before and after.  val (below 2^16)
// travels with key; during a pass its upper half holds the rank, which spares a
// register an item.  xch: kSegThreads * ITEMS pairs of LDS; cnt: kSegWaves * 257;
// wsum: 64.
template <int ITEMS>
__device__ inline void lds_sort32(uint32_t (&key)[ITEMS], uint32_t (&val)[ITEMS], uint32_t m,
                                  uint2 *xch, uint32_t *cnt, uint32_t *wsum)
{
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t li0 = (uint32_t)w * 64 * ITEMS + lane;
    uint64_t lt = lanemask_lt();
#pragma unroll 1
    for (int shift = 0; shift < 32; shift += 8) {
        for (int k = threadIdx.x; k < kSegWaves * 257; k += kSegThreads)
            cnt[k] = 0;
        __syncthreads();
        // rank inside (digit, wave)
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            uint32_t li = li0 + j * 64;
            bool valid = li < m;
            uint32_t d = (key[j] >> shift) & 0xFFu;
            uint64_t peers = match_digit(d, __ballot(valid));
            uint32_t c = valid ? cnt[w * 257 + d] : 0u;
            uint32_t mine = (uint32_t)__popcll(peers & lt);
            if (valid && mine == 0)
                cnt[w * 257 + d] = c + (uint32_t)__popcll(peers);
            val[j] |= (c + mine) << 16;
        }
        __syncthreads();
        {   // exclusive scan of the 4096 counters in (digit, wave) order
            uint32_t v[4], sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t o = threadIdx.x * 4 + q;   // (digit, wave) order
                v[q] = cnt[(o % kSegWaves) * 257 + o / kSegWaves];
                sum += v[q];
            }
            uint32_t total;
            uint32_t run = block_exclusive_scan(sum, wsum, &total);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t o = threadIdx.x * 4 + q;
                cnt[(o % kSegWaves) * 257 + o / kSegWaves] = run;
                run += v[q];
            }
        }
        __syncthreads();
        int again = shift;   // opaque: the digits are formed anew, not kept (and spilled)
        asm volatile("" : "+s"(again));
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (li0 + j * 64 < m)
                xch[cnt[w * 257 + ((key[j] >> again) & 0xFFu)] + (val[j] >> 16)] =
                    make_uint2(key[j], val[j] & 0xFFFFu);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (li0 + j * 64 < m) {
                const uint2 x = xch[li0 + j * 64];
                key[j] = x.x;
                val[j] = x.y;
            }
    }
}

template <int PREC, int TP, bool CODES>
__global__ __launch_bounds__(kSegThreads) void k_slab_build(
    BoxView b, uint32_t slab_size, uint32_t N, uint32_t slab_ticks,
    const unsigned long long *bounds, uint32_t *__restrict__ codes_out, void *tree,
    unsigned int *err)
{
    __shared__ uint2 pairs[kSegCap];
    // counters of (digit, wave), stored wave-major with a 257-word row (see
    // k_radix_downsweep): index w * 257 + d
    __shared__ uint32_t cnt[kSegWaves * 257];
    __shared__ uint32_t wsum[64];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t slab = blockIdx.x;
    uint64_t base = slab * slab_size;
    uint32_t m = slab_size;
    if (base + m > N)
        m = base < N ? (uint32_t)(N - base) : 0u;
    double mn[3], inv[3];
    for (int d = 0; d < 3; ++d) {   // the frame is read only when codes are formed here
        mn[d] = inv[d] = 0.0;
        if (!CODES) {
            mn[d] = from_ordered_bits(bounds[d]);
            double ext = from_ordered_bits(bounds[3 + d]) - mn[d];
            inv[d] = ext > 0.0 ? 1.0 / ext : 0.0;
        }
    }
    uint32_t key[kSegItems], val[kSegItems];
    uint32_t li0 = (uint32_t)w * 64 * kSegItems + lane;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kSegItems; ++j) {
        uint32_t li = li0 + j * 64;
        key[j] = 0xFFFFFFFFu;
        if (li < m) {
            if (CODES) {   // codes written with the boxes: 4 bytes instead of 48
                key[j] = b.code[base + li];
            } else {
                double lo[3], hi[3];
                load_box<PREC>(b, base + li, lo, hi);
                key[j] = morton30(0.5 * (lo[0] + hi[0]), 0.5 * (lo[1] + hi[1]),
                                  0.5 * (lo[2] + hi[2]), mn, inv);
            }
            bad |= (b.t0[base + li] / slab_ticks) != slab;
        }
        val[j] = li;
    }
    if (bad)
        atomicOr(err, 1u);
    lds_sort32(key, val, m, pairs, cnt, wsum);
    __syncthreads();
    // Leaf records.  Reading boxes by sorted position would gather 4-8 byte
    // words from all over the slab; instead each box is read in source order
    // (coalesced) and its whole record is written to its sorted slot.  LDS
    // holds the sorted codes (for the skip links) and the inverse permutation.
    uint32_t *const xch = reinterpret_cast<uint32_t *>(pairs);
    uint32_t *const vsrc = xch + kSegCap;   // source box -> sorted position
#pragma unroll
    for (int j = 0; j < kSegItems; ++j) {
        uint32_t p = li0 + j * 64;
        if (p < m) {
            xch[p] = key[j];
            vsrc[val[j]] = p;
            // the sorted 32-bit codes (a slab's key bits above them are its
            // index); streaming stores: lanes write consecutive words
            __builtin_nontemporal_store(key[j], &codes_out[base + p]);
        }
    }
    __syncthreads();
    const SlabKeys32 K{xch, (uint32_t)base, slab_size, (uint32_t)slab};
    // kScatterBatch boxes per lane at a time: their loads are all in flight
    // before the first record is written
    constexpr int kScatterBatch = 4;
#pragma unroll 1
    for (uint32_t l0 = threadIdx.x; l0 < m; l0 += kSegThreads * kScatterBatch) {
        double lo[kScatterBatch][3], hi[kScatterBatch][3];
        uint32_t t0[kScatterBatch], t1[kScatterBatch], ob[kScatterBatch];
#pragma unroll
        for (int q = 0; q < kScatterBatch; ++q) {
            uint32_t li = l0 + q * kSegThreads;
            if (li < m) {
                uint64_t src = base + li;
                load_box<PREC>(b, src, lo[q], hi[q]);
                t0[q] = b.t0[src];
                t1[q] = b.t1[src];
                ob[q] = b.obj[src];
            }
        }
#pragma unroll
        for (int q = 0; q < kScatterBatch; ++q) {
            uint32_t li = l0 + q * kSegThreads;
            if (li < m) {
                uint32_t p = vsrc[li];
                uint32_t esc = slab_escape32(K, N, (uint32_t)(base + p));
                NodeIO<TP>::put(tree, N, (uint32_t)(N - 1 + base + p), lo[q], hi[q], t0[q],
                                t1[q], ob[q], esc);
            }
        }
    }
}


// Per-object Morton order of each block of slabs: block B's unsorted codes
// (code of object i at ucode[i * es]) are sorted with their object ids; rank
// r's code and object go to scode[r * es] and sobj[r * es].  One workgroup
// per block; blocks are `stride` entries (of es words) apart.
// Run r (grid.y) of block b (grid.x): entries [r S, min(n, (r + 1) S)) of
// the block (entry k at (b stride + k) es words) sorted in LDS by code,
// stable, each with its block-local index; written to the same entries of
// scode / sobj.  With one run (S = n) that is the block's whole order.
//
// ITEMS: keys per lane, chosen to just hold a run (the ranking, 32 instructions
// a key and digit, is done for every place).  Bound: the four digit passes of a
// workgroup, from 5 keys a lane on alone on its CU.  Against 17 keys a lane for
// every size, keys and values exchanged apart: 8 blocks of 1 000 53 -> 9.5 us,
// 150 of 4 999 62 -> 19; 450 blocks of 16 848 121 -> 100 (two rounds of
// workgroups), where the ranks are kept in 16 bits so that no register spills.
template <int ITEMS>
__global__ __launch_bounds__(kSegThreads) void k_block_sort(const uint32_t *ucode, uint32_t n,
                                                            uint32_t S, uint64_t stride,
                                                            uint32_t es, uint32_t *scode,
                                                            uint32_t *sobj)
{
    __shared__ uint2 xch[kSegThreads * ITEMS];
    __shared__ uint32_t cnt[kSegWaves * 257];
    __shared__ uint32_t wsum[64];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t r0 = blockIdx.y * S;
    if (r0 >= n)
        return;   // (the whole workgroup)
    const uint32_t m = n - r0 < S ? n - r0 : S;
    uint64_t base = (uint64_t)blockIdx.x * stride + r0;
    uint32_t key[ITEMS], val[ITEMS];
    uint32_t li0 = (uint32_t)w * 64 * ITEMS + lane;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        uint32_t li = li0 + j * 64;
        key[j] = li < m ? ucode[(base + li) * es] : 0xFFFFFFFFu;
        val[j] = li;
    }
    lds_sort32(key, val, m, xch, cnt, wsum);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        uint32_t r = li0 + j * 64;
        if (r < m) {
            scode[(base + r) * es] = key[j];
            sobj[(base + r) * es] = r0 + val[j];
        }
    }
}

static hipError_t block_sort_runs(const uint32_t *ucode, uint32_t n, uint32_t S, uint32_t R,
                                  uint32_t nblocks, uint64_t stride, uint32_t es,
                                  uint32_t *scode, uint32_t *sobj, hipStream_t s)
{
    auto run = [&](auto kernel) {
        kernel<<<dim3(nblocks, R), kSegThreads, 0, s>>>(ucode, n, S, stride, es, scode, sobj);
        return hipGetLastError();
    };
    const uint32_t items = (S + kSegThreads - 1) / kSegThreads;
    return items <= 1   ? run(k_block_sort<1>)
           : items <= 2 ? run(k_block_sort<2>)
           : items <= 3 ? run(k_block_sort<3>)
           : items <= 5 ? run(k_block_sort<5>)
           : items <= 8 ? run(k_block_sort<8>)
           : items <= 12 ? run(k_block_sort<12>)
                         : run(k_block_sort<kSegItems>);
}

// The R sorted runs of each block merged: entry e of run r goes to position
// (its index in run r) + (entries of earlier runs with a code <= its code) +
// (entries of later runs with a smaller code), which is its place in the
// block's (code, index) order, as one stable sort of the whole block gives.
__global__ __launch_bounds__(256) void k_block_merge(const uint32_t *rcode, const uint32_t *robj,
                                                     uint32_t n, uint32_t S, uint32_t R,
                                                     uint64_t stride, uint32_t es,
                                                     uint32_t *scode, uint32_t *sobj)
{
    const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n)
        return;
    const uint64_t base = (uint64_t)blockIdx.y * stride;
    const uint32_t r = e / S;
    const uint32_t x = rcode[(base + e) * es], id = robj[(base + e) * es];
    uint32_t rank = e - r * S;
    for (uint32_t q = 0; q < R; ++q) {
        if (q == r)
            continue;
        const uint32_t lo0 = q * S, len = n - lo0 < S ? n - lo0 : S;
        // entries of run q before x: code <= x (q < r) or code < x (q > r)
        uint32_t lo = 0, hi = len;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1, c = rcode[(base + lo0 + mid) * es];
            if (q < r ? c <= x : c < x)
                lo = mid + 1;
            else
                hi = mid;
        }
        rank += lo;
    }
    scode[(base + rank) * es] = x;
    sobj[(base + rank) * es] = id;
}

hipError_t launch_block_sort(const uint32_t *ucode, uint32_t n, uint32_t nblocks, uint64_t stride,
                             uint32_t es, uint32_t *scode, uint32_t *sobj, uint32_t *rcode,
                             uint32_t *robj, hipStream_t s)
{
    if (n == 0 || nblocks == 0)
        return hipSuccess;
    const uint32_t R = (uint32_t)((n + kSegCap - 1) / kSegCap);
    if (R > (uint32_t)kBlockRuns || (R > 1 && (!rcode || !robj)))
        return hipErrorInvalidValue;
    const uint32_t S = (n + R - 1) / R;
    if (R == 1)
        return block_sort_runs(ucode, n, S, 1, nblocks, stride, es, scode, sobj, s);
    hipError_t e = block_sort_runs(ucode, n, S, R, nblocks, stride, es, rcode, robj, s);
    if (e != hipSuccess)
        return e;
    k_block_merge<<<dim3((n + 255) / 256, nblocks), 256, 0, s>>>(rcode, robj, n, S, R, stride, es,
                                                                  scode, sobj);
    return hipGetLastError();
}

hipError_t launch_slab_build(const BoxView &b, int box_precision, int tree_precision,
                             uint32_t nslabs, uint32_t slab_size, uint32_t N,
                             uint32_t slab_ticks, const unsigned long long *bounds,
                             uint32_t *codes_out, void *tree, unsigned int *err,
                             hipStream_t s)
{
    if (nslabs == 0 || N == 0)
        return hipSuccess;
    if ((int64_t)slab_size > kSegCap)
        return hipErrorInvalidValue;
#define CD_SLAB_LAUNCH(P, T, C)                                                             \
    k_slab_build<P, T, C><<<nslabs, kSegThreads, 0, s>>>(b, slab_size, N, slab_ticks, bounds,  \
                                                         codes_out, tree, err)
    const bool codes = b.code != nullptr;
    if (box_precision == CD_FP64 && tree_precision == CD_FP64) {
        if (codes)
            CD_SLAB_LAUNCH(CD_FP64, CD_FP64, true);
        else
            CD_SLAB_LAUNCH(CD_FP64, CD_FP64, false);
    } else if (box_precision == CD_FP64) {
        if (codes)
            CD_SLAB_LAUNCH(CD_FP64, CD_FP32, true);
        else
            CD_SLAB_LAUNCH(CD_FP64, CD_FP32, false);
    } else {
        if (codes)
            CD_SLAB_LAUNCH(CD_FP32, CD_FP32, true);
        else
            CD_SLAB_LAUNCH(CD_FP32, CD_FP32, false);
    }
#undef CD_SLAB_LAUNCH
    return hipGetLastError();
}

} // namespace cd
