// rt_split_seg_kernels.h -- splitter passes over long segments: large arrays
// of 64-bit keys (one or two such passes, then leaves) and the long segments
// of batched calls (one pass, then leaves).
//
// A pass cuts every listed segment into up to 256 buckets of neighbouring
// keys and writes them, stably, to the segment's other arrays.  Against the
// 8-bit digit passes of the onesweep form:
//
// * the buckets are chosen from a sample of the segment, so they come out
//   about equal for any distribution of keys, and two passes leave ranges
//   that one block sorts whole in LDS, whatever the key width; four or eight
//   digit passes become two and a leaf;
// * the tiles' counts are taken beforehand, one row of a table per tile, so a
//   tile knows where its runs go without a lookback chain, and tiles may run
//   in any order: each XCD takes a contiguous share of them, so that
//   neighbouring runs, which share cache lines, are written through one L2.
//
// Measured, 2^26 pairs of 64-bit keys with 4-byte values: scatter 350 us a
// pass (24 bytes an item, 4.6 TB/s: an eight-bit digit pass takes 342), count
// 119 (4.5 TB/s), leaves 443, the rest 90; 1814 a sort with its input copy,
// against 3311 by eight digit passes.  2^27 pairs of 32-bit keys in batched
// segments: 1730 us a call against 2787 by four digit passes.
//
// Launches of a pass: k_split_sample (buckets of each segment),
// k_split_tile_count (rows), k_split_scan (rows to prefix sums, totals),
// k_split_starts (bucket bounds: the next pass's segments, or leaf lists) and
// k_split_tile_scatter; then k_split_leaves per leaf size.
#pragma once

#include "rt_seg_kernels.h"
#include "rt_split_kernels.h"

namespace rt {

// A segment's buckets, in its row of the histogram table (kSegPasses *
// kSegRadix words): the buckets' item totals, this, the splitters.
struct SplitSeg {
    uint64_t lo;       // linear: key of bucket 0's start
    uint32_t scale;    // linear: bucket = umulhi((key - lo) >> shift, scale)
    uint32_t shift;
    uint32_t linear;   // 1: equal stretches of the key range; 0: splitters
    uint32_t buckets;  // at most kBuckets
    uint32_t pad[2];
};
constexpr int kSplitRowBytes = kSegPasses * kSegRadix * 4;
constexpr int kSplitSegAt = 1024, kSplittersAt = 2048;
static_assert(kSplittersAt + kBuckets * 8 <= kSplitRowBytes, "64-bit splitters fit the row");

// One leaf of n items: where it starts in the arrays that hold the segments'
// k/v and tk/tv, and whether it holds a single key value (in order as it
// stands).
struct SplitLeaf {
    uint32_t at_k, at_tk, n, one;
};
// Those arrays.
template <typename K, typename V>
struct LeafArrays {
    K *k;
    V *v;
    K *tk;
    V *tv;
};
// Leaf classes (kLeafClasses): what 256-thread blocks hold (17 items a thread;
// 16 of 64-bit keys, so that three such blocks fit a CU's LDS), what the
// largest blocks hold, longer ones, ones for the whole grid.
template <typename K>
constexpr int leaf_ipt() {
    return sizeof(K) == 4 ? 17 : 16;
}
template <typename K>
constexpr uint32_t leaf_max() {
    return sizeof(K) == 4 ? 1024u * 16u : 1024u * 8u;
}

// Items per leaf aimed at: leaves of equal stretches of spread keys then stay
// within four standard deviations of what 256 x 17 blocks hold (4352 items) up
// to segments of 2^20 items.  Fuller leaves cost less per item (a leaf's bins
// are scanned whole): 2^27 pairs in segments of up to 2^20 took 577 us in
// leaves of 1536 to 3072 items.  Blocks of 256 x 16 with 64-bit keys: three to
// a CU instead of two, 2^26 pairs 1858 -> 1814 us a sort.
template <typename K>
constexpr uint32_t leaf_aim() {
    return sizeof(K) == 4 ? 3900u : 3650u;
}

// Quantiles of a sample are less even (30 sample keys a bucket of 2^18 items:
// 18 percent), and a leaf that does not fit 256 threads costs most: items per
// leaf of theirs.  2000 segments of 2^6 to 2^20 keys that are ANDs of four
// words: 1504 -> 1407 us a call.  Batched calls of few items take half of
// that: each then has fewer leaves than the chip has blocks, and a leaf for
// the largest blocks costs the call a launch with work in it (4 segments of
// 2^16 to 2^18 repeated keys: 119.6 -> 88.2 us, by digit passes 91.9); with
// 35 million items the smaller leaves cost more than they save (ANDs of four
// words: 869 -> 929 us).
constexpr uint32_t kQuantileAim = 2900;
constexpr uint32_t kQuantileAimFew = 1500;
constexpr size_t kFewLeafItems = static_cast<size_t>(1) << 24;

__device__ __forceinline__ uint32_t split_bucket_count(uint32_t n, uint32_t aim) {
    return min((n + aim - 1u) / aim, static_cast<uint32_t>(kBuckets));
}

// Buckets of a segment's keys, held in a block.
template <typename K>
struct Splitter {
    K lo;
    uint32_t scale, shift, linear, last;
    const K *split;  // LDS: the tree of kBuckets - 1 (past the segment's: the largest key)
    __device__ __forceinline__ uint32_t stretch(K key) const {
        const K d = key > lo ? static_cast<K>(key - lo) : K(0);
        const K x = d >> shift;
        const uint32_t y = sizeof(K) == 8 && (static_cast<uint64_t>(x) >> 32) ? ~0u : static_cast<uint32_t>(x);
        return min(last, __umulhi(y, scale));
    }
    __device__ __forceinline__ uint32_t search(K key) const { return min(last, bucket_of(key, split)); }
    __device__ __forceinline__ uint32_t operator()(K key) const { return linear ? stretch(key) : search(key); }
};

// The buckets of the segment with this row; every thread calls it, and a
// barrier follows before the splitter is used.
template <int BLOCK, typename K>
__device__ __forceinline__ Splitter<K> load_splitter(const char *rows, uint32_t row, K *lds_split) {
    const char *r = rows + static_cast<size_t>(row) * kSplitRowBytes;
    const SplitSeg *s = reinterpret_cast<const SplitSeg *>(r + kSplitSegAt);
    Splitter<K> f;
    f.lo = static_cast<K>(s->lo);
    f.scale = s->scale;
    f.shift = s->shift;
    f.linear = s->linear;
    f.last = s->buckets - 1u;
    f.split = lds_split;
    if (!f.linear)
        for (uint32_t i = threadIdx.x; i < static_cast<uint32_t>(kBuckets); i += BLOCK)
            if (i > 0) lds_split[i] = reinterpret_cast<const K *>(r + kSplittersAt)[tree_index(i)];
    return f;
}

// Stratified sample of m keys of a segment of n items (m may exceed n).
template <typename K>
struct SegSample {
    const K *k;
    uint32_t n, m;
    __device__ __forceinline__ K key(uint32_t i, uint32_t c = 0) const {
        i += c;
        const uint32_t a = static_cast<uint32_t>(static_cast<uint64_t>(i) * n / m);
        const uint32_t b = static_cast<uint32_t>(static_cast<uint64_t>(i + 1) * n / m);
        return k[min(a + __umulhi((i + 1u) * 0x9E3779B9u, b - a), n - 1u)];
    }
    __device__ __forceinline__ uint32_t val(uint32_t, uint32_t = 0) const { return 0u; }
};
// Takes the quantiles of the sorted sample, every EVERYth key and the last.
template <typename K, uint32_t EVERY>
struct QuantileSink {
    K *picked;
    K *sorted;
    uint32_t buckets, m;
    __device__ __forceinline__ void put(uint32_t base, uint32_t i, K key, uint32_t) const {
        i += base;
        // the first key to complete q + 1 of the buckets' equal shares of m
        const uint32_t q = (i + 1u) * buckets / m;
        if (q != i * buckets / m && q < buckets) picked[q - 1u] = key;
        if (i % EVERY == 0) sorted[i / EVERY] = key;
        if (i == m - 1u) sorted[m / EVERY] = key;
    }
};

// Chooses every listed segment's buckets (fixed_buckets of them if set, else
// as many as its leaves need, of quantile_aim items where quantiles cut them) from BLOCK * SIPT sample keys, and writes its
// tiles' entries of the tile map (as k_seg_tilemap).  2048 sample keys serve
// a pass with leaves: 8192 gave better leaves only to keys of uneven density,
// and cost 60 us more in random reads at 2^28 items.  The buckets are equal
// stretches of the sampled range if no stretch holds far more of the sample
// than its share (no bucket much above the mean, and a key's bucket costs one
// multiplication: 350 us a scatter of 2^26 64-bit pairs, 440 by search), else
// the sample's quantiles.  Bound by latency: random reads, then the sample's
// sort (12 us for 2048 keys, 27 for 8192, with 2^22 items).
template <int BLOCK, int SIPT, typename K>
__global__ __launch_bounds__(BLOCK) void k_split_sample(const SegDesc *__restrict__ descs,
                                                        const uint32_t *__restrict__ list,
                                                        const SegHeader *__restrict__ h,
                                                        const uint32_t *__restrict__ first_tile,
                                                        SegDesc *__restrict__ tile_desc, char *__restrict__ rows,
                                                        uint32_t fixed_buckets, uint32_t quantile_aim) {
    constexpr uint32_t m = BLOCK * SIPT;
    __shared__ BlockSortLds<BLOCK, SIPT, K, uint32_t, false> sort;
    __shared__ K picked[kBuckets];
    constexpr uint32_t EVERY = m * sizeof(K) > 32768 ? 2 : 1;  // (64 KB of LDS more would be too much)
    __shared__ K sorted[m / EVERY + 1];
    __shared__ uint32_t hits[kBuckets];
    __shared__ SplitSeg seg;
    const uint32_t tid = threadIdx.x;
    const uint32_t count = h->count[kSegLarge];
    for (uint32_t e = blockIdx.x; e < count; e += gridDim.x) {
        const SegDesc d = descs[list[e]];
        const uint32_t n = d.n;
        char *row = rows + static_cast<size_t>(d.row) * kSplitRowBytes;
        // (d.pass set: a segment of one key value)
        const uint32_t stretches = d.pass ? 1u : fixed_buckets ? fixed_buckets : split_bucket_count(n, leaf_aim<K>());
        const uint32_t buckets = d.pass ? 1u : fixed_buckets ? fixed_buckets : split_bucket_count(n, quantile_aim);
        {
            SegDesc t = d;
            t.pad = first_tile[e];
            const uint32_t end = first_tile[e + 1];
            for (uint32_t i = t.pad + tid; i < end; i += BLOCK) tile_desc[i] = t;
        }
        const SegSample<K> src{reinterpret_cast<const K *>(d.k), n, m};
        if (tid < kBuckets) {
            picked[tid] = ~K(0);
            hits[tid] = 0u;
        }
        __syncthreads();
        if (buckets > 1)
            block_sort<BLOCK, SIPT, K, uint32_t, false>(src, m, QuantileSink<K, EVERY>{picked, sorted, buckets, m},
                                                        false, sort);
        __syncthreads();
        if (tid == 0) {
            seg.lo = 0;
            seg.scale = seg.shift = 0u;
            seg.linear = 1u;
            seg.buckets = buckets;
            seg.pad[0] = seg.pad[1] = 0u;
            if (buckets > 1) {
                // the sampled range, widened by a sample's mean distance
                const uint64_t a = sorted[0], b = sorted[m / EVERY], top = ~K(0);
                const uint64_t w = (b - a) / m;
                const uint64_t lo = a - min(a, w), hi = b + min(top - b, w);
                const uint32_t bits = key_bits_of(hi - lo);
                seg.shift = bits > 32u ? bits - 32u : 0u;
                const uint64_t span = ((hi - lo) >> seg.shift) + 1u;
                seg.lo = lo;
                seg.linear = span >= 16u * stretches ? 1u : 0u;  // else a stretch is a few values, and uneven
                seg.scale = seg.linear ? static_cast<uint32_t>((static_cast<uint64_t>(stretches) << 32) / span) : 0u;
            }
        }
        __syncthreads();
        if (buckets > 1 && seg.linear) {
            Splitter<K> f;
            f.lo = static_cast<K>(seg.lo);
            f.scale = seg.scale;
            f.shift = seg.shift;
            f.last = stretches - 1u;
            for (uint32_t i = tid; i < m / EVERY; i += BLOCK) atomicAdd(&hits[f.stretch(sorted[i])], 1u);
            __syncthreads();
            // a share of mean s: 6 standard deviations, s + 6 sqrt(s)
            const uint32_t s = m / EVERY / stretches;
            if (tid < stretches && hits[tid] > s && (hits[tid] - s) * (hits[tid] - s) > 36u * s) seg.linear = 0u;
            __syncthreads();
        }
        if (tid < kBuckets - 1) {
            // v the first time, v + 1 from then on (at the largest key: v)
            const K v = picked[tid];
            reinterpret_cast<K *>(row + kSplittersAt)[tid] = tid > 0 && picked[tid - 1] == v && v != ~K(0) ? v + 1u : v;
        }
        if (tid == 0) {
            if (seg.linear) seg.buckets = stretches;
            *reinterpret_cast<SplitSeg *>(row + kSplitSegAt) = seg;
        }
        __syncthreads();
    }
}

// The tile of this block: each XCD (blocks are dealt to them in turn) takes a
// contiguous eighth of the tiles.  Any order is correct.
__device__ __forceinline__ uint32_t split_tile_of(uint32_t block, uint32_t tiles) {
    const uint32_t per = (tiles + kChunks - 1u) / kChunks;
    const uint32_t q = block / kChunks;
    return q < per ? (block % kChunks) * per + q : kNoTile;
}

// Row t of `table`: tile t's items per bucket.
template <int BLOCK, typename K>
__global__ __launch_bounds__(BLOCK) void k_split_tile_count(const SegDesc *__restrict__ tile_desc,
                                                            const SegHeader *__restrict__ h,
                                                            const char *__restrict__ rows,
                                                            uint32_t *__restrict__ table, uint32_t tile_items) {
    constexpr int C = 8;  // lane-class copies of the counters, as in k_histogram
    constexpr int U = 16;  // keys in flight per lane
    __shared__ K split[kBuckets];
    __shared__ uint32_t count[C][kBuckets + 1];
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t total = h->total_tiles;
    const uint32_t tile = split_tile_of(blockIdx.x, total);
    if (tile >= total) return;
    const SegDesc d = tile_desc[tile];
    const uint32_t start = (tile - d.pad) * tile_items;
    const uint32_t valid = min(tile_items, d.n - start);
    const K *src = reinterpret_cast<const K *>(d.k) + start;
    if (reinterpret_cast<const SplitSeg *>(rows + static_cast<size_t>(d.row) * kSplitRowBytes + kSplitSegAt)->buckets == 1u) {
        for (uint32_t i = tid; i < static_cast<uint32_t>(kBuckets); i += BLOCK)
            table[static_cast<size_t>(tile) * kBuckets + i] = i == 0 ? valid : 0u;
        return;
    }
    // the first keys are on their way while the splitters are read
    K k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = *gptr<K, true>(src, min(u * BLOCK + tid, valid - 1u));
    const Splitter<K> f = load_splitter<BLOCK, K>(rows, d.row, split);
    for (uint32_t i = tid; i < C * (kBuckets + 1); i += BLOCK) (&count[0][0])[i] = 0u;
    __syncthreads();
    uint32_t *mine = count[lane % C];
    for (uint32_t base = 0; base < valid; base += BLOCK * U) {
        uint32_t b[U];
        if (f.linear) {
#pragma unroll
            for (int u = 0; u < U; ++u) b[u] = f.stretch(k[u]);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) b[u] = f.search(k[u]);
        }
        if (base + BLOCK * U < valid) {  // the next keys
#pragma unroll
            for (int u = 0; u < U; ++u) k[u] = *gptr<K, true>(src, min(base + (U + u) * BLOCK + tid, valid - 1u));
        }
        const uint32_t b0 = __builtin_amdgcn_readfirstlane(b[0]);
        uint32_t differ = base + BLOCK * U <= valid ? 0u : 1u;
#pragma unroll
        for (int u = 0; u < U; ++u) differ |= b[u] ^ b0;
        if (__builtin_amdgcn_ballot_w64(differ != 0u) == 0) {
            if (lane == 0) atomicAdd(&mine[b0], static_cast<uint32_t>(64 * U));
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (base + u * BLOCK + tid < valid) atomicAdd(&mine[b[u]], 1u);
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < static_cast<uint32_t>(kBuckets); i += BLOCK) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < C; ++w) c += count[w][i];
        table[static_cast<size_t>(tile) * kBuckets + i] = c;
    }
}

// The tiles of a segment are summed in chunks of kScanChunk; a chunk's row in
// the chunk table.
constexpr uint32_t kScanChunk = 2048;
__device__ __forceinline__ uint32_t chunk_row(uint32_t first_tile, uint32_t row, uint32_t tile) {
    return first_tile / kScanChunk + row + (tile - first_tile) / kScanChunk;
}

// Per listed segment, 32 of its buckets and chunk blockIdx.y of its tiles:
// the tiles' rows become exclusive prefix sums inside the chunk, and the
// chunk's totals go to the chunk table.  32 threads share a bucket's rows,
// eight loads in flight each.
static __global__ __launch_bounds__(1024) void k_split_scan(const uint32_t *__restrict__ first_tile,
                                                            const SegHeader *__restrict__ h,
                                                            uint32_t *__restrict__ table,
                                                            uint32_t *__restrict__ chunks) {
    constexpr uint32_t SLICES = kBuckets / 32;
    constexpr int U = 8;
    __shared__ uint32_t sums[32][33];
    const uint32_t b = threadIdx.x & 31u, g = threadIdx.x >> 5;
    const uint32_t work = h->count[kSegLarge] * SLICES;
    for (uint32_t w = blockIdx.x; w < work; w += gridDim.x) {
        const uint32_t e = w / SLICES, col = (w % SLICES) * 32u + b;
        const uint32_t f = first_tile[e];
        const uint32_t t0 = f + blockIdx.y * kScanChunk;
        if (t0 >= first_tile[e + 1]) continue;
        const uint32_t tiles = min(first_tile[e + 1] - t0, kScanChunk);
        const uint32_t lo = t0 + g * tiles / 32u, hi = t0 + (g + 1u) * tiles / 32u;
        uint32_t sum = 0;
        for (uint32_t t = lo; t < hi; t += U) {
            uint32_t c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = table[static_cast<size_t>(min(t + u, hi - 1u)) * kBuckets + col];
#pragma unroll
            for (int u = 0; u < U; ++u) sum += t + u < hi ? c[u] : 0u;
        }
        sums[g][b] = sum;
        __syncthreads();
        uint32_t run = 0;
        for (uint32_t q = 0; q < g; ++q) run += sums[q][b];
        if (g == 31u) chunks[static_cast<size_t>(chunk_row(f, e, t0)) * kBuckets + col] = run + sum;
        for (uint32_t t = lo; t < hi; t += U) {
            uint32_t c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = table[static_cast<size_t>(min(t + u, hi - 1u)) * kBuckets + col];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t + u < hi) {
                    table[static_cast<size_t>(t + u) * kBuckets + col] = run;
                    run += c[u];
                }
        }
        __syncthreads();
    }
}

// Per listed segment: its chunks' totals become prefix sums, its buckets'
// totals go to its row, and where the buckets start: sub set (one segment):
// to sub[0..kBuckets], the segments of the next pass, and a bit for each that
// holds one key value, from sub[kSubOnes]; lists set: a leaf per bucket that is
// not in order as it stands (of every bucket, if `all`: the leaves go to other
// arrays) to the list of its size.
constexpr uint32_t kSubOnes = kBuckets + 4;
template <typename K>
__global__ __launch_bounds__(256) void k_split_starts(const SegDesc *__restrict__ descs,
                                                      const uint32_t *__restrict__ list,
                                                      SegHeader *__restrict__ h,
                                                      const uint32_t *__restrict__ first_tile, char *__restrict__ rows,
                                                      uint32_t *__restrict__ chunks, uint32_t *__restrict__ sub,
                                                      const K *k0, const K *tk0, LeafLists *__restrict__ lists,
                                                      SplitLeaf *__restrict__ leaves, uint32_t all) {
    __shared__ uint32_t s_wsum[4];
    __shared__ uint32_t all_one;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t count = h->count[kSegLarge];
    if (tid == 0) all_one = 0u;
    for (uint32_t e = blockIdx.x; e < count; e += gridDim.x) {
        const SegDesc d = descs[list[e]];
        char *row = rows + static_cast<size_t>(d.row) * kSplitRowBytes;
        const uint32_t f = first_tile[e], tiles = first_tile[e + 1] - f;
        uint32_t c = 0;
        for (uint32_t t = 0; t < tiles; t += kScanChunk) {
            uint32_t *p = chunks + static_cast<size_t>(chunk_row(f, e, f + t)) * kBuckets + tid;
            const uint32_t x = *p;
            *p = c;
            c += x;
        }
        reinterpret_cast<uint32_t *>(row)[tid] = c;
        const uint32_t start = block_exclusive_sum<256>(c, s_wsum);
        const SplitSeg *seg = reinterpret_cast<const SplitSeg *>(row + kSplitSegAt);
        const K *split = reinterpret_cast<const K *>(row + kSplittersAt);
        uint32_t one = d.pass;  // the bucket holds one key value
        if (!seg->linear && tid > 0)
            one = tid + 1u < seg->buckets ? (static_cast<K>(split[tid] - split[tid - 1]) == K(1))
                                          : (split[tid - 1] == ~K(0));
        if (sub != nullptr) {
            // one value in all: the segment is in order, nothing is left to do
            if (one && c == d.n) all_one = 1u;
            __syncthreads();
            const bool done = all_one != 0u;
            sub[tid] = done ? 0u : start;
            if (tid == 255) sub[256] = done ? 0u : d.n;
            const uint64_t ones = __builtin_amdgcn_ballot_w64(one != 0u);
            if (lane == 0) {
                sub[kSubOnes + tid / 32] = static_cast<uint32_t>(ones);
                sub[kSubOnes + tid / 32 + 1] = static_cast<uint32_t>(ones >> 32);
            }
            if (done && tid == 0) h->total_tiles = 0u;
        }
        if (lists != nullptr) {
            const uint32_t at_k = static_cast<uint32_t>(reinterpret_cast<const K *>(d.k) - k0);
            const uint32_t at_tk = static_cast<uint32_t>(reinterpret_cast<const K *>(d.tk) - tk0);
            int q = -1;
            constexpr uint32_t small = 256u * leaf_ipt<K>();
            if (one) {
                // in place, one value is in order already; else it is copied,
                // by as many blocks as have a leaf of it
                const uint32_t parts = all ? (c + small - 1u) / small : 0u;
                uint32_t at = parts ? atomicAdd(&lists->count[0], parts) : 0u;
                for (uint32_t i = 0; i < c && parts; i += small, ++at)
                    if (at < lists->capacity)
                        leaves[at] = SplitLeaf{at_k + start + i, at_tk + start + i, min(small, c - i), 1u};
            } else if (c >= (all ? 1u : 2u)) {
                q = c <= small ? 0 : c <= leaf_max<K>() ? 1 : c <= kAloneMax ? 2 : 3;
            }
#pragma unroll
            for (int i = 0; i < kLeafClasses; ++i) {
                const uint64_t mine = __builtin_amdgcn_ballot_w64(q == i);
                if (mine == 0) continue;
                uint32_t first = 0;
                if (lane == 0) first = atomicAdd(&lists->count[i], static_cast<uint32_t>(__popcll(mine)));
                first = __shfl(first, 0, 64);
                const uint32_t at = first + __builtin_amdgcn_mbcnt_hi(
                                                static_cast<uint32_t>(mine >> 32),
                                                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mine), 0u));
                if (q == i && at < lists->capacity)
                    leaves[static_cast<size_t>(i) * lists->capacity + at] =
                        SplitLeaf{at_k + start, at_tk + start, c, 0u};
            }
        }
        __syncthreads();
    }
}

// Scatters the tile of this block by bucket from k/v to tk/tv of its segment:
// stably with values; keys alone, where equal keys cannot be told apart, in
// any order inside a bucket, so that an LDS add ranks an item (3 vector
// instructions against about 50 of ballot matching).  SEQ: the values go
// through the keys' stage after them.
template <int BLOCK, int IPT, typename K, typename V, bool VALS, bool SEQ, bool SMALL>
__global__ __launch_bounds__(BLOCK) void k_split_tile_scatter(const SegDesc *__restrict__ tile_desc,
                                                              const SegHeader *__restrict__ h,
                                                              const char *__restrict__ rows,
                                                              const uint32_t *__restrict__ table,
                                                              const uint32_t *__restrict__ chunks) {
    constexpr int WAVES = BLOCK / 64;
    constexpr uint32_t TILE = BLOCK * IPT;
    __shared__ K stage_k[TILE];
    __shared__ V stage_v2[VALS && !SEQ ? TILE : 1];
    __shared__ uint32_t whist[WAVES * kBuckets + WAVES * 64];
    __shared__ uint32_t gbase[kBuckets];
    __shared__ K split[kBuckets];
    __shared__ uint32_t wsum[2][WAVES];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tile = split_tile_of(blockIdx.x, h->total_tiles);
    if (tile >= h->total_tiles) return;
    const SegDesc d = tile_desc[tile];
    const uint32_t item0 = (tile - d.pad) * TILE;
    const uint32_t valid = min(TILE, d.n - item0);
    const bool full = valid == TILE;
    const uint32_t slot0 = wave * 64 * IPT + lane;  // slot j of the lane holds tile item slot0 + 64 j
    const K *src_k = reinterpret_cast<const K *>(d.k) + item0;
    const V *src_v = reinterpret_cast<const V *>(d.v) + (VALS ? item0 : 0u);
    K *dst_k = reinterpret_cast<K *>(d.tk);
    V *dst_v = reinterpret_cast<V *>(d.tv);
    if (reinterpret_cast<const SplitSeg *>(rows + static_cast<size_t>(d.row) * kSplitRowBytes + kSplitSegAt)->buckets == 1u) {
        for (uint32_t i = tid; i < valid; i += BLOCK) {  // one bucket: a copy
            dst_k[item0 + i] = src_k[i];
            if constexpr (VALS) dst_v[item0 + i] = src_v[i];
        }
        return;
    }

    K key[IPT];
    V val[VALS ? IPT : 1];
    if (full) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) key[j] = *gptr<K, true>(src_k, slot0 + j * 64);
    } else {
#pragma unroll
        for (int j = 0; j < IPT; ++j) key[j] = *gptr<K, true>(src_k, min(slot0 + j * 64, valid - 1u));
    }
    const Splitter<K> f = load_splitter<BLOCK, K>(rows, d.row, split);
    uint32_t total = 0, before = 0;
    if (tid < kBuckets) {
        total = reinterpret_cast<const uint32_t *>(rows + static_cast<size_t>(d.row) * kSplitRowBytes)[tid];
        before = table[static_cast<size_t>(tile) * kBuckets + tid] +
                 chunks[static_cast<size_t>(chunk_row(d.pad, d.row, tile)) * kBuckets + tid];
    }
    uint32_t *wh = whist + (VALS ? wave * kBuckets : 0);
    uint32_t *scratch = whist + WAVES * kBuckets + wave * 64 + lane;
    for (uint32_t i = lane; i < static_cast<uint32_t>(kBuckets); i += 64) wh[i] = 0u;
    __syncthreads();

    // ---- stable rank inside the wave, slot by slot; lanes past the end count
    // as the last bucket, behind every item.  rb: rank, and the bucket above it
    uint32_t rb[IPT];
    if (f.linear) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) rb[j] = f.stretch(key[j]);
    } else {
#pragma unroll
        for (int j = 0; j < IPT; ++j) rb[j] = f.search(key[j]);
    }
    if (!full) {
#pragma unroll
        for (int j = 0; j < IPT; ++j)
            if (slot0 + j * 64 >= valid) rb[j] = kBuckets - 1;
    }
    if constexpr (!VALS) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t b = rb[j];
            if (!full && slot0 + j * 64 >= valid) continue;
            // a slot of one bucket (sorted or repeated keys) takes one add
            uint32_t r;
            if (__builtin_amdgcn_ballot_w64(b != __builtin_amdgcn_readfirstlane(b)) == 0) {
                const uint64_t live = __builtin_amdgcn_ballot_w64(true);
                const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                    static_cast<uint32_t>(live >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(live), 0u));
                uint32_t first = 0;
                if (below == 0) first = atomicAdd(&whist[b], static_cast<uint32_t>(__popcll(live)));
                r = __builtin_amdgcn_readfirstlane(first) + below;
            } else {
                r = atomicAdd(&whist[b], 1u);
            }
            rb[j] = r | (b << 16);
        }
    }
#pragma unroll
    for (int j = 0; VALS && j < IPT; ++j) {
        const uint32_t b = rb[j];
        uint32_t lo, hi;
        match_digit<8>(b, lo, hi);
        const uint32_t cnt = wh[b];
        const uint32_t r = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, cnt));
        rb[j] = r | (b << 16);
        uint32_t *dst = r == cnt ? wh + b : scratch;
        uint32_t t;
        asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(t) : "v"(lo), "v"(cnt));
        asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(t) : "v"(hi), "v"(t));
        *dst = t;
        compiler_fence();
        if constexpr (VALS) {
            if (j == IPT / 2 - 1) {  // the values: on their way while the rest is ranked
#pragma unroll
                for (int q = 0; q < IPT; ++q)
                    val[q] = *gptr<V, true>(src_v, full ? slot0 + q * 64 : min(slot0 + q * 64, valid - 1u));
            }
        }
    }
    __syncthreads();

    // ---- per bucket: each wave's offset in the tile, and where its run goes
    constexpr int TABLES = VALS ? WAVES : 1;
    uint32_t mine = 0;
    uint32_t wrun[TABLES];
    if (tid < kBuckets) {
#pragma unroll
        for (int w = 0; w < TABLES; ++w) {
            wrun[w] = mine;
            mine += whist[w * kBuckets + tid];
        }
    }
    const uint32_t texcl = block_exclusive_sum<BLOCK>(mine, wsum[0]);
    const uint32_t start = block_exclusive_sum<BLOCK>(total, wsum[1]);
    if (tid < kBuckets) {
#pragma unroll
        for (int w = 0; w < TABLES; ++w) whist[w * kBuckets + tid] = wrun[w] + texcl;
        gbase[tid] = start + before - texcl;
    }
    __syncthreads();

    // ---- gather by bucket in LDS, then write each bucket's run
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        if (!VALS && !full && slot0 + j * 64 >= valid) continue;
        const uint32_t r = wh[rb[j] >> 16] + (rb[j] & 0xFFFFu);
        stage_k[r] = key[j];
        if constexpr (VALS && !SEQ) stage_v2[r] = val[j];
        if constexpr (SEQ) rb[j] = r;
    }
    __syncthreads();
    const uint32_t last = d.n - 1u;
    uint32_t sp[IPT];
    K sk[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) sk[j] = stage_k[j * BLOCK + tid];
    if (f.linear) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) sp[j] = f.stretch(sk[j]);
    } else {
#pragma unroll
        for (int j = 0; j < IPT; ++j) sp[j] = f.search(sk[j]);
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) sp[j] = min(gbase[sp[j]] + j * BLOCK + tid, last);
    if (full) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            *gptr<K, SMALL>(dst_k, sp[j]) = sk[j];
            if constexpr (VALS && !SEQ) *gptr<V, SMALL>(dst_v, sp[j]) = stage_v2[j * BLOCK + tid];
        }
    } else {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            if (j * BLOCK + tid >= valid) continue;
            *gptr<K, SMALL>(dst_k, sp[j]) = sk[j];
            if constexpr (VALS && !SEQ) *gptr<V, SMALL>(dst_v, sp[j]) = stage_v2[j * BLOCK + tid];
        }
    }
    if constexpr (SEQ) {
        __syncthreads();  // every key out of the stage
        V *stage_v = reinterpret_cast<V *>(stage_k);
#pragma unroll
        for (int j = 0; j < IPT; ++j) stage_v[rb[j]] = val[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; ++j)
            if (full || j * BLOCK + tid < valid) *gptr<V, SMALL>(dst_v, sp[j]) = stage_v[j * BLOCK + tid];
    }
}

// A leaf of one key value, from tk/tv to k/v.
template <int BLOCK, typename K, typename V, bool VALS>
__device__ __forceinline__ void copy_leaf(const LeafArrays<K, V> &a, const SplitLeaf &l) {
    constexpr int U = 8;  // loads in flight per lane
    const K *from_k = a.tk + l.at_tk;
    const V *from_v = VALS ? a.tv + l.at_tk : nullptr;
    K *to_k = a.k + l.at_k;
    V *to_v = VALS ? a.v + l.at_k : nullptr;
    for (uint32_t base = threadIdx.x; base < l.n; base += BLOCK * U) {
        K k[U];
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            k[u] = from_k[min(base + u * BLOCK, l.n - 1u)];
            if constexpr (VALS) v[u] = from_v[min(base + u * BLOCK, l.n - 1u)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u * BLOCK >= l.n) break;
            to_k[base + u * BLOCK] = k[u];
            if constexpr (VALS) to_v[base + u * BLOCK] = v[u];
        }
    }
}

// Sorts the leaves of the first list whole in LDS, from the arrays the pass
// wrote into the others, or in place.  The next leaf's bounds are read while
// this one is sorted.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__global__ __launch_bounds__(BLOCK, sizeof(K) == 4 ? 4 : 3) void k_split_leaves(LeafArrays<K, V> a,
                                                                               const LeafLists *__restrict__ lists,
                                                                               const SplitLeaf *__restrict__ leaves,
                                                                               int in_place) {
    __shared__ BlockSortLds<BLOCK, IPT, K, V, VALS> lds;
    const uint32_t count = min(lists->count[0], lists->capacity);
    uint32_t e = blockIdx.x;
    if (e >= count) return;
    SplitLeaf l = leaves[e];
    for (;;) {
        e += gridDim.x;
        const SplitLeaf next = leaves[min(e, count - 1u)];
        if (l.one) {  // (never in place)
            copy_leaf<BLOCK, K, V, VALS>(a, l);
            if (e >= count) return;
            l = next;
            continue;
        }
        const uint32_t to = in_place ? l.at_tk : l.at_k;
        block_sort<BLOCK, IPT, K, V, VALS>(
            ArraySource<K, V>{a.tk + l.at_tk, VALS ? a.tv + l.at_tk : nullptr}, l.n,
            ArraySink<K, V, VALS>{(in_place ? a.tk : a.k) + to, VALS ? (in_place ? a.tv : a.v) + to : nullptr},
            in_place != 0, lds);
        if (e >= count) return;
        l = next;
        __syncthreads();
    }
}

// The other leaves: those the largest blocks hold, as above; longer ones are
// sorted by one block through global memory, and those above kAloneMax by the
// whole grid (2^22 64-bit pairs, nearly all in one leaf: 1.0 ms a sort, 77 by
// one block).
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__global__ __launch_bounds__(BLOCK) void k_split_long_leaves(LeafArrays<K, V> a, const LeafLists *__restrict__ lists,
                                                             const SplitLeaf *__restrict__ leaves, int in_place,
                                                             uint32_t *table, GridWords *words, uint32_t *error) {
    __shared__ BlockSortLds<BLOCK, IPT, K, V, VALS> lds;
    static_assert(BLOCK * IPT == leaf_max<K>(), "the largest leaf");
    for (int which = 1; which < 3; ++which) {
        const uint32_t count = min(lists->count[which], lists->capacity);
        const SplitLeaf *list = leaves + static_cast<size_t>(which) * lists->capacity;
        for (uint32_t e = blockIdx.x; e < count; e += gridDim.x) {
            const SplitLeaf l = list[e];
            K *from_k = a.tk + l.at_tk, *to_k = a.k + l.at_k;
            V *from_v = VALS ? a.tv + l.at_tk : nullptr;
            V *to_v = VALS ? a.v + l.at_k : nullptr;
            if (which == 1) {
                block_sort<BLOCK, IPT, K, V, VALS>(
                    ArraySource<K, V>{from_k, from_v}, l.n,
                    ArraySink<K, V, VALS>{in_place ? from_k : to_k, in_place ? from_v : to_v}, in_place != 0, lds);
                __syncthreads();
            } else {
                if (!in_place)
                    for (uint32_t i = threadIdx.x; i < l.n; i += BLOCK) {
                        to_k[i] = from_k[i];
                        if constexpr (VALS) to_v[i] = from_v[i];
                    }
                if (in_place) block_sort_global<BLOCK, K, V, VALS>(from_k, from_v, to_k, to_v, l.n, lds.whist, lds.wsum);
                else block_sort_global<BLOCK, K, V, VALS>(to_k, to_v, from_k, from_v, l.n, lds.whist, lds.wsum);
            }
        }
    }
    // (fewer than 2^30 items, so fewer than that; their first tiles take the place of the block sort's words)
    constexpr uint32_t MAX = (1u << 30) / kAloneMax;
    static_assert(sizeof(lds.b.word) >= (MAX + 1) * sizeof(uint32_t), "room for the first tiles");
    const uint32_t longs = min(min(lists->count[3], lists->capacity), MAX);
    if (longs == 0) return;
    const SplitLeaf *list = leaves + 3 * static_cast<size_t>(lists->capacity);
    const auto leaf = [&](uint32_t i) {
        const SplitLeaf l = list[i];
        LongLeaf<K, V> x{a.k + l.at_k, VALS ? a.v + l.at_k : nullptr, a.tk + l.at_tk, VALS ? a.tv + l.at_tk : nullptr, l.n, 1u};
        if (in_place) x = LongLeaf<K, V>{x.tk, x.tv, x.k, x.v, l.n, 0u};
        return x;
    };
    __syncthreads();
    grid_sort_long<BLOCK, K, V, VALS>(leaf, longs, reinterpret_cast<uint32_t *>(lds.b.word), table, words, error,
                                      lds.whist, lds.wsum);
}

// The segments of a pass of the two-pass sort, in one block: offsets off[0..
// count] (as k_split_starts leaves them; one segment of n items if NULL) become
// descriptors, the tiled list, first tiles and the header, as k_seg_classify
// and k_seg_tiles make them.  A one-item segment is copied to tk/tv here.
// gate (if set): a gate that is open leaves this pass and the next, whose
// segments are in `sub`, nothing to do (see k_narrow_probe).
template <typename K, typename V, bool VALS>
__global__ __launch_bounds__(256) void k_split_segments(const uint32_t *__restrict__ off, uint32_t count, uint32_t n,
                                                        K *k, V *v, K *tk, V *tv, uint32_t tile,
                                                        SegDesc *__restrict__ descs, uint32_t *__restrict__ list,
                                                        uint32_t *__restrict__ first_tile, SegHeader *__restrict__ h,
                                                        LeafLists *__restrict__ leaf_lists, uint32_t leaf_capacity,
                                                        const uint32_t *__restrict__ gate, uint32_t *__restrict__ sub) {
    __shared__ uint32_t wsum[2][4];
    const uint32_t s = threadIdx.x;
    if (gate != nullptr && *gate != 0u) {
        count = 0u;
        for (uint32_t i = s; i < kSubOnes + kBuckets / 32; i += 256) sub[i] = 0u;
    }
    const uint32_t a = off == nullptr || s >= count ? 0u : off[s];
    const uint32_t e = s >= count ? 0u : off == nullptr ? n : off[s + 1];
    const uint32_t len = e - a;
    const uint32_t listed = len >= 2u ? 1u : 0u, tiles = listed ? (len - 1u) / tile + 1u : 0u;
    const uint32_t at = block_exclusive_sum<256>(listed, wsum[0]);
    const uint32_t t0 = block_exclusive_sum<256>(tiles, wsum[1]);
    if (len == 1u) {
        tk[a] = k[a];
        if constexpr (VALS) tv[a] = v[a];
    }
    if (listed) {
        SegDesc d;
        d.k = reinterpret_cast<uint32_t *>(k + a);
        d.v = VALS ? reinterpret_cast<uint32_t *>(v + a) : nullptr;
        d.tk = reinterpret_cast<uint32_t *>(tk + a);
        d.tv = VALS ? reinterpret_cast<uint32_t *>(tv + a) : nullptr;
        d.n = len;
        d.pass = off == nullptr ? 0u : (off[kSubOnes + s / 32] >> (s % 32)) & 1u;
        d.row = at;
        d.pad = t0;
        descs[at] = d;
        list[at] = at;
        first_tile[at] = t0;
    }
    if (s == 255u) {
        first_tile[at + listed] = t0 + tiles;
        h->count[kSegLarge] = at + listed;
        h->total_tiles = t0 + tiles;
    }
    if (s < kLeafListsZero) reinterpret_cast<uint32_t *>(leaf_lists)[s] = 0u;
    if (s == kLeafListsZero) leaf_lists->capacity = leaf_capacity;
}

}  // namespace rt
