// rt_split_kernels.h -- the splitter sort of arrays too long for one block
// and too short for passes over the whole chip.
//
// At these sizes a sort is a chain of dependent launches, each of which costs
// about 5 us however little it does; eight-bit passes need one per digit and
// three before them.  Here three launches sort keys of any width:
//
// 1. k_split_count: every block sorts the same sample of the keys in its LDS
//    and takes kBuckets - 1 splitters from it, then counts its own tile's
//    keys per bucket into one row of a table (no table needs clearing).
// 2. k_split_scatter: every block adds up the table's columns for its
//    buckets' starts and its own offsets in them, ranks its tile stably by
//    bucket and writes it, bucket by bucket, to the temporary arrays.
// 3. k_split_leaf: one block sorts each bucket whole in LDS into the caller's
//    arrays.
//
// A value that fills two or more places of the splitter list gets a bucket of
// its own (splitters v and v + 1), which is in order as it stands, so
// repeated keys cost nothing extra.  The buckets of other values have about
// n / kBuckets items, at most four times that but for a chance of about 1e-5
// (a bucket of spread keys holds eight or more sample keys); one that does
// not fit the leaf's LDS is sorted through global memory, slowly but with the
// same result: by its block, and by all of them together if it is long.
//
// Measured (a pass, the input copy included; before: the four- or eight-pass
// sort): 60001 pairs 62.9 -> 25.0 us, 2^20 keys 79.8 -> 43.2 us, 300007 64-bit
// keys with values 133.9 -> 44.7 us.  Bound by latency: count 9 to 15 us (the
// sample's sort is most of it), scatter 7 to 12, leaves 5 to 16.
//
// The count and the stable scatter are Section 3's counting sort with the
// bucket number in the digit's place.
#pragma once

#include "rt_block_sort.h"

namespace rt {

constexpr int kBuckets = 256;

// Counters of grid_sort_long, zero before the launch, and its error word.
struct GridWords {
    uint32_t claim, done, error;
};

// Splitters are searched in the order of a binary tree (node i's children
// are 2i and 2i + 1, the root is 1): a level is a run of consecutive LDS
// words, which lanes read without bank conflicts.  Node i holds the splitter
// of this index.
__device__ __forceinline__ uint32_t tree_index(uint32_t i) {
    const uint32_t level = 31u - __builtin_clz(i);
    return ((2u * (i - (1u << level)) + 1u) << (7u - level)) - 1u;
}
static_assert(kBuckets == 256, "eight levels");

// Bucket of a key: the number of splitters at or below it (kBuckets - 1 of
// them), from their tree.
template <typename K>
__device__ __forceinline__ uint32_t bucket_of(K key, const K *tree) {
    uint32_t i = 1;
#pragma unroll
    for (int level = 0; level < 8; ++level) i = 2u * i + (key >= tree[i] ? 1u : 0u);
    return i - kBuckets;
}

// Sample key i of M: a pseudo-random item of the i-th of M equal stretches.
template <typename K, int M>
struct SampleSource {
    const K *k;
    uint32_t n;
    __device__ __forceinline__ K key(uint32_t i, uint32_t c = 0) const {
        i += c;
        const uint32_t a = static_cast<uint32_t>(static_cast<uint64_t>(i) * n / M);
        const uint32_t b = static_cast<uint32_t>(static_cast<uint64_t>(i + 1) * n / M);
        return *gptr<K, sizeof(K) == 4>(k, a + __umulhi((i + 1u) * 0x9E3779B9u, b - a));
    }
    __device__ __forceinline__ uint32_t val(uint32_t, uint32_t = 0) const { return 0u; }
};
// Every (M / kBuckets)-th sorted sample key.
template <typename K, int M>
struct SplitterSink {
    K *split;
    __device__ __forceinline__ void put(uint32_t base, uint32_t i, K key, uint32_t) const {
        i += base;
        constexpr uint32_t EVERY = M / kBuckets;
        if (i % EVERY == EVERY - 1u && i / EVERY < kBuckets - 1u) split[i / EVERY] = key;
    }
};

// Tile t: items [t * BLOCK * IPT, ...).  Row t of `table`: the tile's count
// per bucket.  Block 0 writes the splitters.
template <int BLOCK, int IPT, typename K>
__global__ __launch_bounds__(BLOCK) void k_split_count(const K *__restrict__ keys, uint32_t n, K *__restrict__ splitters,
                                                       uint32_t *__restrict__ table) {
    constexpr int SIPT = BLOCK >= 512 ? 4 : 8;
    constexpr int M = BLOCK * SIPT;  // 2048 or 4096 sample keys
    __shared__ BlockSortLds<BLOCK, SIPT, K, uint32_t, false> sort;
    __shared__ K picked[kBuckets];
    __shared__ K sorted[kBuckets];
    __shared__ K split[kBuckets];
    __shared__ uint32_t count[kBuckets];
    const uint32_t tid = threadIdx.x;
    K key[IPT];
    const uint32_t tile0 = blockIdx.x * (BLOCK * IPT);
#pragma unroll
    for (int j = 0; j < IPT; ++j) key[j] = *gptr<K, sizeof(K) == 4>(keys, min(tile0 + j * BLOCK + tid, n - 1u));
    block_sort<BLOCK, SIPT, K, uint32_t, false>(SampleSource<K, M>{keys, n}, M, SplitterSink<K, M>{picked}, false, sort);
    if (tid < kBuckets) count[tid] = 0u;
    __syncthreads();
    if (tid < kBuckets - 1) {
        // v the first time, v + 1 from then on (at the largest key: v)
        const K v = picked[tid];
        const K s = tid > 0 && picked[tid - 1] == v && v != ~K(0) ? v + 1u : v;
        sorted[tid] = s;
        if (blockIdx.x == 0) splitters[tid] = s;
    }
    __syncthreads();
    if (tid > 0 && tid < kBuckets) split[tid] = sorted[tree_index(tid)];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j)
        if (tile0 + j * BLOCK + tid < n) atomicAdd(&count[bucket_of(key[j], split)], 1u);
    __syncthreads();
    if (tid < kBuckets) table[blockIdx.x * kBuckets + tid] = count[tid];
}

// Scatters tile blockIdx.x of the k_split_count with the same tiles by bucket
// into out_k/out_v, stably.  Block 0 writes the buckets' starts
// (kBuckets + 1 words), and the leaves' counters after them start at zero.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__global__ __launch_bounds__(BLOCK) void k_split_scatter(const K *__restrict__ keys, const V *__restrict__ vals,
                                                         uint32_t n, const K *__restrict__ splitters,
                                                         const uint32_t *__restrict__ table, K *__restrict__ out_k,
                                                         V *__restrict__ out_v, uint32_t *__restrict__ starts) {
    constexpr int WAVES = BLOCK / 64;
    constexpr uint32_t TILE = BLOCK * IPT;
    constexpr int GROUPS = BLOCK / kBuckets;
    constexpr bool SMALL = sizeof(K) == 4;
    __shared__ K split[kBuckets];
    __shared__ K stage_k[TILE];
    __shared__ V stage_v[VALS ? TILE : 1];
    __shared__ uint8_t stage_b[TILE];
    __shared__ uint32_t whist[WAVES * kBuckets + WAVES * 64];
    __shared__ uint32_t part[2][GROUPS][kBuckets];
    __shared__ uint32_t gbase[kBuckets];
    __shared__ uint32_t wsum[2][WAVES];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tile = blockIdx.x, tiles = gridDim.x;
    const uint32_t tile0 = tile * TILE;
    const uint32_t valid = min(TILE, n - tile0);
    const uint32_t slot0 = wave * 64 * IPT + lane;  // slot j of the lane holds tile item slot0 + 64 j

    K key[IPT];
    V val[VALS ? IPT : 1];
#pragma unroll
    for (int j = 0; j < IPT; ++j) key[j] = *gptr<K, SMALL>(keys, tile0 + min(slot0 + j * 64, valid - 1u));
    if constexpr (VALS) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) val[j] = *gptr<V, sizeof(V) == 4>(vals, tile0 + min(slot0 + j * 64, valid - 1u));
    }
    if (tid > 0 && tid < kBuckets) split[tid] = splitters[tree_index(tid)];
    for (uint32_t i = tid; i < WAVES * kBuckets; i += BLOCK) whist[i] = 0u;
    // the table's column sums: all tiles, and the tiles before this one
    {
        const uint32_t d = tid % kBuckets, g = tid / kBuckets;
        uint32_t all = 0, before = 0;
#pragma unroll 8
        for (uint32_t t = g; t < tiles; t += GROUPS) {
            const uint32_t c = table[t * kBuckets + d];
            all += c;
            before += t < tile ? c : 0u;
        }
        part[0][g][d] = all;
        part[1][g][d] = before;
    }
    __syncthreads();

    // stable rank inside the wave; lanes past the end count as the last bucket
    uint32_t rnk[IPT], bkt[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        bkt[j] = bucket_of(key[j], split);
        if (slot0 + j * 64 >= valid) bkt[j] = kBuckets - 1;
    }
    uint32_t *wh = whist + wave * kBuckets;
    uint32_t *scratch = whist + WAVES * kBuckets + wave * 64 + lane;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        uint32_t lo, hi;
        match_digit<8>(bkt[j], lo, hi);
        const uint32_t cnt = wh[bkt[j]];
        const uint32_t r = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, cnt));
        rnk[j] = r;
        uint32_t *dst = r == cnt ? wh + bkt[j] : scratch;
        uint32_t t;
        asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(t) : "v"(lo), "v"(cnt));
        asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(t) : "v"(hi), "v"(t));
        *dst = t;
        compiler_fence();
    }
    __syncthreads();

    // per bucket: the waves' offsets in the tile, and where its run goes
    uint32_t mine = 0, total = 0, before = 0;
    uint32_t wrun[WAVES];
    if (tid < kBuckets) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            wrun[w] = mine;
            mine += whist[w * kBuckets + tid];
        }
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            total += part[0][g][tid];
            before += part[1][g][tid];
        }
    }
    const uint32_t texcl = block_exclusive_sum<BLOCK>(mine, wsum[0]);
    const uint32_t start = block_exclusive_sum<BLOCK>(total, wsum[1]);
    if (tid < kBuckets) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) whist[w * kBuckets + tid] = wrun[w] + texcl;
        gbase[tid] = start + before - texcl;
        if (tile == 0) {
            starts[tid] = start;
            if (tid == kBuckets - 1) starts[kBuckets] = n;
            if (tid < sizeof(GridWords) / 4) starts[kBuckets + 1 + tid] = 0u;
        }
    }
    __syncthreads();

    // gather by bucket in LDS, then write each bucket's run
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t r = wh[bkt[j]] + rnk[j];
        stage_k[r] = key[j];
        stage_b[r] = static_cast<uint8_t>(bkt[j]);
        if constexpr (VALS) stage_v[r] = val[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = j * BLOCK + tid;
        if (i >= valid) continue;
        const uint32_t p = min(gbase[stage_b[i]] + i, n - 1u);
        *gptr<K, SMALL>(out_k, p) = stage_k[i];
        if constexpr (VALS) *gptr<V, sizeof(V) == 4>(out_v, p) = stage_v[i];
    }
}

// Moves items [base, min(base + BLOCK, end)) of a to b, stably, by the digit at
// bit sh: next[d] (LDS) is where digit d's next item goes, and moves on.
// Positions are clamped to [0, m): a batched call's malformed offsets can give
// two blocks overlapping items, which change between the count and this read.
template <int BLOCK, typename K, typename V, bool VALS>
__device__ __forceinline__ void block_scatter_step(const K *a_k, const V *a_v, K *b_k, V *b_v, uint32_t base, uint32_t end,
                                                   uint32_t m, uint32_t sh, uint32_t *next, uint32_t *whist) {
    constexpr int WAVES = BLOCK / 64;
    const uint32_t tid = threadIdx.x, wave = tid >> 6;
    for (uint32_t i = tid; i < WAVES * 256; i += BLOCK) whist[i] = 0u;
    __syncthreads();
    const uint32_t i = base + tid;
    const K k = i < end ? a_k[i] : K(0);
    const uint32_t d = static_cast<uint32_t>(k >> sh) & 255u;
    uint32_t lo, hi;
    match_digit<8>(d, lo, hi);
    const uint64_t live = __builtin_amdgcn_ballot_w64(i < end);
    lo &= static_cast<uint32_t>(live);
    hi &= static_cast<uint32_t>(live >> 32);
    const uint32_t r = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    if (i < end && r == 0) whist[wave * 256 + d] = __popc(lo) + __popc(hi);
    __syncthreads();
    if (tid < 256) {
        uint32_t run = next[tid];
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t x = whist[w * 256 + tid];
            whist[w * 256 + tid] = run;
            run += x;
        }
        next[tid] = run;
    }
    __syncthreads();
    if (i < end) {
        const uint32_t p = min(whist[wave * 256 + d] + r, m - 1u);
        b_k[p] = k;
        if constexpr (VALS) b_v[p] = a_v[i];
    }
    __syncthreads();
}

// Longest bucket that one block sorts through global memory (64-bit keys: 64
// steps a digit, about 3 ms); longer ones take the whole grid.
constexpr uint32_t kAloneMax = 1u << 16;
constexpr uint32_t kGridTile = 1u << 14;  // items a block takes at a time then

// A bucket of n items of k/v (`copied`: first copied there from tk/tv) to be
// sorted in k/v, with tk/tv to work in.
template <typename K, typename V>
struct LongLeaf {
    K *k;
    V *v;
    K *tk;
    V *tv;
    uint32_t n, copied;
};

// LSD passes (8-bit digits) of the whole grid over `count` buckets, leaf(i)
// the i-th, for keys that the sample missed: whatever the keys, the time is
// that of about two passes over the buckets a digit.  Per digit: counts of
// each tile to its row of `table`, each bucket's rows to output positions, a
// stable scatter of each tile.  One counter numbers the units of all phases
// in order; a block that has claimed one waits until the units of the phases
// before are done, which blocks that run have claimed, so it does not matter
// which blocks of the grid are on the chip.  The wait is bounded as the
// lookback's is (*error is raised then).  All threads call it; first: LDS, count + 1
// words.
template <int BLOCK, typename K, typename V, bool VALS, typename Leaves>
__device__ __forceinline__ void grid_sort_long(const Leaves &leaf, uint32_t count, uint32_t *first, uint32_t *table,
                                               GridWords *words, uint32_t *error, uint32_t *whist, uint32_t *wsum) {
    __shared__ uint32_t next[256];  // counts, or where the digit's next item goes
    __shared__ uint32_t shared;     // thread 0's word for the block
    const uint32_t tid = threadIdx.x;
    uint32_t tiles = 0;
    for (uint32_t base = 0; base < count; base += BLOCK) {
        const uint32_t c = base + tid < count ? (leaf(base + tid).n - 1u) / kGridTile + 1u : 0u;
        const uint32_t at = block_exclusive_sum<BLOCK>(c, wsum);
        if (base + tid < count) first[base + tid] = tiles + at;
        if (tid == BLOCK - 1) shared = at + c;
        __syncthreads();
        tiles += shared;
        __syncthreads();
    }
    if (tid == 0) first[count] = tiles;
    constexpr uint32_t PHASES = 1 + 3 * sizeof(K);  // copies; per digit: counts, positions, scatter
    uint32_t phase = 0, begin = 0, size = tiles, ready = 0;
    for (;;) {
        __syncthreads();
        if (tid == 0) shared = atomicAdd(&words->claim, 1u);
        __syncthreads();
        const uint32_t unit = shared;
        while (unit - begin >= size) {
            begin += size;
            if (++phase == PHASES) return;
            size = phase % 3u == 2u ? count : tiles;
        }
        if (phase != ready) {
            __syncthreads();
            if (tid == 0) {
                uint32_t polls = 0;
                while (status_load(&words->done) < begin && ++polls <= kLookbackSpinLimit) backoff(16);
                shared = polls <= kLookbackSpinLimit ? 1u : 0u;
                if (!shared) atomicOr(error, kErrLookbackTimeout);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            __syncthreads();
            if (!shared) return;
            ready = phase;
        }
        uint32_t e = unit - begin;
        if (phase % 3u == 2u) {  // one bucket's rows
            uint32_t *row = table + static_cast<size_t>(first[e]) * 256u + (tid & 255u);
            const uint32_t rows = first[e + 1] - first[e];
            constexpr uint32_t U = 8;  // loads in flight
            const auto load = [&](uint32_t t, uint32_t (&x)[U]) {
#pragma unroll
                for (uint32_t i = 0; i < U; ++i) x[i] = t + i < rows ? row[static_cast<size_t>(t + i) * 256u] : 0u;
            };
            uint32_t c = 0, x[U];
            for (uint32_t t = 0; t < rows && tid < 256; t += U) {
                load(t, x);
#pragma unroll
                for (uint32_t i = 0; i < U; ++i) c += x[i];
            }
            uint32_t run = block_exclusive_sum<BLOCK>(c, wsum);
            for (uint32_t t = 0; t < rows && tid < 256; t += U) {
                load(t, x);
#pragma unroll
                for (uint32_t i = 0; i < U; ++i) {
                    if (t + i < rows) row[static_cast<size_t>(t + i) * 256u] = run;
                    run += x[i];
                }
            }
        } else {
            const uint32_t tile = e;
            uint32_t hi = count - 1u;  // the bucket: the last with first <= tile
            for (e = 0; e < hi;) {
                const uint32_t mid = (e + hi + 1u) / 2u;
                if (first[mid] <= tile) e = mid;
                else hi = mid - 1u;
            }
            const LongLeaf<K, V> l = leaf(e);
            const uint32_t m = l.n, i0 = (tile - first[e]) * kGridTile, i1 = min(m, i0 + kGridTile);
            const uint32_t digit = phase == 0u ? 0u : (phase - 1u) / 3u, sh = 8u * digit;
            K *a_k = digit & 1u ? l.tk : l.k, *b_k = digit & 1u ? l.k : l.tk;
            V *a_v = digit & 1u ? l.tv : l.v, *b_v = digit & 1u ? l.v : l.tv;
            uint32_t *row = table + static_cast<size_t>(tile) * 256u;
            if (phase == 0u) {
                for (uint32_t i = i0 + tid; i < i1 && l.copied; i += BLOCK) {
                    a_k[i] = b_k[i];
                    if constexpr (VALS) a_v[i] = b_v[i];
                }
            } else if (phase % 3u == 1u) {
                if (tid < 256) next[tid] = 0u;
                __syncthreads();
                for (uint32_t i = i0 + tid; i < i1; i += BLOCK) atomicAdd(&next[static_cast<uint32_t>(a_k[i] >> sh) & 255u], 1u);
                __syncthreads();
                if (tid < 256) row[tid] = next[tid];
            } else {
                if (tid < 256) next[tid] = row[tid];
                for (uint32_t base = i0; base < i1; base += BLOCK) block_scatter_step<BLOCK, K, V, VALS>(a_k, a_v, b_k, b_v, base, i1, m, sh, next, whist);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            atomicAdd(&words->done, 1u);
        }
    }
}

// LSD passes of one block over items [0, m) of a/b in global memory (8-bit
// digits; an even number of passes, so the result ends in a): for a bucket
// that no leaf holds.
template <int BLOCK, typename K, typename V, bool VALS>
__device__ __forceinline__ void block_sort_global(K *a_k, V *a_v, K *b_k, V *b_v, uint32_t m, uint32_t *whist, uint32_t *wsum) {
    __shared__ uint32_t next[256];  // where the digit's next item goes
    const uint32_t tid = threadIdx.x;
    for (uint32_t sh = 0; sh < 8 * sizeof(K); sh += 8) {
        __syncthreads();
        if (tid < 256) next[tid] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < m; i += BLOCK) atomicAdd(&next[static_cast<uint32_t>(a_k[i] >> sh) & 255u], 1u);
        __syncthreads();
        const uint32_t c = tid < 256 ? next[tid] : 0u;
        const uint32_t first = block_exclusive_sum<BLOCK>(c, wsum);
        if (tid < 256) next[tid] = first;
        for (uint32_t base = 0; base < m; base += BLOCK)
            block_scatter_step<BLOCK, K, V, VALS>(a_k, a_v, b_k, b_v, base, m, m, sh, next, whist);
        K *sk = a_k; a_k = b_k; b_k = sk;
        V *sv = a_v; a_v = b_v; b_v = sv;
    }
    __syncthreads();
}

// The arguments of k_split_leaf, as they lie in memory (pointers, one after the
// other).
template <typename K, typename V>
struct SplitLeafArgs {
    K *tk;
    V *tv;
    K *keys;
    V *vals;
    const K *splitters;
    const uint32_t *starts;
    uint32_t *table;
    GridWords *words;
};

// The kernel's arguments, from its first on, read again: what follows a long
// phase then keeps no registers through it (with them, the leaves' sort spilled
// twice as many and took 1 to 4 us longer).
template <typename T>
__device__ __forceinline__ T reread_args() {
    static_assert(sizeof(T) % 8 == 0, "read in 8-byte words");
    typedef const __attribute__((address_space(4))) uint64_t ct;
    ct *p = (ct *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    uint64_t w[sizeof(T) / 8];
#pragma unroll
    for (uint32_t i = 0; i < sizeof(T) / 8; ++i) w[i] = p[i];
    T x;
    __builtin_memcpy(&x, w, sizeof x);
    return x;
}

// Sorts bucket blockIdx.x of the temporary arrays into the caller's.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__global__ __launch_bounds__(BLOCK) void k_split_leaf(K *__restrict__ tk, V *__restrict__ tv, K *__restrict__ keys,
                                                      V *__restrict__ vals, const K *__restrict__ splitters,
                                                      const uint32_t *__restrict__ starts, uint32_t *, GridWords *) {
    constexpr uint32_t CAP = BLOCK * IPT;
    __shared__ BlockSortLds<BLOCK, IPT, K, V, VALS> lds;
    // buckets of one value, and buckets for the whole grid
    __shared__ uint64_t big_mask[kBuckets / 64], long_mask[kBuckets / 64];
    const uint32_t tid = threadIdx.x, b = blockIdx.x;
    // one-value buckets too long for a leaf are in order: every block copies
    // its share of them
    if (tid < kBuckets) {
        bool copy = false;
        const uint32_t m = starts[tid + 1] - starts[tid];
        if (m > CAP && tid > 0)
            copy = tid < kBuckets - 1 ? static_cast<K>(splitters[tid] - splitters[tid - 1]) == K(1)
                                      : splitters[tid - 1] == ~K(0);
        const uint64_t mask = __builtin_amdgcn_ballot_w64(copy), grid = __builtin_amdgcn_ballot_w64(!copy && m > kAloneMax);
        if ((tid & 63u) == 0) {
            big_mask[tid >> 6] = mask;
            long_mask[tid >> 6] = grid;
        }
    }
    const uint32_t first = starts[b], m = starts[b + 1] - first;
    __syncthreads();
    for (int q = 0; q < kBuckets / 64; ++q)
        for (uint64_t mask = big_mask[q]; mask != 0; mask &= mask - 1u) {
            const uint32_t x = q * 64 + __builtin_ctzll(mask);
            const uint32_t e = starts[x + 1];
            for (uint32_t i = starts[x] + b * BLOCK + tid; i < e; i += kBuckets * BLOCK) {
                keys[i] = tk[i];
                if constexpr (VALS) vals[i] = tv[i];
            }
        }
    if (m != 0 && m <= CAP) {
        block_sort<BLOCK, IPT, K, V, VALS>(ArraySource<K, V>{tk + first, VALS ? tv + first : nullptr}, m,
                                           ArraySink<K, V, VALS>{keys + first, VALS ? vals + first : nullptr}, false,
                                           lds);
    } else if (m > CAP && m <= kAloneMax && !((big_mask[b / 64] >> (b % 64)) & 1u)) {
        for (uint32_t i = tid; i < m; i += BLOCK) {
            keys[first + i] = tk[first + i];
            if constexpr (VALS) vals[first + i] = tv[first + i];
        }
        block_sort_global<BLOCK, K, V, VALS>(keys + first, VALS ? vals + first : nullptr, tk + first,
                                             VALS ? tv + first : nullptr, m, lds.whist, lds.wsum);
    }
    uint32_t longs = 0;
    for (int q = 0; q < kBuckets / 64; ++q) longs += static_cast<uint32_t>(__popcll(long_mask[q]));
    if (longs == 0) return;
    const SplitLeafArgs<K, V> g = reread_args<SplitLeafArgs<K, V>>();
    const auto leaf = [&](uint32_t i) {
        uint32_t x = 0;  // the i-th long bucket
        for (int q = 0; q < kBuckets / 64; ++q) {
            uint64_t mask = long_mask[q];
            const uint32_t c = static_cast<uint32_t>(__popcll(mask));
            if (i < c) {
                for (; i != 0; --i) mask &= mask - 1u;
                x = q * 64 + __builtin_ctzll(mask);
                break;
            }
            i -= c;
        }
        const uint32_t at = g.starts[x];
        return LongLeaf<K, V>{g.keys + at, VALS ? g.vals + at : nullptr, g.tk + at, VALS ? g.tv + at : nullptr,
                              g.starts[x + 1] - at, 1u};
    };
    __syncthreads();
    grid_sort_long<BLOCK, K, V, VALS>(leaf, longs, lds.b.bin, g.table, g.words, &g.words->error, lds.whist, lds.wsum);
}

}  // namespace rt
