// rt_block_sort.h -- one block sorts up to BLOCK * IPT items whole in LDS.
//
// Two methods share the LDS:
//
// * The bin sort.  The items' key range [lo, hi] is cut into NB equal bins
//   (NB = the power of two at or below the block's capacity, so about one
//   item per bin).  An LDS add counts each bin and hands its items slots in
//   arrival order; a prefix sum over the bins gives each bin's start; each
//   item then writes one word (the key's bits below the bin, then the item's
//   index) to its slot, and counts the smaller words of its own bin: bin
//   start + that count is its final position.  The words are distinct and
//   ordered by (key, index), so the order is stable and does not depend on
//   the arrival order.  Its cost per item is one LDS add, one word in and
//   out of LDS, and as many compares as the fullest bin holds; the key's
//   width does not matter.
// * The digit passes (Section 3's counting sort per 8-bit digit of the key's
//   offset from lo, Section 4's LSD order), ranked with wave64 ballots, for
//   items that crowd a few bins (repeated or clustered keys): about 57 vector
//   instructions per item and digit, whatever the keys.
//
// The bin sort counts first and gives way to the digit passes when some bin
// holds more than kBinLimit items.
#pragma once

#include <cstddef>
#include <type_traits>
#include <utility>

#include "rt_kernels.h"

namespace rt {

// Fullest bin the bin sort ranks: its compares (4 instructions each) then
// cost less than two digit passes.  For n uniform keys in NB >= n / 1.1 bins
// the fullest bin holds 6 to 8 items.
constexpr uint32_t kBinLimit = 24;
constexpr int kSlotGroup = 4;  // slots whose LDS reads go out together
constexpr int kCrowded = 8;    // of 64 sampled keys in one of 256 cells
constexpr uint32_t kDense = 8;  // items per value of a small key range

constexpr int floor_log2(int x) { return x <= 1 ? 0 : 1 + floor_log2(x / 2); }
constexpr int ceil_log2(int x) { return x <= 1 ? 0 : 1 + floor_log2(x - 1); }

// Aligned for its 16-byte accesses (the bins are cleared and scanned four at
// a time), whatever stands beside it in a kernel's LDS.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
struct alignas(16) BlockSortLds {
    static constexpr int WAVES = BLOCK / 64;
    static constexpr int CAP = BLOCK * IPT;
    static constexpr int LOG_NB = floor_log2(CAP);
    static constexpr int NB = 1 << LOG_NB;
    static constexpr int PER = NB >= BLOCK ? NB / BLOCK : 1;  // bins per thread of the scan
    static constexpr int IDX_BITS = ceil_log2(CAP);
    static constexpr uint32_t NONE = CAP + kBinLimit;       // word: larger than any (two of them)
    static constexpr uint32_t SPARE = CAP + kBinLimit + 2;  // word: written by lanes without an item
    static_assert(PER % 4 == 0, "the scan reads four bins at a time");
    union {
        struct {
            uint32_t bin[NB + 4];          // counts, then starts; bin[NB] = n
            K word[CAP + kBinLimit + 4];   // a rank may read past its bin, and past the end
        } b;
        struct {
            K k[CAP];
            V v[VALS ? CAP : 1];
        } s;
    };
    uint32_t whist[WAVES * 256 + WAVES * 64];  // digit passes: per-wave counters, scratch row
    uint32_t wsum[WAVES];
    uint32_t wmax[WAVES];
    K wlo[WAVES], whi[WAVES];
};
typedef BlockSortLds<256, 17, uint32_t, uint32_t, true> BlockSortLds32;
typedef BlockSortLds<256, 16, uint64_t, uint32_t, true> BlockSortLds64;
static_assert(alignof(BlockSortLds32) >= alignof(uint4) && alignof(BlockSortLds64) >= alignof(uint4) &&
                  offsetof(BlockSortLds32, b) == 0 && offsetof(BlockSortLds64, b) == 0,
              "the bins are read as uint4");
// three 256 x 16 blocks with 64-bit keys and 4-byte values share a CU's LDS
static_assert(3 * sizeof(BlockSortLds64) <= kLdsBytesPerCu, "three blocks to a CU");

__device__ __forceinline__ uint32_t key_bits_of(uint32_t span) { return 32u - __builtin_clz(span | 1u) - (span == 0u); }
__device__ __forceinline__ uint32_t key_bits_of(uint64_t span) {
    return span == 0u ? 0u : 64u - static_cast<uint32_t>(__builtin_clzll(span));
}

// x from another lane, as wave_inclusive_sum moves it (DPP control CTRL,
// rows MASK); a lane without a source keeps its own x.
template <int CTRL, int MASK>
__device__ __forceinline__ uint32_t dpp_from(uint32_t x) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(static_cast<int>(x), static_cast<int>(x), CTRL, MASK, 0xf, false));
}
template <int CTRL, int MASK>
__device__ __forceinline__ uint64_t dpp_from(uint64_t x) {
    return (static_cast<uint64_t>(dpp_from<CTRL, MASK>(static_cast<uint32_t>(x >> 32))) << 32) |
           dpp_from<CTRL, MASK>(static_cast<uint32_t>(x));
}
__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return __builtin_amdgcn_readlane(x, 63); }
__device__ __forceinline__ uint64_t last_lane(uint64_t x) {
    return (static_cast<uint64_t>(last_lane(static_cast<uint32_t>(x >> 32))) << 32) | last_lane(static_cast<uint32_t>(x));
}

// op over the wave's lanes (idempotent: a minimum or maximum), uniform.
template <typename T, typename F>
__device__ __forceinline__ T wave_fold(T x, F op) {
    x = op(x, dpp_from<0x111, 0xf>(x));
    x = op(x, dpp_from<0x112, 0xf>(x));
    x = op(x, dpp_from<0x114, 0xf>(x));
    x = op(x, dpp_from<0x118, 0xf>(x));
    x = op(x, dpp_from<0x142, 0xa>(x));
    x = op(x, dpp_from<0x143, 0xc>(x));
    return last_lane(x);
}

// Makes x opaque: what was derived from it is derived again, not kept in
// registers across a phase.
__device__ __forceinline__ void forget(uint32_t &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void forget(uint64_t &x) { asm volatile("" : "+v"(x)); }

// f(0), f(1), ..., f(N - 1) with compile-time arguments.  (Loops nested over
// a register array left it one register tuple, copied whole at each branch.)
template <int... I, typename F>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_each(std::make_integer_sequence<int, N>{}, f);
}
// f of each slot of group g (kSlotGroup of them, fewer in the last group).
template <int IPT, int G, typename F>
__device__ __forceinline__ void group_slots(F &&f) {
    static_for<(IPT - G < kSlotGroup ? IPT - G : kSlotGroup)>(
        [&](auto q) { f(std::integral_constant<int, G + decltype(q)::value>{}); });
}

// Where block_sort reads its items and puts the sorted ones.
template <typename K, typename V>
struct ArraySource {
    const K *k;
    const V *v;
    // item i + c; c a constant that the load's immediate offset takes
    __device__ __forceinline__ K key(uint32_t i, uint32_t c = 0) const {
        return *((const __attribute__((address_space(1))) K *)((const g_char *)k + static_cast<uint32_t>(i * sizeof(K))) + c);
    }
    __device__ __forceinline__ V val(uint32_t i, uint32_t c = 0) const {
        return *((const __attribute__((address_space(1))) V *)((const g_char *)v + static_cast<uint32_t>(i * sizeof(V))) + c);
    }
};
template <typename K, typename V, bool VALS>
struct ArraySink {
    K *k;
    V *v;
    // item base + i, base uniform
    __device__ __forceinline__ void put(uint32_t base, uint32_t i, K key, V val) const {
        *gptr<K, true>(k + base, i) = key;
        if constexpr (VALS) *gptr<V, true>(v + base, i) = val;
    }
};

// The staged items, each key plus lo, to the sink: kSlotGroup slots' LDS reads
// go out together.
template <int BLOCK, int IPT, typename K, typename V, bool VALS, typename Sink>
__device__ __forceinline__ void block_store(const BlockSortLds<BLOCK, IPT, K, V, VALS> &lds, uint32_t tid, uint32_t n,
                                            K lo, const Sink &sink) {
    constexpr int GRP = kSlotGroup;
    static_for<(IPT + GRP - 1) / GRP>([&](auto group) {
        constexpr int g = group * GRP;
        if (static_cast<uint32_t>(g * BLOCK) >= n) return;
        K k[GRP];
        V v[GRP];
        group_slots<IPT, g>([&](auto slot) {
            constexpr int j = slot, q = j - g;
            k[q] = lds.s.k[j * BLOCK + tid] + lo;
            v[q] = 0;
            if constexpr (VALS) v[q] = lds.s.v[j * BLOCK + tid];
        });
        if (static_cast<uint32_t>((g + GRP < IPT ? g + GRP : IPT) * BLOCK) <= n) {
            group_slots<IPT, g>([&](auto slot) { sink.put(slot * BLOCK, tid, k[slot - g], v[slot - g]); });
        } else {
            group_slots<IPT, g>([&](auto slot) {
                if (slot * BLOCK + tid < n) sink.put(slot * BLOCK, tid, k[slot - g], v[slot - g]);
            });
        }
    });
}

// Items that are ranked by comparing all pairs: up to here that takes fewer
// instructions (2 a pair, no bins to clear and scan, one barrier instead of
// seven) whatever the keys.  65536 segments of 16 to 120 pairs: 272 -> 216 us
// uniform, 340 -> 216 repeated keys; up to 256 items it took longer than the
// bins (40000 segments of 128 to 256 pairs: 281 us against 201).
constexpr uint32_t kPairwise = 128;

// block_sort of n <= kPairwise items, one a thread.
template <typename K, typename V, bool VALS, typename Source, typename Sink, typename Lds>
__device__ __forceinline__ void block_sort_pairwise(const Source &src, uint32_t n, const Sink &sink, Lds &lds) {
    constexpr uint32_t STEP = 16 / sizeof(K);  // keys a read
    const uint32_t i = threadIdx.x;
    const uint32_t wave0 = __builtin_amdgcn_readfirstlane(i & ~63u);
    K key = ~K(0);
    V val = 0;
    if (i < n) {
        key = src.key(i);
        if constexpr (VALS) val = src.val(i);
    }
    if (i < kPairwise) lds.s.k[i] = key;  // the places past the end: no smaller than any
    if constexpr (VALS) {
        if (i < kPairwise) lds.s.v[i] = val;  // (every value is read before one is overwritten)
    }
    __syncthreads();
    if (i >= n) return;
    // equal keys: those before this item count, those behind it do not
    uint32_t r = 0;
    const uint32_t mine_end = min(wave0 + 64u, (n + STEP - 1u) / STEP * STEP);
    for (uint32_t j = 0; j < wave0; j += STEP) {
#pragma unroll
        for (uint32_t q = 0; q < STEP; ++q) r += static_cast<uint32_t>(lds.s.k[j + q] <= key);
    }
    for (uint32_t j = wave0; j < mine_end; j += STEP) {
#pragma unroll
        for (uint32_t q = 0; q < STEP; ++q) {
            const K x = lds.s.k[j + q];
            r += static_cast<uint32_t>((x < key) | ((x == key) & (j + q < i)));
        }
    }
    for (uint32_t j = mine_end; j < n; j += STEP) {
#pragma unroll
        for (uint32_t q = 0; q < STEP; ++q) r += static_cast<uint32_t>(lds.s.k[j + q] < key);
    }
    sink.put(0, r, key, val);
}

// Sorts items [0, n) of src (1 <= n <= BLOCK * IPT) into sink, which may be
// the same arrays (in_place).  Every thread of the block must call it; the
// LDS is free again after the next barrier.
//
// Each wave owns `slots` * 64 consecutive items, lane l the items l, l + 64,
// ... of them: the items are spread over all waves whatever n is, and slot by
// slot, lane by lane is input order.  Where an LDS read is followed by its
// use, kSlotGroup slots are taken together and without a test per item, so
// that their reads overlap: past the end, a lane writes to a spare place.
template <int BLOCK, int IPT, typename K, typename V, bool VALS, typename Source, typename Sink>
__device__ __forceinline__ void block_sort(const Source &src, uint32_t n, const Sink &sink, bool in_place,
                                           BlockSortLds<BLOCK, IPT, K, V, VALS> &lds) {
    typedef BlockSortLds<BLOCK, IPT, K, V, VALS> L;
    constexpr int WAVES = L::WAVES;
    constexpr int PER = L::PER;
    constexpr int GRP = kSlotGroup, GROUPS = (IPT + GRP - 1) / GRP;
    constexpr uint32_t NB = L::NB;
    uint32_t tid = threadIdx.x;
    forget(tid);
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    n = __builtin_amdgcn_readfirstlane(n);
    if constexpr (BLOCK >= kPairwise) {
        if (n <= kPairwise) {
            block_sort_pairwise<K, V, VALS>(src, n, sink, lds);
            return;
        }
    }
    const int slots = static_cast<int>((n + BLOCK - 1) / BLOCK);
    const uint32_t slot0 = wave * 64u * slots;
    uint32_t item0 = slot0 + lane;
    // whether slot j holds an item of this lane
#define RT_LIVE(j) (item0 + (j) * 64 < ((j) < slots ? n : 0u))
    // whether the slots of group g all hold an item in every lane of the wave
    const int full_slots = min(slots, static_cast<int>((max(n, slot0) - slot0) / 64u));
#define RT_FULL(g) (((g) + GRP < IPT ? (g) + GRP : IPT) <= full_slots)

    // ---- load, clear the bins, key range
    K key[IPT];
    K lo = ~K(0), hi = 0;
    static_for<GROUPS>([&](auto group) {
        constexpr int g = group * GRP;
        if (RT_FULL(g)) group_slots<IPT, g>([&](auto j) { key[j] = src.key(item0, j * 64); });
        else if (g < slots) group_slots<IPT, g>([&](auto j) { key[j] = src.key(min(item0 + j * 64, n - 1u)); });
    });
    for (uint32_t i = tid; i < NB / 4; i += BLOCK) reinterpret_cast<uint4 *>(lds.b.bin)[i] = make_uint4(0u, 0u, 0u, 0u);
    static_for<GROUPS>([&](auto group) {
        constexpr int g = group * GRP;
        if (g < slots)
            group_slots<IPT, g>([&](auto j) {
                lo = key[j] < lo ? key[j] : lo;
                hi = key[j] > hi ? key[j] : hi;
            });
    });
    lo = wave_fold(lo, [](K x, K y) { return x < y ? x : y; });
    hi = wave_fold(hi, [](K x, K y) { return x < y ? y : x; });
    // Keys that crowd a few bins go straight to the digit passes, which would
    // otherwise start after a bin count in vain: of one key per lane (from two
    // slots, so that a sorted input looks spread), more than kCrowded share
    // one of 128 to 256 cells of the wave's own range with one of six of them
    // (spread keys: hardly ever more than 4).
    bool crowded = false;
    {
        K pick = key[0];
        if (IPT / 2 < slots) {
            K other = key[IPT / 2];
            forget(other);  // (a choice of two elements would put the keys in scratch memory)
            if ((lane & 1u) && item0 + IPT / 2 * 64 < n) pick = other;
        }
        const uint32_t wbits = key_bits_of(static_cast<K>(hi - lo));
        uint32_t cell = static_cast<uint32_t>((pick - lo) >> (wbits > 8 ? wbits - 8 : 0u));
        if (item0 >= n) cell = 256u + lane;
#pragma unroll
        for (int q = 0; q < 6; ++q)
            crowded |= __popcll(__builtin_amdgcn_ballot_w64(cell == __builtin_amdgcn_readlane(cell, 11 * q))) > kCrowded;
    }
    if (lane == 0) {
        lds.wlo[wave] = lo;
        lds.whi[wave] = hi;
        lds.wmax[wave] = crowded ? 1u : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const K a = lds.wlo[w], b = lds.whi[w];
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
        crowded = crowded || lds.wmax[w] != 0u;
    }
    const uint32_t bits = __builtin_amdgcn_readfirstlane(key_bits_of(static_cast<K>(hi - lo)));
    if (bits == 0) {  // one key value: the input order stands
        if (in_place) return;
        for (uint32_t i = tid; i < n; i += BLOCK) {
            V v = 0;
            if constexpr (VALS) v = src.val(i);
            sink.put(0, i, lo, v);
        }
        return;
    }
    const uint32_t shift = bits > static_cast<uint32_t>(L::LOG_NB) ? bits - L::LOG_NB : 0u;
    // few values, each many times: the bins would overflow, and their counts
    // be taken in vain
    if (bits < 16u && (n >> bits) >= kDense) crowded = true;
    V val[VALS ? IPT : 1];

    // ---- bin sort, if an item's word holds its bits below the bin and its index
    if (!crowded && shift + L::IDX_BITS <= 8 * sizeof(K)) {
        uint32_t at[IPT];  // slot in the bin, then the final position
        static_for<GROUPS>([&](auto group) {
            constexpr int g = group * GRP;
            if (RT_FULL(g))
                group_slots<IPT, g>([&](auto j) {
                    at[j] = atomicAdd(&lds.b.bin[static_cast<uint32_t>((key[j] - lo) >> shift)], 1u);
                });
            else if (g < slots)
                group_slots<IPT, g>([&](auto j) {
                    at[j] = 0;
                    if (RT_LIVE(j)) at[j] = atomicAdd(&lds.b.bin[static_cast<uint32_t>((key[j] - lo) >> shift)], 1u);
                });
        });
        __syncthreads();
        // exclusive prefix sum: wave w owns bins [w, w + 1) * 64 * PER, four
        // consecutive bins a lane and step
        uint4 c[PER / 4];
        uint32_t run = 0, most = 0;
        uint4 *row = reinterpret_cast<uint4 *>(lds.b.bin) + wave * (16 * PER);
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) c[q] = row[q * 64 + lane];
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) {
            most = max(max(most, max(c[q].x, c[q].y)), max(c[q].z, c[q].w));
            const uint32_t s1 = c[q].x + c[q].y, s2 = s1 + c[q].z, sum = s2 + c[q].w;
            const uint32_t incl = wave_inclusive_sum(sum);
            const uint32_t excl = run + incl - sum;
            run += last_lane(incl);
            c[q] = make_uint4(excl, excl + c[q].x, excl + s1, excl + s2);
        }
        most = wave_fold(most, [](uint32_t x, uint32_t y) { return max(x, y); });
        if (lane == 0) {
            lds.wsum[wave] = run;
            lds.wmax[wave] = most;
        }
        __syncthreads();
        uint32_t before = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            if (w < static_cast<int>(wave)) before += lds.wsum[w];
            most = max(most, lds.wmax[w]);
        }
        most = __builtin_amdgcn_readfirstlane(most);
        if (most <= kBinLimit) {
#pragma unroll
            for (int q = 0; q < PER / 4; ++q)
                row[q * 64 + lane] = make_uint4(c[q].x + before, c[q].y + before, c[q].z + before, c[q].w + before);
            if (tid == 0) lds.b.bin[NB] = n;
            // words past the end compare as larger than any
            if (tid < kBinLimit) lds.b.word[n + tid] = ~K(0);
            if (tid < 2) lds.b.word[L::NONE + tid] = ~K(0);
            __syncthreads();
            // ---- one word per item, in its bin's slots: the key's bits below
            // the bin (all its bits, if they fit), then the item's index; and
            // the values on their way.  at then holds the bin's start and,
            // above it, its count.
            const bool whole = bits + L::IDX_BITS <= 8 * sizeof(K);
            const K below = whole ? ~K(0) : (K(1) << shift) - 1u;
            forget(item0);
            static_for<GROUPS>([&](auto group) {
                constexpr int g = group * GRP;
                if (g >= slots) return;
                uint32_t first[GRP], next[GRP];
                group_slots<IPT, g>([&](auto j) {
                    forget(key[j]);
                    const uint32_t b = static_cast<uint32_t>((key[j] - lo) >> shift);
                    first[j - g] = lds.b.bin[b];
                    next[j - g] = lds.b.bin[b + 1];
                });
                const auto word = [&](auto j) { return (((key[j] - lo) & below) << L::IDX_BITS) | (item0 + j * 64); };
                if (RT_FULL(g)) {
                    group_slots<IPT, g>([&](auto j) {
                        lds.b.word[first[j - g] + at[j]] = word(j);
                        if constexpr (VALS) val[j] = src.val(item0, j * 64);
                    });
                } else {
                    group_slots<IPT, g>([&](auto j) {
                        lds.b.word[RT_LIVE(j) ? first[j - g] + at[j] : static_cast<uint32_t>(L::SPARE)] = word(j);
                        if constexpr (VALS) val[j] = src.val(min(item0 + j * 64, n - 1u));
                    });
                }
                group_slots<IPT, g>([&](auto j) { at[j] = first[j - g] | ((next[j - g] - first[j - g]) << 16); });
            });
            __syncthreads();
            // ---- rank in the bin: the smaller words among its slots, two a
            // step.  An item alone in its bin, or past its bin's end, reads a
            // word that never counts, with the other such lanes (one LDS
            // access).  Words of whole keys need no test for the bin's end:
            // what follows it is larger.
            static_for<GROUPS>([&](auto group) {
                constexpr int g = group * GRP;
                if (g >= slots) return;
                uint32_t first[GRP], cnt[GRP], r[GRP];
                K mine[GRP];
                forget(item0);
                uint32_t longest = 0;
                group_slots<IPT, g>([&](auto j) {
                    constexpr int q = j - g;
                    forget(key[j]);
                    mine[q] = (((key[j] - lo) & below) << L::IDX_BITS) | (item0 + j * 64);
                    r[q] = first[q] = at[j] & 0xFFFFu;
                    cnt[q] = at[j] >> 16;
                    if (cnt[q] == 1u) cnt[q] = 0u;
                    longest = max(longest, cnt[q]);
                });
                K w0[GRP], w1[GRP];
                const auto read = [&](uint32_t t) {
                    group_slots<IPT, g>([&](auto j) {
                        constexpr int q = j - g;
                        const uint32_t p = t < cnt[q] ? first[q] + t : static_cast<uint32_t>(L::NONE);
                        w0[q] = lds.b.word[p];
                        w1[q] = lds.b.word[p + 1];
                    });
                    __builtin_amdgcn_sched_barrier(0);  // all reads out before the first is waited for
                };
                if (whole) {
                    for (uint32_t t = 0; __builtin_amdgcn_ballot_w64(t < longest) != 0u; t += 2) {
                        read(t);
                        group_slots<IPT, g>([&](auto j) {
                            constexpr int q = j - g;
                            r[q] += static_cast<uint32_t>(w0[q] < mine[q]);
                            r[q] += static_cast<uint32_t>(w1[q] < mine[q]);
                        });
                    }
                } else {
                    for (uint32_t t = 0; __builtin_amdgcn_ballot_w64(t < longest) != 0u; t += 2) {
                        read(t);
                        group_slots<IPT, g>([&](auto j) {
                            constexpr int q = j - g;
                            r[q] += static_cast<uint32_t>(w0[q] < mine[q]);
                            r[q] += static_cast<uint32_t>((t + 1 < cnt[q]) & (w1[q] < mine[q]));
                        });
                    }
                }
                group_slots<IPT, g>([&](auto j) { at[j] = r[j - g]; });
            });
            __syncthreads();
            // ---- gather by position, then write consecutive addresses
            forget(item0);
            static_for<GROUPS>([&](auto group) {
                constexpr int g = group * GRP;
                if (RT_FULL(g))
                    group_slots<IPT, g>([&](auto j) {
                        lds.s.k[at[j]] = key[j];
                        if constexpr (VALS) lds.s.v[at[j]] = val[j];
                    });
                else if (g < slots)
                    group_slots<IPT, g>([&](auto j) {
                        if (!RT_LIVE(j)) return;
                        lds.s.k[at[j]] = key[j];
                        if constexpr (VALS) lds.s.v[at[j]] = val[j];
                    });
            });
            __syncthreads();
            forget(tid);
            block_store<BLOCK, IPT, K, V, VALS>(lds, tid, n, K(0), sink);
            return;
        }
    }
    __syncthreads();  // the digit passes reuse the LDS

    // ---- digit passes, ranked in input order.  Slots wholly past the end are
    // neither ranked nor staged; the empty lanes of the slot that holds the
    // end take the highest digit, behind every item.
    forget(item0);
    uint32_t *wh = lds.whist + wave * 256;
    uint32_t *scratch = lds.whist + WAVES * 256 + wave * 64 + lane;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        key[j] = RT_LIVE(j) ? static_cast<K>(key[j] - lo) : ~K(0);
        if constexpr (VALS) val[j] = RT_LIVE(j) ? src.val(item0 + j * 64) : V(0);
    }
    for (uint32_t sh = 0; sh < bits; sh += 8) {
        for (uint32_t i = lane; i < 256; i += 64) wh[i] = 0u;
        // (the previous pass finished reading wh before its last barrier)
        uint32_t rnk[IPT];
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            if (j >= slots || slot0 + j * 64 >= n) continue;
            const uint32_t dg = static_cast<uint32_t>(key[j] >> sh) & 255u;
            uint32_t mlo, mhi;
            match_digit<8>(dg, mlo, mhi);
            const uint32_t cnt = wh[dg];
            // mbcnt and bcnt add the counter while they count
            const uint32_t r = __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, cnt));
            rnk[j] = r;
            uint32_t *dst = r == cnt ? wh + dg : scratch;
            uint32_t t;
            asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(t) : "v"(mlo), "v"(cnt));
            asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(t) : "v"(mhi), "v"(t));
            *dst = t;
            compiler_fence();
        }
        __syncthreads();
        // counts of earlier waves, then the digit's start, per digit
        constexpr int R = 256 >= BLOCK ? 256 / BLOCK : 1;
        constexpr int DT = 256 / R;
        uint32_t tcount[R];
        uint32_t tsum = 0;
        if (tid < DT) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t dg = tid * R + r;
                uint32_t run = 0;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) {
                    const uint32_t x = lds.whist[w * 256 + dg];
                    lds.whist[w * 256 + dg] = run;
                    run += x;
                }
                tcount[r] = run;
                tsum += run;
            }
        }
        const uint32_t texcl = block_exclusive_sum<BLOCK>(tid < DT ? tsum : 0u, lds.wsum);
        if (tid < DT) {
            uint32_t run = texcl;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t dg = tid * R + r;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) lds.whist[w * 256 + dg] += run;
                run += tcount[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            if (j >= slots || slot0 + j * 64 >= n) continue;
            const uint32_t r = wh[static_cast<uint32_t>(key[j] >> sh) & 255u] + rnk[j];
            lds.s.k[r] = key[j];
            if constexpr (VALS) lds.s.v[r] = val[j];
        }
        __syncthreads();
        if (sh + 8 < bits) {
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const uint32_t i = item0 + j * 64;
                key[j] = RT_LIVE(j) ? lds.s.k[i] : ~K(0);
                if constexpr (VALS) val[j] = RT_LIVE(j) ? lds.s.v[i] : V(0);
            }
            // the stage is rewritten only after the next pass's first barrier
        }
    }
    block_store<BLOCK, IPT, K, V, VALS>(lds, tid, n, lo, sink);
#undef RT_LIVE
#undef RT_FULL
}

// A whole array of at most BLOCK * IPT items, sorted in place by one block:
// one launch, one read and one write.  Bound by the latency of its phases
// (one CU works).  5000 uniform keys: 9.5 us a call, against 53 us for the
// eight launches of the general sort (fill, histogram, plan, four passes,
// copy back), each of which costs about 5 us however little it does.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__global__ __launch_bounds__(BLOCK) void k_block_sort(K *__restrict__ keys, V *__restrict__ vals, uint32_t n) {
    __shared__ BlockSortLds<BLOCK, IPT, K, V, VALS> lds;
    block_sort<BLOCK, IPT, K, V, VALS>(ArraySource<K, V>{keys, vals}, n, ArraySink<K, V, VALS>{keys, vals}, true, lds);
}

}  // namespace rt
