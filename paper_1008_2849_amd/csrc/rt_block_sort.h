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
#include "rt_kernels.h"

namespace rt {

// Fullest bin the bin sort ranks: its compares (4 instructions each) then
// cost less than two digit passes.  For n uniform keys in NB >= n / 1.1 bins
// the fullest bin holds 6 to 8 items.
constexpr uint32_t kBinLimit = 24;

constexpr int floor_log2(int x) { return x <= 1 ? 0 : 1 + floor_log2(x / 2); }
constexpr int ceil_log2(int x) { return x <= 1 ? 0 : 1 + floor_log2(x - 1); }

template <int BLOCK, int IPT, typename K, typename V, bool VALS>
struct BlockSortLds {
    static constexpr int WAVES = BLOCK / 64;
    static constexpr int CAP = BLOCK * IPT;
    static constexpr int LOG_NB = floor_log2(CAP);
    static constexpr int NB = 1 << LOG_NB;
    static constexpr int PER = NB >= BLOCK ? NB / BLOCK : 1;  // bins per thread of the scan
    static constexpr int IDX_BITS = ceil_log2(CAP);
    static_assert(PER % 4 == 0, "the scan reads four bins at a time");
    union {
        struct {
            uint32_t bin[NB + 4];          // counts, then starts; bin[NB] = n
            K word[CAP + kBinLimit];       // a rank may read past its bin, never past this
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

// Sorts items [0, n) of in_k/in_v (n <= BLOCK * IPT) into out_k/out_v, which
// may be the same arrays.  Every thread of the block must call it; the LDS
// is free again after the next barrier.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__device__ __forceinline__ void block_sort(const K *in_k, const V *in_v, uint32_t n, K *out_k, V *out_v,
                                           BlockSortLds<BLOCK, IPT, K, V, VALS> &lds) {
    typedef BlockSortLds<BLOCK, IPT, K, V, VALS> L;
    constexpr int WAVES = L::WAVES;
    constexpr int PER = L::PER;
    constexpr uint32_t NB = L::NB;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = tid >> 6;

    // ---- load (item j * BLOCK + tid in slot j), clear the bins, key range
    K key[IPT];
    V val[VALS ? IPT : 1];
    K lo = ~K(0), hi = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = j * BLOCK + tid;
        if (i < n) key[j] = in_k[i];
    }
    if constexpr (VALS) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t i = j * BLOCK + tid;
            if (i < n) val[j] = in_v[i];
        }
    }
    for (uint32_t i = tid; i < NB / 4; i += BLOCK) reinterpret_cast<uint4 *>(lds.b.bin)[i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        if (j * BLOCK + tid >= n) continue;
        lo = key[j] < lo ? key[j] : lo;
        hi = key[j] > hi ? key[j] : hi;
    }
    lo = wave_fold(lo, [](K x, K y) { return x < y ? x : y; });
    hi = wave_fold(hi, [](K x, K y) { return x < y ? y : x; });
    if (lane == 0) {
        lds.wlo[wave] = lo;
        lds.whi[wave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const K a = lds.wlo[w], b = lds.whi[w];
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    const uint32_t bits = key_bits_of(static_cast<K>(hi - lo));
    if (bits == 0) {  // one key value: the input order stands
        if (out_k != in_k) {
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const uint32_t i = j * BLOCK + tid;
                if (i >= n) continue;
                out_k[i] = key[j];
                if constexpr (VALS) out_v[i] = val[j];
            }
        }
        return;
    }
    const uint32_t shift = bits > static_cast<uint32_t>(L::LOG_NB) ? bits - L::LOG_NB : 0u;

    // ---- bin sort, if an item's word holds its bits below the bin and its index
    if (shift + L::IDX_BITS <= 8 * sizeof(K)) {
        uint32_t at[IPT];  // slot in the bin, then the bin's start
#pragma unroll
        for (int j = 0; j < IPT; ++j)
            if (j * BLOCK + tid < n) at[j] = atomicAdd(&lds.b.bin[static_cast<uint32_t>((key[j] - lo) >> shift)], 1u);
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
        if (most <= kBinLimit) {
#pragma unroll
            for (int q = 0; q < PER / 4; ++q)
                row[q * 64 + lane] = make_uint4(c[q].x + before, c[q].y + before, c[q].z + before, c[q].w + before);
            if (tid == 0) lds.b.bin[NB] = n;
            __syncthreads();
            // ---- one word per item, in its bin's slots
            K mine[IPT];
            uint32_t cnt[IPT], pos[IPT];
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const uint32_t i = j * BLOCK + tid;
                cnt[j] = 0;
                mine[j] = 0;
                if (i >= n) {
                    at[j] = 0;
                    continue;
                }
                const K rel = key[j] - lo;
                const uint32_t b = static_cast<uint32_t>(rel >> shift);
                const uint32_t first = lds.b.bin[b];
                cnt[j] = lds.b.bin[b + 1] - first;
                mine[j] = ((rel & ((K(1) << shift) - 1u)) << L::IDX_BITS) | i;
                lds.b.word[first + at[j]] = mine[j];
                at[j] = first;
                pos[j] = first;
            }
            __syncthreads();
            // ---- rank in the bin: the smaller words among its slots (the
            // reads past a shorter bin hit later words and do not count)
            for (uint32_t t = 0; t < most; ++t) {
#pragma unroll
                for (int j = 0; j < IPT; ++j) {
                    if (j * BLOCK >= n) continue;
                    const K w = lds.b.word[at[j] + t];
                    pos[j] += static_cast<uint32_t>((t < cnt[j]) & (w < mine[j]));
                }
            }
            __syncthreads();
            // ---- gather by position, then write consecutive addresses
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                if (j * BLOCK + tid >= n) continue;
                lds.s.k[pos[j]] = key[j];
                if constexpr (VALS) lds.s.v[pos[j]] = val[j];
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const uint32_t i = j * BLOCK + tid;
                if (i >= n) continue;
                out_k[i] = lds.s.k[i];
                if constexpr (VALS) out_v[i] = lds.s.v[i];
            }
            return;
        }
        __syncthreads();  // the bins are read: the digit passes reuse the LDS
    }

    // ---- digit passes.  Wave w owns items [w, w + 1) * 64 * IPT and lane l
    // holds item s * 64 + l of them in slot s, so that slot-by-slot,
    // lane-by-lane ranking follows input order.  Slots wholly past the end
    // are neither ranked nor staged; the empty lanes of the slot that holds
    // the end take the highest digit, behind every item.
    constexpr int WAVE_ITEMS = 64 * IPT;
    const uint32_t wslot0 = wave * WAVE_ITEMS + lane;
    uint32_t *wh = lds.whist + wave * 256;
    uint32_t *scratch = lds.whist + WAVES * 256 + wave * 64 + lane;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = wslot0 + j * 64;
        key[j] = i < n ? static_cast<K>(in_k[i] - lo) : ~K(0);
        if constexpr (VALS) val[j] = i < n ? in_v[i] : V(0);
    }
    for (uint32_t sh = 0; sh < bits; sh += 8) {
        for (uint32_t i = lane; i < 256; i += 64) wh[i] = 0u;
        // (the previous pass finished reading wh before its last barrier)
        uint32_t rnk[IPT];
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            if (wave * WAVE_ITEMS + j * 64 >= n) continue;
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
            if (wave * WAVE_ITEMS + j * 64 >= n) continue;
            const uint32_t r = wh[static_cast<uint32_t>(key[j] >> sh) & 255u] + rnk[j];
            lds.s.k[r] = key[j];
            if constexpr (VALS) lds.s.v[r] = val[j];
        }
        __syncthreads();
        if (sh + 8 < bits) {
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const uint32_t i = wslot0 + j * 64;
                key[j] = i < n ? lds.s.k[i] : ~K(0);
                if constexpr (VALS) val[j] = i < n ? lds.s.v[i] : V(0);
            }
            // the stage is rewritten only after the next pass's first barrier
        }
    }
    for (uint32_t i = tid; i < n; i += BLOCK) {
        out_k[i] = lds.s.k[i] + lo;
        if constexpr (VALS) out_v[i] = lds.s.v[i];
    }
}

// A whole array of at most BLOCK * IPT items, sorted in place by one block:
// one launch, one read and one write.  Bound by the latency of its phases
// (one CU works).  5000 uniform keys: 9.5 us a call, against 53 us for the
// eight launches of the general sort (fill, histogram, plan, four passes,
// copy back), each of which costs about 5 us however little it does.
template <int BLOCK, int IPT, typename K, typename V, bool VALS>
__global__ __launch_bounds__(BLOCK) void k_block_sort(K *__restrict__ keys, V *__restrict__ vals, uint32_t n) {
    __shared__ BlockSortLds<BLOCK, IPT, K, V, VALS> lds;
    block_sort<BLOCK, IPT, K, V, VALS>(keys, vals, n, keys, vals, lds);
}

}  // namespace rt
