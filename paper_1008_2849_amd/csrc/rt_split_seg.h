// rt_split_seg.h -- host side of the splitter passes over segments: launch
// sequence, shapes by type, and the two-pass sort of a large array.
#pragma once

#include <cstddef>

#include "rt_common.h"
#include "rt_split_seg_kernels.h"

namespace rt {

inline uint32_t split_grid(size_t want, uint32_t cap) {
    if (want < 1) want = 1;
    return static_cast<uint32_t>(want < cap ? want : cap);
}

// Threads and items per thread of a scatter tile: 16K items, staged keys then
// values through one stage where they do not fit the LDS together (12K with
// 8-byte keys and values); 32-bit keys alone in 512 x 32 blocks, two to a CU.
template <typename K, typename V, bool VALS>
struct SplitTile {
    static constexpr int BLOCK = sizeof(K) == 4 && !VALS ? 512 : 1024;
    static constexpr int IPT = BLOCK == 512 ? 32 : (sizeof(K) == 8 && VALS && sizeof(V) == 8) ? 12 : 16;
    static constexpr bool SEQ = sizeof(K) == 8 && VALS;
    static constexpr int ITEMS = BLOCK * IPT;
};

// A pass's tables inside a SegLayout workspace: rows in the histogram rows,
// the table, chunk rows and leaf lists in the lookback words.
struct SplitTables {
    char *rows;
    uint32_t *table, *chunks;
    LeafLists *lists;
    SplitLeaf *leaves;
    uint32_t leaf_capacity;
};
inline uint32_t quantile_aim(const SegLayout &L, size_t key_bytes) {
    return key_bytes == 4 && L.capacity <= kFewLeafItems ? kQuantileAimFew : kQuantileAim;
}
inline SplitTables split_tables(char *ws, const SegLayout &L) {
    SplitTables t;
    t.rows = ws + L.hist;
    t.table = reinterpret_cast<uint32_t *>(ws + L.status);
    t.chunks = reinterpret_cast<uint32_t *>(ws + L.status + L.status_pass);
    t.lists = reinterpret_cast<LeafLists *>(ws + L.status + 2 * L.status_pass);
    t.leaves = reinterpret_cast<SplitLeaf *>(ws + L.status + 2 * L.status_pass + 256);
    // a segment of n items has at most n / kQuantileAimFew + 1 buckets, one that is
    // the whole array (32 tiles or more, so there is room) up to kBuckets, and
    // buckets of one value make a leaf for every 4096 of their items besides
    t.leaf_capacity = static_cast<uint32_t>(L.capacity / kQuantileAimFew + L.large_capacity);
    if (L.max_tiles >= 32) t.leaf_capacity = std::max<uint32_t>(t.leaf_capacity, kBuckets);
    t.leaf_capacity += static_cast<uint32_t>(L.capacity / 4096);
    return t;
}
static_assert(sizeof(LeafLists) <= 256, "the lists' header");

// What becomes of the buckets: the segments of a next pass (sub[0..kBuckets],
// one listed segment), or leaves, sorted from tk/tv into k/v or in place in
// tk/tv.
enum class SplitEnd { kNextPass, kLeavesBack, kLeavesInPlace };

// Up to here the first of two passes samples 2048 keys of the array, not 8192
// (12 us against 28): its buckets may differ by half, as the second pass cuts
// them by their own sizes and they stay far below the 2^20 items it makes full
// leaves of.  Above, 16 us are less than 0.6 percent of the sort, and the
// longest of the buckets comes near those.
constexpr size_t kSampleFew = static_cast<size_t>(1) << 26;

// arrays: those the segments lie in.  error: the word that the leaves raise, or
// NULL (their own, in the leaf lists' header).
// One splitter pass over the tiled list of a SegLayout whose descriptors,
// list, first tiles and leaf lists' header are on the device.
template <typename T, typename K, typename V, bool VALS>
void launch_split_pass(const SegPointers &P, const SegLayout &L, uint32_t list_stride, SplitEnd end, uint32_t *sub,
                       const LeafArrays<K, V> &arrays, char *ws, hipStream_t stream, uint32_t *error) {
    const uint32_t cus = static_cast<uint32_t>(device_cu_count());
    const SplitTables t = split_tables(ws, L);
    const uint32_t *list = P.lists + static_cast<size_t>(kSegLarge) * list_stride;
    const uint32_t segs = std::max<uint32_t>(1u, L.large_capacity);
    const bool leaves = end != SplitEnd::kNextPass;
    // (a whole array's buckets may all be used, whatever its size)
    const uint32_t fixed = sub != nullptr && segs == 1 ? static_cast<uint32_t>(kBuckets) : 0u;
    const uint32_t aim = quantile_aim(L, sizeof(K));
    if (fixed == 0u)
        hipLaunchKernelGGL((k_split_sample<256, 8, K>), dim3(split_grid(segs, cus * 6)), dim3(256), 0, stream, P.descs,
                           list, P.header, P.first_tile, P.tile_seg, t.rows, fixed, aim);
    else if (!leaves && L.capacity <= kSampleFew)
        hipLaunchKernelGGL((k_split_sample<512, 4, K>), dim3(segs), dim3(512), 0, stream, P.descs, list, P.header,
                           P.first_tile, P.tile_seg, t.rows, fixed, aim);
    else
        hipLaunchKernelGGL((k_split_sample<1024, 8, K>), dim3(segs), dim3(1024), 0, stream, P.descs, list, P.header,
                           P.first_tile, P.tile_seg, t.rows, fixed, aim);
    prof_mark(stream, RT_KIND_PROBE);
    const uint32_t tiles = (L.max_tiles + kChunks - 1) / kChunks * kChunks;
    hipLaunchKernelGGL((k_split_tile_count<512, K>), dim3(tiles), dim3(512), 0, stream, P.tile_seg, P.header, t.rows,
                       t.table, static_cast<uint32_t>(T::ITEMS));
    prof_mark(stream, RT_KIND_HISTOGRAM);
    hipLaunchKernelGGL(k_split_scan,
                       dim3(split_grid(static_cast<size_t>(segs) * (kBuckets / 32), cus * 8),
                            (L.max_tiles + kScanChunk - 1) / kScanChunk),
                       dim3(1024), 0, stream, P.first_tile, P.header, t.table, t.chunks);
    hipLaunchKernelGGL((k_split_starts<K>), dim3(split_grid(segs, cus * 4)), dim3(256), 0, stream, P.descs, list,
                       P.header, P.first_tile, t.rows, t.chunks, leaves ? nullptr : sub, arrays.k, arrays.tk, leaves ? t.lists : nullptr,
                       t.leaves, end == SplitEnd::kLeavesBack ? 1u : 0u);
    prof_mark(stream, RT_KIND_PLAN);
    hipLaunchKernelGGL((k_split_tile_scatter<T::BLOCK, T::IPT, K, V, VALS, T::SEQ, sizeof(K) == 4>), dim3(tiles),
                       dim3(T::BLOCK), 0, stream, P.tile_seg, P.header, t.rows, t.table, t.chunks);
    prof_mark(stream, RT_KIND_PASS);
    if (!leaves) return;
    const int in_place = end == SplitEnd::kLeavesInPlace ? 1 : 0;
    // (the table's rows and the chunk rows behind them: leaves of more than
    // kAloneMax items have at most 5 / 4 of a row for kGridTile items)
    GridWords *words = reinterpret_cast<GridWords *>(t.lists->words);
    hipLaunchKernelGGL((k_split_leaves<256, leaf_ipt<K>(), K, V, VALS>), dim3(split_grid(t.leaf_capacity, cus * 4)), dim3(256), 0,
                       stream, arrays, t.lists, t.leaves, in_place);
    hipLaunchKernelGGL((k_split_long_leaves<1024, sizeof(K) == 4 ? 16 : 8, K, V, VALS>), dim3(cus), dim3(1024), 0,
                       stream, arrays, t.lists, t.leaves, in_place, t.table, words, error ? error : &words->error);
    prof_mark(stream, RT_KIND_SEG_SMALL);
}

// Workspace of the two-pass sort of one array: the first pass's buckets as
// segment offsets, then the passes' tables (one pass at a time), beside the
// temporaries.
struct SplitSortLayout {
    size_t offsets, seg, total;
    SegLayout first, second;
};
// Where the error word of a sort of n items lies.
inline size_t split_sort_error_at(const SplitSortLayout &S, bool two_passes) {
    const SegLayout &L = two_passes ? S.second : S.first;
    return S.seg + L.status + 2 * L.status_pass + offsetof(LeafLists, words) + offsetof(GridWords, error);
}
inline SplitSortLayout make_split_sort_layout(size_t n, int block, int ipt) {
    SplitSortLayout S{};
    SegClassTable t = seg_class_table();
    t.tile_block = block;
    t.tile_ipt = ipt;
    S.offsets = 0;
    S.seg = 2048;
    S.first = make_seg_layout(1, n, false, false, true, &t);
    S.second = make_seg_layout(kBuckets, n, false, false, true, &t);
    S.total = S.seg + std::max(S.first.total, S.second.total);
    return S;
}

template <typename K>
inline int split_sort_passes(size_t n) {
    return n <= kBuckets * leaf_aim<K>() ? 1 : 2;
}

// Sorts n items of keys/vals in place (2 <= n <= kSplitTwoMax64): one pass
// where its buckets are leaves as they come.
template <typename K, typename V, bool VALS>
void launch_split_sort(K *keys, V *vals, uint32_t n, K *tk, V *tv, const SplitSortLayout &S, char *ws,
                       hipStream_t stream, const uint32_t *gate, uint32_t *error) {
    uint32_t *off = reinterpret_cast<uint32_t *>(ws + S.offsets);
    char *seg = ws + S.seg;
    const int passes = split_sort_passes<K>(n);
    if (gate == nullptr) prof_begin(stream);
    for (int pass = 0; pass < passes; ++pass) {
        const SegLayout &L = pass == 0 ? S.first : S.second;
        const SegPointers P = seg_pointers(seg, L);
        const uint32_t num = pass == 0 ? 1u : static_cast<uint32_t>(kBuckets);
        const SplitEnd end = pass == 1 ? SplitEnd::kLeavesInPlace
                             : passes == 1 ? SplitEnd::kLeavesBack : SplitEnd::kNextPass;
        K *a_k = pass == 0 ? keys : tk, *b_k = pass == 0 ? tk : keys;
        V *a_v = pass == 0 ? vals : tv, *b_v = pass == 0 ? tv : vals;
        const SplitTables t = split_tables(seg, L);
        hipLaunchKernelGGL((k_split_segments<K, V, VALS>), dim3(1), dim3(256), 0, stream, pass == 0 ? nullptr : off,
                           num, n, a_k, a_v, b_k, b_v, L.tile, P.descs,
                           P.lists + static_cast<size_t>(kSegLarge) * num, P.first_tile, P.header, t.lists,
                           t.leaf_capacity, pass == 0 ? gate : nullptr, pass == 0 ? off : nullptr);
        prof_mark(stream, RT_KIND_SEGMENTED);
        launch_split_pass<SplitTile<K, V, VALS>, K, V, VALS>(P, L, num, end, off, LeafArrays<K, V>{a_k, a_v, b_k, b_v},
                                                             seg, stream, error);
    }
}

}  // namespace rt
