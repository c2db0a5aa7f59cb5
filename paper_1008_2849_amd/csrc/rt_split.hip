// rt_split.hip -- host side of the splitter sort: shapes by size and launches.
#include <cstddef>

#include "rt_common.h"
#include "rt_split_kernels.h"

namespace rt {

static size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// Tiles of 1024, 2048 or 4096 items: at most 256 of them (one row of the
// table each, and every block reads the whole table), enough to give each CU
// one from 2^18 items.
static uint32_t split_tile(size_t n) {
    return n <= (static_cast<size_t>(1) << 17) ? 1024u : n <= (static_cast<size_t>(1) << 18) ? 2048u : 4096u;
}

// The buckets' starts, then the leaves' counters.
static size_t starts_bytes() { return align256((kBuckets + 1) * sizeof(uint32_t) + sizeof(GridWords)); }

size_t split_scratch_bytes(size_t n, size_t key_bytes) {
    const size_t tiles = (n + split_tile(n) - 1) / split_tile(n);
    return align256(tiles * kBuckets * sizeof(uint32_t)) + starts_bytes() +
           align256(kBuckets * key_bytes);
}

size_t split_error_at(size_t n) {
    const size_t tiles = (n + split_tile(n) - 1) / split_tile(n);
    return align256(tiles * kBuckets * sizeof(uint32_t)) + (kBuckets + 1) * sizeof(uint32_t) + offsetof(GridWords, error);
}

template <typename K, typename V, bool VALS>
static void launch(K *keys, V *vals, uint32_t n, K *tk, V *tv, char *scratch, hipStream_t stream) {
    const uint32_t tile = split_tile(n), tiles = (n + tile - 1) / tile;
    uint32_t *table = reinterpret_cast<uint32_t *>(scratch);
    scratch += align256(static_cast<size_t>(tiles) * kBuckets * sizeof(uint32_t));
    uint32_t *starts = reinterpret_cast<uint32_t *>(scratch);
    scratch += starts_bytes();
    K *splitters = reinterpret_cast<K *>(scratch);
    prof_begin(stream);
#define RT_SPLIT_TILES(BLK)                                                                                         \
    do {                                                                                                            \
        hipLaunchKernelGGL((k_split_count<BLK, 4, K>), dim3(tiles), dim3(BLK), 0, stream, keys, n, splitters, table); \
        prof_mark(stream, RT_KIND_HISTOGRAM);                                                                       \
        hipLaunchKernelGGL((k_split_scatter<BLK, 4, K, V, VALS>), dim3(tiles), dim3(BLK), 0, stream, keys, vals, n,  \
                           splitters, table, tk, tv, starts);                                                       \
        prof_mark(stream, RT_KIND_PASS);                                                                            \
    } while (0)
    if (tile == 1024) RT_SPLIT_TILES(256);
    else if (tile == 2048) RT_SPLIT_TILES(512);
    else RT_SPLIT_TILES(1024);
#undef RT_SPLIT_TILES
    // leaves that hold four times the mean bucket
#define RT_SPLIT_LEAF(BLK, I)                                                                                       \
    hipLaunchKernelGGL((k_split_leaf<BLK, I, K, V, VALS>), dim3(kBuckets), dim3(BLK), 0, stream, tk, tv, keys, vals, \
                       splitters, starts, table, reinterpret_cast<GridWords *>(starts + kBuckets + 1))
    if (n <= (1u << 16)) RT_SPLIT_LEAF(256, 4);
    else if (n <= (1u << 18)) RT_SPLIT_LEAF(1024, 4);
    else if (n <= (1u << 19)) RT_SPLIT_LEAF(1024, 8);
    else if constexpr (sizeof(K) == 4) RT_SPLIT_LEAF(1024, 16);
#undef RT_SPLIT_LEAF
    prof_mark(stream, RT_KIND_SEG_SMALL);
}

void launch_split(uint32_t *keys, uint32_t *vals, uint32_t n, uint32_t *tk, uint32_t *tv, char *scratch,
                  hipStream_t stream) {
    if (vals) launch<uint32_t, uint32_t, true>(keys, vals, n, tk, tv, scratch, stream);
    else launch<uint32_t, uint32_t, false>(keys, vals, n, tk, tv, scratch, stream);
}

void launch_split64(uint64_t *keys, uint32_t *vals, uint32_t value_words, uint32_t n, uint64_t *tk, uint32_t *tv,
                    char *scratch, hipStream_t stream) {
    if (value_words == 2)
        launch<uint64_t, uint64_t, true>(keys, reinterpret_cast<uint64_t *>(vals), n, tk,
                                         reinterpret_cast<uint64_t *>(tv), scratch, stream);
    else if (value_words == 1)
        launch<uint64_t, uint32_t, true>(keys, vals, n, tk, tv, scratch, stream);
    else
        launch<uint64_t, uint32_t, false>(keys, vals, n, tk, tv, scratch, stream);
}

}  // namespace rt
