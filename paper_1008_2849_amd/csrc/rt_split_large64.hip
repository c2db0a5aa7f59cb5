// rt_split_large64.hip -- the two-pass splitter sort of large arrays of 64-bit
// keys.
#include <algorithm>

#include "rt_split_seg.h"

namespace rt {

static SplitSortLayout layout64(size_t n, uint32_t value_words) {
    return make_split_sort_layout(n, 1024,
                                  value_words == 2 ? SplitTile<uint64_t, uint64_t, true>::IPT
                                                   : SplitTile<uint64_t, uint32_t, true>::IPT);
}

size_t split_large_scratch_bytes64(size_t n, uint32_t value_words) { return layout64(n, value_words).total; }

size_t split_large_error_at64(size_t n, uint32_t value_words) {
    return split_sort_error_at(layout64(n, value_words), split_sort_passes<uint64_t>(n) == 2);
}

void launch_split_large64(uint64_t *keys, uint32_t *vals, uint32_t value_words, uint32_t n, uint64_t *tk, uint32_t *tv,
                          char *scratch, hipStream_t stream, const uint32_t *gate, uint32_t *error) {
    const SplitSortLayout S = layout64(n, value_words);
    if (value_words == 2)
        launch_split_sort<uint64_t, uint64_t, true>(keys, reinterpret_cast<uint64_t *>(vals), n, tk,
                                                    reinterpret_cast<uint64_t *>(tv), S, scratch, stream, gate, error);
    else if (value_words == 1)
        launch_split_sort<uint64_t, uint32_t, true>(keys, vals, n, tk, tv, S, scratch, stream, gate, error);
    else
        launch_split_sort<uint64_t, uint32_t, false>(keys, nullptr, n, tk, nullptr, S, scratch, stream, gate, error);
}

}  // namespace rt
