// rt_split_large.hip -- the two-pass splitter sort of large arrays of 32-bit
// keys.
#include <algorithm>

#include "rt_split_seg.h"

namespace rt {

static SplitSortLayout layout32(size_t n, bool vals) {
    return vals ? make_split_sort_layout(n, SplitTile<uint32_t, uint32_t, true>::BLOCK,
                                         SplitTile<uint32_t, uint32_t, true>::IPT)
                : make_split_sort_layout(n, SplitTile<uint32_t, uint32_t, false>::BLOCK,
                                         SplitTile<uint32_t, uint32_t, false>::IPT);
}

size_t split_large_scratch_bytes(size_t n, bool vals) { return layout32(n, vals).total; }

void launch_split_large(uint32_t *keys, uint32_t *vals, uint32_t n, uint32_t *tk, uint32_t *tv, char *scratch,
                        hipStream_t stream) {
    const SplitSortLayout S = layout32(n, vals != nullptr);
    if (vals) launch_split_sort<uint32_t, uint32_t, true>(keys, vals, n, tk, tv, S, scratch, stream);
    else launch_split_sort<uint32_t, uint32_t, false>(keys, vals, n, tk, tv, S, scratch, stream);
}

}  // namespace rt
