// rt_block_sort.hip -- arrays that one block sorts whole in LDS: the shapes
// and their launch.
#include "rt_block_sort.h"
#include "rt_common.h"

namespace rt {

// The smallest shape that holds n, of the most threads: with one block per
// launch only its waves hide the latency of its phases.
template <typename K, typename V, bool VALS>
static void launch_shape(K *keys, V *vals, uint32_t n, hipStream_t stream) {
#define RT_BLOCK_SORT(BLK, I)                                                                              \
    hipLaunchKernelGGL((k_block_sort<BLK, I, K, V, VALS>), dim3(1), dim3(BLK), 0, stream, keys, vals, n)
    if (n <= 1024) RT_BLOCK_SORT(256, 4);
    else if (n <= 4096) RT_BLOCK_SORT(1024, 4);
    else if (n <= 8192) RT_BLOCK_SORT(1024, 8);
    else if constexpr (sizeof(K) == 4) RT_BLOCK_SORT(1024, 16);
#undef RT_BLOCK_SORT
}

void launch_block_sort(uint32_t *keys, uint32_t *vals, uint32_t n, hipStream_t stream) {
    prof_begin(stream);
    if (vals) launch_shape<uint32_t, uint32_t, true>(keys, vals, n, stream);
    else launch_shape<uint32_t, uint32_t, false>(keys, vals, n, stream);
    prof_mark(stream, RT_KIND_SEG_SMALL);
}

void launch_block_sort64(uint64_t *keys, uint32_t *vals, uint32_t value_words, uint32_t n, hipStream_t stream) {
    prof_begin(stream);
    if (value_words == 2)
        launch_shape<uint64_t, uint64_t, true>(keys, reinterpret_cast<uint64_t *>(vals), n, stream);
    else if (value_words == 1)
        launch_shape<uint64_t, uint32_t, true>(keys, vals, n, stream);
    else
        launch_shape<uint64_t, uint32_t, false>(keys, nullptr, n, stream);
    prof_mark(stream, RT_KIND_SEG_SMALL);
}

bool default_method(const rt_config *cfg) {
    return cfg == nullptr || (cfg->num_passes == 0 && cfg->block_threads == 0 && cfg->items_per_thread == 0 &&
                              (cfg->flags & ~static_cast<uint32_t>(RT_FLAG_VALIDATE)) == 0);
}

rt_status finish_waited(const rt_config *cfg, hipStream_t stream, const char *what, const void *error) {
    const rt_status s = finish_call(stream, what);
    const bool wait = (cfg != nullptr && (cfg->flags & RT_FLAG_VALIDATE)) || (error != nullptr && debug_sync_enabled());
    if (s != RT_OK || !wait) return s;
    if (error != nullptr) {
        uint32_t err = 0;
        const rt_status r = read_device_word(error, stream, &err, what);
        return r == RT_OK && err ? set_error(RT_ERR_HIP, "%s: device error word 0x%x", what, err) : r;
    }
    const hipError_t e = hipStreamSynchronize(stream);
    return e == hipSuccess ? RT_OK : set_error(RT_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace rt
