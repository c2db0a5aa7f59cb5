// rt_common.h -- host-side declarations shared by the library's sources.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "rt_internal.h"

// Tile shapes (digit bits class, threads per block, items per thread) for
// which onesweep kernels are compiled.  512 x 32 (16K items, two blocks per
// CU) is built for the staged pass with plain stores only.
#define RT_FOR_EACH_SHAPE(X) \
    X(8, 256, 16)            \
    X(8, 512, 16)            \
    X(8, 1024, 8)            \
    X(8, 1024, 12)           \
    X(8, 1024, 16)           \
    X(8, 512, 32)            \
    X(11, 256, 16)           \
    X(11, 512, 8)            \
    X(11, 512, 16)

namespace rt {

// A validated sort configuration.
struct Resolved {
    uint32_t num_passes;
    uint32_t shift[kMaxPasses];
    uint32_t width[kMaxPasses];
    int block;
    int ipt;
    uint32_t flags;
    bool with_values;
    bool chunked;  // passes may run in XCD chunks (every digit of at most 8 bits)
    bool probe;    // chunked: the probe kernel decides per sort (else chunks always)
    bool fused;    // RT_FLAG_FUSED_HISTOGRAM: passes count the next pass's digit
};

// Byte offsets of the workspace regions.
struct Layout {
    size_t hist, base, cbase, plan, ctr, status, status_bytes;
    size_t status_pass[kMaxPasses];
    size_t t1k, t1v, t2k, t2v;
    size_t total;
    uint32_t tiles;       // tiles of the global grid per pass
    uint32_t grid_tiles;  // blocks per pass: the grid cut at up to kChunks - 1 chunk ends
    bool wide_status;     // n >= 2^30: 64-bit lookback words and byte offsets
};

rt_status set_error(rt_status s, const char *fmt, ...);
const char *last_error();
bool debug_sync_enabled();
rt_status finish_call(hipStream_t stream, const char *what);
int device_cu_count();

bool shape_supported(int bits_class, int block, int ipt);

// Histogram arguments of a sort (32- or 64-bit keys) and the first pass's
// positional XCD chunks: chunk x reads input items [bound[x], bound[x + 1]),
// whole tiles, kChunks nearly equal shares of the tile grid.  chunked:
// per-chunk counts (see k_histogram).
struct HistArgs;
void pos_bounds(size_t n, const Resolved &r, uint32_t bound[kChunks + 1]);
HistArgs hist_args(const Resolved &r, size_t n, bool chunked);
rt_status resolve_config(const rt_config *cfg, size_t n, int with_values, Resolved *out);
Layout make_layout(size_t n, const Resolved &r, bool direct);
rt_status cached_workspace(size_t bytes, hipStream_t stream, void **out);
// Waits for the stream, then copies one u32 of device memory to *out.
rt_status read_device_word(const void *word, hipStream_t stream, uint32_t *out, const char *what);
// The whole sort (direct == false) or one explicit pass (direct == true:
// keys/vals read, direct_out_* written).  Pass p's timing mark has kind
// pass_kind + p.  After the plan kernel, the workspace's base table holds
// pass p's exclusive digit offsets at p * kMaxRadix, with every bin past the
// digit's range equal to n.
void launch_sort(uint32_t *keys, uint32_t *vals, uint32_t n, const Resolved &r, const Layout &L, char *ws,
                 bool direct, uint32_t *direct_out_k, uint32_t *direct_out_v, hipStream_t stream,
                 uint32_t pass_kind = RT_KIND_PASS);

// Whole-in-LDS kernel shapes (threads, items per thread, digit bits)
// compiled for the segmented sort; a shape holds segments of up to threads
// x items.  8-bit digits sort a 32-bit key in four passes, 11-bit digits in
// three (11, 11, 10); the 11-bit per-wave counters (8 KiB a wave) limit
// those to 512 threads.
#define RT_FOR_EACH_SEG_SMALL_SHAPE(X) \
    X(64, 4, 8)                        \
    X(64, 8, 8)                        \
    X(128, 4, 8)                       \
    X(128, 8, 8)                       \
    X(256, 4, 8)                       \
    X(256, 8, 8)                       \
    X(512, 4, 8)                       \
    X(512, 8, 8)                       \
    X(256, 16, 8)                      \
    X(128, 9, 8)                       \
    X(256, 9, 8)                       \
    X(256, 17, 8)                      \
    X(512, 16, 8)                      \
    X(1024, 8, 8)                      \
    X(1024, 16, 8)                     \
    X(64, 4, 11)                       \
    X(64, 8, 11)                       \
    X(128, 4, 11)                      \
    X(128, 8, 11)                      \
    X(256, 4, 11)                      \
    X(256, 8, 11)                      \
    X(256, 16, 11)                     \
    X(512, 4, 11)                      \
    X(512, 8, 11)                      \
    X(512, 16, 11)

// Tile shapes (threads, items per thread) of the tiled segments' passes.
#define RT_FOR_EACH_SEG_TILE_SHAPE(X) \
    X(1024, 16)                       \
    X(512, 16)

// The whole-in-LDS size classes of the segmented sort: class c holds the
// segments of more than cls[c - 1].max_n and at most cls[c].max_n items and
// sorts each with one block of the given shape.  Built in: up to 2048 items
// with 256x8, up to 8192 with 512x16, up to 16384 with 1024x16; a tuning
// table's "segments" entries replace it.
struct SegClass {
    uint32_t max_n;
    int block, ipt;
    int bits;  // digit width of the class's passes: 8 or 11
};
// The classes, and the tile shape (tile_block x tile_ipt items) of the
// tiled segments' passes (the server keeps 1024 x 16).
struct SegClassTable {
    uint32_t count;
    SegClass cls[kSegMaxClasses];
    int tile_block, tile_ipt;
    SegClassLimits limits() const;
    uint32_t lds_max() const { return count ? cls[count - 1].max_n : 0u; }
    uint32_t tile() const { return static_cast<uint32_t>(tile_block * tile_ipt); }
};
SegClassTable seg_class_table();
bool seg_small_shape_supported(int block, int ipt, int bits);
bool seg_tile_shape_supported(int block, int ipt);
// Launches the whole-in-LDS kernel of class `which` over its list; the
// segments are sorted on their low `key_bits` bits.
void launch_seg_small(const SegClass &c, bool vals, uint32_t max_listed, hipStream_t stream,
                      const SegDesc *descs, const uint32_t *list, const SegHeader *h, int which, int key_bits,
                      int to_temp);

// Workspace of a segmented sort (byte offsets) and its device pointers.
struct SegLayout {
    uint32_t num_segments;
    size_t capacity;          // temporaries hold this many items
    uint32_t large_capacity;  // most segments the tiled path can hold
    uint32_t max_tiles;
    uint32_t tile;            // items per tile of the tiled segments' passes
    bool wide_status;
    SegClassTable classes;    // size classes the layout was made for
    size_t header, descs, lists, first_tile, tile_seg, hist, base, status, status_pass, tk, tv;
    size_t total;
};

// Chunks of a segmented pass's tile list: kChunks when the segments hold
// kSegChunkMinTiles tiles or more on average (items / segments) and there
// are at least kSegChunkMinSegments of them, else 1.  Chunks end at segment
// ends, so they balance only with many segments per chunk; short segments
// (many partial tiles, short lookback chains) measured faster on one chain.
constexpr uint32_t kSegChunkMinTiles = 16;
constexpr uint32_t kSegChunkMinSegments = 16 * kChunks;
inline uint32_t seg_chunk_count(size_t items, size_t segments, uint32_t tile) {
    return segments >= kSegChunkMinSegments && items / segments >= static_cast<size_t>(kSegChunkMinTiles) * tile
               ? kChunks
               : 1u;
}

struct SegPointers {
    SegHeader *header;
    uint32_t *header_words;
    SegDesc *descs;
    uint32_t *lists;
    uint32_t *first_tile;
    SegDesc *tile_seg;  // per tile: its segment's descriptor, pad = the segment's first tile
    uint32_t *hist;
    uint32_t *base;
    char *status;
    uint32_t *tk;
    uint32_t *tv;
};

// own_temps: the workspace holds the temporaries (capacity items each);
// otherwise the caller supplies them.  The layout takes the current size
// classes (or `classes` when given), and a call uses those of its layout;
// tiled_only: none, every segment of two or more items goes through the
// tiled passes.
SegLayout make_seg_layout(uint32_t num_segments, size_t capacity, bool with_values, bool own_temps,
                          bool tiled_only = false, const SegClassTable *classes = nullptr);
SegPointers seg_pointers(char *ws, const SegLayout &L);
// Sorts segment s = [offsets[s], offsets[s+1]) of keys/vals on digits
// digit0..digit0 + passes - 1 with temporaries tk/tv at the same distance
// from offsets[0]; an even pass count leaves the result in keys/vals, an odd
// one (to_temp set) in tk/tv.  digit0 > 0 needs a tiled_only layout (the
// whole-in-LDS classes sort from digit 0).  persistent: the tiled passes run
// one block per CU that claims tiles until none is left, for calls whose
// tiled segments are usually few.
void launch_segments(uint32_t *keys, uint32_t *vals, uint32_t *tk, uint32_t *tv, const uint32_t *offsets,
                     uint32_t num_segments, const SegLayout &L, char *ws, int passes, int to_temp,
                     hipStream_t stream, uint32_t digit0 = 0, bool persistent = false);
void launch_batched(uint32_t *keys, uint32_t *vals, const uint32_t *offsets, uint32_t num_segments,
                    const SegLayout &L, char *ws, hipStream_t stream);

// Most items one block sorts whole in LDS (rt_block_sort.h): 32-bit keys, and
// 64-bit keys with values of up to 8 bytes.
constexpr size_t kBlockSortMax32 = 16384;
constexpr size_t kBlockSortMax64 = 8192;
// A whole array of 2 to that many items in one launch; vals NULL: keys only
// (value_words 0, 1 or 2 with 64-bit keys).
void launch_block_sort(uint32_t *keys, uint32_t *vals, uint32_t n, hipStream_t stream);
void launch_block_sort64(uint64_t *keys, uint32_t *vals, uint32_t value_words, uint32_t n, hipStream_t stream);
// The splitter sort (rt_split_kernels.h) takes the sizes above those, up to
// these.  tk/tv: temporaries of n items; scratch: split_scratch_bytes() bytes,
// 256-byte aligned.
constexpr size_t kSplitMax32 = static_cast<size_t>(1) << 20;
constexpr size_t kSplitMax64 = static_cast<size_t>(1) << 19;
size_t split_scratch_bytes(size_t n, size_t key_bytes);
size_t split_error_at(size_t n);  // of its device error word, in the scratch
void launch_split(uint32_t *keys, uint32_t *vals, uint32_t n, uint32_t *tk, uint32_t *tv, char *scratch,
                  hipStream_t stream);
void launch_split64(uint64_t *keys, uint32_t *vals, uint32_t value_words, uint32_t n, uint64_t *tk, uint32_t *tv,
                    char *scratch, hipStream_t stream);
// The splitter passes over a large array of 64-bit keys
// (rt_split_seg_kernels.h): one pass and leaves up to kSplitOneMax64, two and
// leaves from kSplitTwoMin64 to kSplitTwoMax64.  scratch as above,
// split_large_scratch_bytes64() long.  us, the digit passes against these,
// pairs with 4-byte values:
//
//             spread keys  ANDs of two   below 2^32   below 2^20
//   600000     156    83    154   145    101    82    86    81
//   2^20       183   100    182   194    115    99    95    99
//   2^21       227   154    223   292                117   142   (two)
//   2^22       367   189    365   308    221   209   179   193
//   2^24       998   508    981   878                461   510
//   2^26      3311  1814   3414  3096   2338  1830  1577  1814
//
// and without the input's copy:
//
//   2^27      5759  2847  5923  5302  3831  2854  2357  2806
//   2^28     11311  6143 11825 11407  7568  6077  4659  6486
//   1.25 2^28 13600 7954 13921 16340  9317  8007  5943  9609
//   1.8 2^28 20242 10541 21551 33033 13178 10333  8445 19248
//
// The lines are where keys of all eight digits gain whatever their
// distribution.  Two passes do not gain where the digit passes skip five of
// eight (the table is without the choice below).  They end where the mean
// of their at most 65536 leaves (2^28: 4096 items) still leaves uneven cuts
// room in the largest leaf (8192): above, leaves that no LDS holds are sorted
// through global memory.
constexpr size_t kSplitOneMax64 = 256 * 2344;  // uneven leaves (18 percent) then fit: at 700000 ANDs of two took 186, not 165
constexpr size_t kSplitTwoMin64 = static_cast<size_t>(1) << 22;
constexpr size_t kSplitTwoMax64 = static_cast<size_t>(1) << 28;
// From here a sample of the keys chooses: keys that differ in at most
// kNarrowBytes of their bytes take the digit passes.  The launches of both
// methods are made, and those not chosen find nothing to do: 55 us of 2870 for
// spread keys at 2^27, 90 of 2440 for keys below 2^20 (2820 by splitter passes;
// 2^28: 4820 and 6490).  Below, spread keys would lose more by it than such keys gain.
constexpr size_t kSplitGateMin64 = static_cast<size_t>(1) << 27;
constexpr uint32_t kNarrowBytes = 3;
size_t split_large_scratch_bytes64(size_t n, uint32_t value_words);
size_t split_large_error_at64(size_t n, uint32_t value_words);
// gate: they run if it is zero (see k_narrow_probe), or NULL; error: their
// error word, or NULL (it is in the scratch then).
void launch_split_large64(uint64_t *keys, uint32_t *vals, uint32_t value_words, uint32_t n, uint64_t *tk, uint32_t *tv,
                          char *scratch, hipStream_t stream, const uint32_t *gate, uint32_t *error);
// Whether cfg leaves the method to the library: no digits, shape or flags
// but RT_FLAG_VALIDATE.
bool default_method(const rt_config *cfg);
// Whether the tuning table sets the digit passes of a default call of n items.
bool tuned_digits(size_t n, int with_values);
// The end of a call that ran one of the methods above: finish_call, and with
// RT_FLAG_VALIDATE the wait it asks for and what *error (device; NULL: the
// call's kernels raise none) says.
rt_status finish_waited(const rt_config *cfg, hipStream_t stream, const char *what, const void *error = nullptr);

// Kernel timing marks (see rt_profile_start); cheap no-ops when disabled.
void prof_begin(hipStream_t stream);
void prof_mark(hipStream_t stream, uint32_t kind);

// Tuned configuration for n items (from the loaded table, else built in).
void tuned_config(size_t n, int with_values, rt_config *out);

}  // namespace rt
