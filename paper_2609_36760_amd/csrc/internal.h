// Internal interface between the host ABI (mla_abi.cpp) and the HIP kernels.
// Not part of the public C ABI.
#pragma once

#include <cmath>
#include <cstdint>

#include <hip/hip_runtime_api.h>

namespace mla {

// Resolved byte geometry of a packed page (layout documented in mla_lowbit.h).
struct PageGeom {
    int32_t page_size;      // tokens per page
    int32_t c_bits;         // 4 or 2
    int32_t cc_bytes;       // content code bytes per token
    int32_t cr_bytes;       // RoPE code bytes per token
    int32_t off_cr;         // region offsets inside a page
    int32_t off_mc;
    int32_t off_mr;         // (fp16 metadata only)
    int64_t page_bytes;
    int32_t paper_meta;     // 1: the paper's metadata record at off_mc
    uint32_t page_magic;    // floor(2^32 / page_size): split_slot in writer_common.h
};

struct AppendArgs {
    const uint16_t* c_kv;
    int64_t c_kv_stride;
    const uint16_t* k_rope;
    int64_t k_rope_stride;
    const int64_t* slot_mapping;
    int32_t n;
    uint8_t* cache;
    int64_t num_slots;      // num_pages * page_size
    PageGeom g;
    // BF16 protection writes (lowbit_append_kernel<CBITS, true> only)
    uint8_t* prot;
    int64_t num_prot;
    const int32_t* token_seq;   // [n] sequence of each token
    const int32_t* positions;   // [n] position of each token in its sequence
    const int32_t* seq_lens;    // [B] lengths after the append
    const int32_t* prot_slot;   // [B] buffer of each sequence
    int32_t B;
    int32_t sink, recent;
};

// Low-bit kinds: content bits and metadata storage (P: the paper's record).
enum CacheKind { KIND_C4R4 = 0, KIND_C2R4 = 1, KIND_BF16 = 2, KIND_C4R4P = 3, KIND_C2R4P = 4 };

// Query rows and waves of a workgroup: 16 or 32 rows (decode_narrow.hip: one,
// two or four waves on one row block, each with its part of the keys), or 64 or
// 128 (decode_attn.hip: four waves on one tile).
struct LaunchShape {
    int32_t rows, waves;
};

struct DecodeArgs {
    LaunchShape shape;      // of the launch (choose_shape)
    const uint16_t* q_lat;
    const uint16_t* q_rope;
    const uint8_t* cache;
    int64_t num_pages;
    const int32_t* block_table;
    int32_t max_pages;
    const int32_t* seq_lens;
    int32_t B, s_q, H;
    float scale_log2;       // softmax_scale * log2(e)
    int32_t split_tokens;   // 0: unsplit
    const int32_t* split_indptr;
    int32_t num_work;       // B (unsplit) or total splits
    uint16_t* out;
    float* lse;
    float* part_m;
    float* part_s;
    uint16_t* part_o;       // fp16, normalized by part_s
    PageGeom g;             // for BF16: page_size and page_bytes only
    // BF16 protection (decode_kernel<KIND, true> only)
    const uint8_t* prot;    // protection buffers, num_prot x (sink + recent) rows of 1152 bytes
    int64_t num_prot;
    const int32_t* prot_slot;   // [B] buffer of each sequence
    int32_t sink, recent;
    // In-launch append (decode_kernel only; new_c == nullptr: none): token (b, i)
    // of [B][s_q], position seq_lens[b] - s_q + i of sequence b, quantized (or
    // copied, BF16) into slot new_slots[b * s_q + i] before it is read; under
    // protection also its bf16 row into the protection buffer.
    const uint16_t* new_c;
    int64_t new_c_stride;
    const uint16_t* new_k;
    int64_t new_k_stride;
    const int64_t* new_slots;
};

struct CombineArgs {
    const float* part_m;
    const float* part_s;
    const uint16_t* part_o;
    const int32_t* split_indptr;
    int32_t B, s_q, H;
    uint16_t* out;
    float* lse;
};

// Events for the next decode-kernel dispatch on this host thread (both null
// when none); take_launch_events() returns them and clears them.
struct LaunchEvents {
    hipEvent_t start, stop;
};
LaunchEvents take_launch_events();

hipError_t launch_lowbit_append(const AppendArgs& a, hipStream_t stream);
hipError_t launch_bf16_append(const AppendArgs& a, hipStream_t stream);
// Decode in a.shape.  launch_decode takes every shape (those of 16 and 32 rows it
// hands on), launch_decode_narrow, for up to kNarrowRows query rows, those of 16
// and 32 rows; a shape that neither kernel has is refused.
constexpr int kNarrowRows = 32;
hipError_t launch_decode(CacheKind kind, const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_protected(CacheKind kind, const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_narrow(CacheKind kind, const DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_narrow_protected(CacheKind kind, const DecodeArgs& a, hipStream_t stream);

// Launch shapes, for the host's size checks (each kernel file asserts its own
// constants against these).  A dispatch packet holds the launch's work-item
// count in 32 bits, so a launch of more than kMaxDispatchItems work items
// cannot be expressed: the host refuses such shapes before any HIP call.
constexpr int64_t kMaxDispatchItems = 0xFFFFFFFFll;
constexpr int kWaveThreads = 64;
constexpr int kDecodeThreads = 256;          // decode_attn.hip: 4 waves per workgroup
constexpr int kDecodeRowsPerBlock = 128;     // query rows of its widest shape
constexpr int kNarrowThreads = 64;           // decode_narrow.hip in its largest launch: one wave per workgroup
constexpr int kNarrowRowsPerBlock = 16;      // of 16 rows
constexpr int kWorkGroupRound = 8;           // work items padded to a multiple of the 8 XCDs
constexpr int kCombineThreads = 256;         // combine.hip: at most one row per workgroup
constexpr int kAppendThreadsPerToken = 72;   // quant_append.hip: 9 groups x 8 lanes
constexpr int64_t kMaxAppendTokens = int64_t(1) << 25;
static_assert(kMaxAppendTokens * kAppendThreadsPerToken + 256 <= kMaxDispatchItems, "append launch size");

// Work items of a launch over the split (or unsplit) work list: padded to the
// XCD round, times the row blocks; the caller multiplies by the threads.
constexpr int64_t decode_workgroups(int64_t num_work, int64_t rows, int64_t rows_per_block) {
    return (num_work + kWorkGroupRound - 1) / kWorkGroupRound * kWorkGroupRound *
           ((rows + rows_per_block - 1) / rows_per_block);
}

// Indexes that come from device-resident values, kept inside their table for any
// values (split_indptr not as planned, a plan for other lengths): the page-table
// column of token t, and the first list tile of a split of a protected sequence.
constexpr int32_t page_column(int32_t t, int32_t page_size, int32_t max_pages) {
    const int32_t c = t / page_size;
    return c < 0 ? 0 : c < max_pages ? c : max_pages - 1;
}
constexpr int32_t split_tile(int32_t split, int32_t split_tokens, int32_t n_list) {
    const int64_t u = static_cast<int64_t>(split) * (split_tokens / 32);
    return u < 0 ? 0 : u < n_list ? static_cast<int32_t>(u) : n_list;
}

// Waves per 16- or 32-row workgroup: they share the work item's keys.  A
// workgroup of w waves takes w of a compute unit's four SIMDs, so up to 256
// workgroups four waves cost nothing, up to 512 two; past that the extra waves
// only queue.  16 rows, INT4, us at 1 / 2 / 4 waves:
//                 64 tokens           256                  480                 1 024
//   256 items  10.7 /  9.9 / 10.3  22.3 / 16.7 / 14.9  35.7 / 24.4 / 19.9  68.2 / 41.0 / 28.4
//   264        11.3 / 11.9 / 18.4  23.5 / 18.4 / 26.6  37.4 / 26.1 / 34.5  71.5 / 42.3 / 51.2
//   512        13.1 / 13.6 / 20.5  26.1 / 20.6 / 30.3  39.8 / 28.9 / 39.4  74.5 / 49.4 / 59.4
//   520        13.6 / 21.6 / 28.9  26.1 / 34.1 / 42.4  40.2 / 49.5 / 54.8  74.7 / 82.7 / 81.6
// INT2 and the BF16 cache, and 32 rows (at 64 heads two row blocks: the same
// lines at 128 and 256 items), fall the same way.
constexpr int kCus = 256;
constexpr int narrow_waves(int64_t blocks) { return blocks <= kCus ? 4 : blocks <= 2 * kCus ? 2 : 1; }

// The shape a launch runs in: the shortest by a cost of rounds x (fixed + tiles
// x per-tile) us, tiles of 32 tokens per wave.  Fewer rows per workgroup repeat
// the dequantization (and the reads) for every row block, but a launch of few
// work items leaves most of the chip to them; the constants are fits to kernel
// times over 4 to 512 work items of 64 to 2 048 tokens at 64, 128 and 256 rows
// (INT4; INT2 within 5 %).  For 128 rows, at 16 / 32 / 128 rows per workgroup:
//   16 items of 512 tokens    21.6 /  28.3 /  39.3 us
//   64 items of 512           33.0 /  31.2 /  42.1
//   64 items of 2 048         83.2 /  66.4 / 114.9
//   128 items of 64           19.2 /  21.4 /  19.9
//   128 items of 2 048       148.7 / 110.9 / 117.7
//   256 items of 512          89.3 /  67.0 /  51.4
// and for 64 rows, at 16 / 32 / 64:
//   128 items of 512          31.8 /  30.7 /  38.7
//   256 items of 512          47.9 /  42.8 /  44.0
//   272 items of 64           25.2 /  21.9 /  33.6 (the 64-row ones in two rounds)
//   272 items of 2 048       269.9 / 198.5 / 188.5
struct ShapeCost { float fixed, per_tile; };
// Tokens per work item that an unsplit launch is taken to have.  Its lengths are
// on the device, and the page table's width says little about them (a table is
// padded to its longest sequence, or to the longest one that may come); a width
// in the rule would also let the padding choose the order of a sequence's sums.
// By the cost below, over up to 96 sequences of 192 to 512 tokens the shape for
// 2 048 is at most 10 % from the best one (0.3 % on average), and over any
// number of any length at most 5 % from the 64- or 128-row one; the shape for
// 512 tokens is up to 35 % from that one on long sequences.  Measured at 8 to
// 256 sequences of 200, 330 and 512 tokens, the shape for their own length is
// the faster only at 200, in 4 of 40 launches (64 heads, 96 x 200: 17.3 us
// against 19.3).
constexpr int64_t kUnsplitTokens = 2048;
inline LaunchShape choose_shape(bool lowbit, int64_t rows, int64_t num_work, int64_t tokens) {
    // [16 rows, 32 rows][4, 2, 1 waves], then 64 and 128 rows
    static constexpr ShapeCost kNarrowLowbit[2][3] = {{{12.0f, 0.62f}, {13.5f, 1.07f}, {14.8f, 2.08f}},
                                                      {{17.5f, 0.72f}, {18.5f, 1.45f}, {20.0f, 2.95f}}};
    static constexpr ShapeCost kNarrowBf16[2][3] = {{{11.5f, 0.82f}, {13.0f, 1.8f}, {15.5f, 3.4f}},
                                                    {{15.5f, 1.05f}, {18.5f, 2.2f}, {21.0f, 3.9f}}};
    static constexpr ShapeCost kWide[2][2] = {{{18.5f, 1.25f}, {17.5f, 1.6f}}, {{17.5f, 1.1f}, {17.5f, 1.4f}}};
    if (rows <= 16) return {16, narrow_waves(decode_workgroups(num_work, rows, 16))};
    LaunchShape best{32, 1};        // (up to 32 rows; replaced below in any case)
    float least = HUGE_VALF;
    const float n = static_cast<float>((tokens + 31) / 32);
    if (rows > kNarrowRows) {
        const bool half = rows <= 64;
        const ShapeCost c = kWide[lowbit ? 0 : 1][half ? 0 : 1];
        best = {half ? 64 : 128, 4};
        const int64_t blocks = decode_workgroups(num_work, rows, kDecodeRowsPerBlock);
        least = static_cast<float>((blocks + kCus - 1) / kCus) * (c.fixed + n * c.per_tile);
    }
    for (int i = 0; i < 2; ++i) {
        const int64_t blocks = decode_workgroups(num_work, rows, i == 0 ? 16 : 32);
        const int w = narrow_waves(blocks);
        if (blocks * w * kWaveThreads > kMaxDispatchItems) continue;        // (the host checked the other shapes)
        // the bf16 weights of one-wave workgroups (decode_narrow.hip) are left to
        // launches of at most 32 rows
        if (!lowbit && w == 1 && rows > kNarrowRows) continue;
        const ShapeCost c = (lowbit ? kNarrowLowbit : kNarrowBf16)[i][w == 4 ? 0 : w == 2 ? 1 : 2];
        const float rounds = static_cast<float>((blocks * w + 4 * kCus - 1) / (4 * kCus));
        const float cost = rounds * (c.fixed + n * c.per_tile);
        if (cost < least) {
            least = cost;
            best = {i == 0 ? 16 : 32, w};
        }
    }
    return best;
}
// Whether a decode of `rows` query rows may run in shape s: one that choose_shape
// gives to some launch of that many rows, and that fits one dispatch.
inline bool shape_allowed(bool lowbit, int64_t rows, int64_t num_work, LaunchShape s) {
    if (decode_workgroups(num_work, rows, s.rows > 0 ? s.rows : 1) * s.waves * kWaveThreads > kMaxDispatchItems) return false;
    if (s.rows == 64) return s.waves == 4 && rows > kNarrowRows && rows <= 64;
    if (s.rows == 128) return s.waves == 4 && rows > 64;
    if (s.rows != 16 && !(s.rows == 32 && rows > 16)) return false;
    return s.waves == 4 || s.waves == 2 || (s.waves == 1 && (lowbit || rows <= kNarrowRows));
}

// For tests and measurements of one shape (exported, not part of the public ABI).
// mla_internal_decode_shape: the shape a decode call runs in, 8 * rows + waves
// (split_tokens = 0: unsplit).  mla_internal_shape_next_decode: the calling
// thread's next decode call that launches runs in this shape, or returns
// MLA_EINVAL if the shape is not one for its rows; one-shot, 0 and 0 clear it.
extern "C" int32_t mla_internal_decode_shape(int32_t lowbit, int32_t rows, int32_t num_work, int32_t split_tokens);
extern "C" void mla_internal_shape_next_decode(int32_t rows, int32_t waves);

hipError_t launch_lowbit_append_protected(const AppendArgs& a, hipStream_t stream);
// num_splits (split_indptr[B]) chooses between one wave per row and four waves sharing a row.
hipError_t launch_combine(const CombineArgs& a, int32_t num_splits, hipStream_t stream);

// Split-partial storage owned by the library for the allocation-free decode
// entry point: at most kNoallocSplitRows partial rows (split x query row) of
// kNoallocRowBytes (fp16 latent, fp32 max and sum).  Returns this device's
// part_m / part_s / part_o addresses (resolved on the device's first call).
constexpr int64_t kNoallocSplitRows = 65536;
constexpr int64_t kNoallocRowBytes = 512 * 2 + 2 * 4;
hipError_t noalloc_partials(float** part_m, float** part_s, uint16_t** part_o);

}  // namespace mla
