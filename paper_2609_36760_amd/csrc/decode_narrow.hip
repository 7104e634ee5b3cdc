// Decode attention in workgroups of 16 or 32 query rows: the regime of 16 heads
// and one query token (Appendix F.1, "Native Attention") or of 32 rows, where
// the kernels of decode_attn.hip would leave most of every matrix instruction
// idle, and launches of few work items at any number of rows, where they would
// leave most of the chip idle (choose_shape in internal.h).  Same computation and results contract:
// absorbed MLA scores z_t = tau (q_lat . C_hat_t + q_rope . K_hat_t), softmax,
// latent aggregation O = A C_hat (Sec. 2.1, eq. mla_compact), split partials as
// in Appendix C.5 "Global attention normalization", BF16 protection of sink and
// recent tokens as in Appendix C.5 "BF16 protection and cache lifecycle".
//
// A wave owns kR = 16 or 32 query rows and a key range: a work item (sequence
// or key split), or one of the kW contiguous parts of it that the kW waves of a
// workgroup share and merge at the end.  Waves run one per SIMD, without
// barriers in the loop.  Lane l works in lane group g = l / 16 on index
// i = l % 16.
//
// Per tile of kTok tokens (32 at 16 rows, 16 at 32 rows; low-bit cache):
//   1. each lane loads its own codes from the page straight into registers: of
//      token i (of each 16-token block) the 32 channels 128 j + 32 g .. of each
//      128-channel slice j, one 16-byte load (4 bits) -- 64 consecutive bytes
//      per token and load.  A slice's registers are loaded for the next tile as
//      soon as this tile has used them, one step ahead of their use;
//   2. scores S^T[token][row] = K_tile . Q^T with v_mfma_f32_16x16x32_f16.  The
//      order of the channels in a product's K does not matter as long as both
//      operands agree: k-step 4 j + w takes channels 128 j + 32 g + 8 w .. +8
//      from lane group g, one 32-bit word of 4-bit codes, dequantized in
//      registers (x_hat = scale * (q - zero), one fp16 rounding); the queries
//      are loaded in the same order.  The dequantized content channels are also
//      stored to an fp16 tile in LDS;
//   3. softmax: 16 rows: a lane holds tokens 4 g .. 4 g + 3 of each block for
//      row i; 32 rows: v_permlane16_swap gives lane l tokens 8 (l / 32) .. +8 of
//      row l % 32;
//   4. aggregation O^T[channel][row] += V^T . P^T over the tile's tokens with
//      v_mfma_f32_16x16x32_f16 (16 rows) or v_mfma_f32_32x32x16_f16 (32 rows):
//      V^T read transposed from the fp16 tile with ds_read_b64_tr_b16, P^T
//      straight from the score registers.
// BF16 rows (the BF16 cache, and protected rows from a protection buffer) are
// staged raw into a padded tile of 16 tokens and feed both products directly.
//
// Online softmax as in decode_attn.hip: a per-row reference (log2 units) that
// moves only when a tile exceeds it by more than 2^10, the accumulators
// rescaled on the move; the true maximum is tracked for the split partials.
//
// What bounds it.  A wave alone on its SIMD issues an 8-byte vector instruction
// every 5.1 cycles and a 4-byte one every 4.2 (measured, dependent or not), and
// products hide behind them, so the time is the instruction count: 849 per 32
// tokens at 16 rows, 579 of them vector instructions and 468 of those the
// dequantization; 547 per 16 tokens at 32 rows.  Staging the codes through LDS
// (20 more LDS reads and 6 direct-to-LDS loads per 16 tokens), a 16-token step
// and K = 16 aggregation products took about 480 instructions per 16 tokens.
// Long contexts are also held by the board's power limit: 32 x 64K at 16 heads
// takes 180 us (204 us so) at 1 389 W and 2.06 GHz (2.35 GHz so).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "internal.h"
#include "kernel_common.h"
#include "writer_common.h"

namespace mla {
namespace {

using namespace kc;

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxRows = kNarrowRows;   // rows of the widest wave
constexpr int kDc = 512;
constexpr int kQSteps = 18;         // 576 channels / 32 per k-step
constexpr float kRefSlack = 10.0f;
constexpr float kLn2 = 0.693147180559945309f;

// LDS tiles, in 16-byte units.  Row r of the fp16 content tile starts at unit
// 66 r + r / 8, row r of a raw bf16 tile at 74 r + r / 8: the dequantization
// stores and score reads (16 rows, one chunk each) and the transposing reads
// (per half wave 8 rows of 32 bytes, or 4 rows of two 32-byte pieces 128 bytes
// apart) then fall on distinct banks.
__host__ __device__ constexpr int f16_row(int r) { return 66 * r + (r >> 3); }
__host__ __device__ constexpr int bf_row(int r) { return 74 * r + (r >> 3); }
constexpr int f16_tile_bytes(int tokens) { return 16 * (f16_row(tokens - 1) + 64); }
constexpr int kBfTok = 16;          // tokens per bf16 tile
constexpr int kBfUnits = (bf_row(kBfTok - 1) + 72 + 63) / 64 * 64;
constexpr int kBfTileBytes = 16 * kBfUnits;
constexpr int kBfLoads = kBfUnits / 64;
constexpr int kBfSlots = 2;         // tile slots; the next tile is staged one tile ahead
static_assert(kBfLoads == 19, "bf16 tile staging loads");

template <int KIND> struct NCfg {
    static constexpr bool lowbit = KIND != KIND_BF16;
    static constexpr bool pmeta = KIND == KIND_C4R4P || KIND == KIND_C2R4P;
    static constexpr int cbits = (KIND == KIND_C4R4 || KIND == KIND_C4R4P) ? 4 : 2;
    static constexpr int cc = 512 * cbits / 8;            // content code bytes per token
};

// Tokens per low-bit tile.  16 rows: 32, so that the softmax's and the step's
// fixed work is shared by two 16-token blocks and the aggregation runs at
// K = 32.  32 rows: 16 (the output accumulators and the queries take 400 of the
// 512 registers, which leaves room for one block's codes).
constexpr int narrow_tok(int rows) { return rows == 16 ? 32 : 16; }

// LDS of one wave: the fp16 tile or the bf16 slots, reused by the epilogue (the
// rows on their way out; with several waves the fp32 rows they merge, in two
// halves of the channels at 32 rows).
constexpr int kOutPitch = 1040;
constexpr int merge_pitch(int rows) { return (rows == 16 ? 2048 : 1024) + 16; }
template <int KIND, bool kProt, int kR, int kW>
constexpr int narrow_lds() {
    int n = NCfg<KIND>::lowbit ? f16_tile_bytes(narrow_tok(kR)) : 0;
    if (kProt || !NCfg<KIND>::lowbit) n = n > kBfSlots * kBfTileBytes ? n : kBfSlots * kBfTileBytes;
    const int out = kW == 1 ? kR * kOutPitch : kR * merge_pitch(kR);
    n = n > out ? n : out;
    return (n + 1023) / 1024 * 1024;
}

template <int N>
__device__ __forceinline__ void wait_loads() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(N) : "memory");
}

// value and its copies in lanes ^16, ^32, ^48 combined
__device__ __forceinline__ float max4(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum4(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// max / sum over lane ^ 32
__device__ __forceinline__ float max2(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum2(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Score product of a 32-row wave, accumulating in vector registers: the output
// accumulators fill the accumulation registers, and a score tile kept there
// would push output tiles out and back on every step.  Issued as inline
// assembly, so the waits the compiler would insert are written here: two wait
// states between the vector instruction that wrote an operand and the product,
// and score_ready() before vector instructions read the results (12, more than
// a 16 x 16 x 32 product's result needs).
__device__ __forceinline__ void score_mfma(f32x4& c, f16x8 a, f16x8 b, bool first) {
    if (first)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
    else
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void score_mfma(f32x4& c, bf16x8 a, bf16x8 b, bool first) {
    if (first)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
    else
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void score_ready(f32x4& c0, f32x4& c1) {
    asm volatile("s_nop 7\n\ts_nop 3" : "+v"(c0), "+v"(c1));
}

// 4 x 4 transpose of registers across lane groups: lane group g of register w
// receives what lane group w of register g held.
__device__ __forceinline__ void group_transpose(uint32_t& a0, uint32_t& a1, uint32_t& a2, uint32_t& a3) {
    const auto p = __builtin_amdgcn_permlane32_swap(a0, a2, false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(a1, a3, false, false);
    const auto u = __builtin_amdgcn_permlane16_swap(p[0], q[0], false, false);
    const auto v = __builtin_amdgcn_permlane16_swap(p[1], q[1], false, false);
    a0 = u[0];
    a1 = u[1];
    a2 = v[0];
    a3 = v[1];
}

// Staging of one raw bf16 tile (576 channels per row) into the padded layout:
// unit u belongs to the last row starting at or before it; padding units
// re-read column 71.  Row tok of the tile starts at byte row_start(tok).
template <class RowStart>
__device__ __forceinline__ void stage_narrow_bf16(int k, const uint8_t* src, RowStart row_start, int nvalid,
                                                  uint32_t lds, int lane) {
    const int u = 64 * k + lane;
    int r = min(u / 74, 15);
    if (u < bf_row(r)) --r;
    const int col = min(u - bf_row(r), 71);
    dma16_m0(src, row_start(min(r, nvalid - 1)) + 16 * col, lds + 64 * 16 * k);
}

// Dequantization of 8 channels into fp16 pairs (2p, 2p+1).  In the code layout a
// channel pair sits at one bit offset of the two 16-bit halves of a word: the
// 8 channels are the word's pairs at bit offsets sh0 + CBITS p (a 4-bit word
// holds exactly 8 channels, sh0 = 0; a 2-bit word 16, sh0 = 0 or 8).  A pair
// is extracted in place at its offset o within a byte: masked and or'ed with
// 0x6400 it is the fp16 value 1024 + 2^o q.  For o = 0, subtracting
// zz = 1024 + zero leaves q - zero; otherwise one fused multiply-add by 2^-o
// adds zo = -(1024 / 2^o + zero) (zo[o / 2 - 1]).  Both are exact, so the
// word is shifted only by whole bytes, and the one rounding is the multiply
// by the scale.
struct DqWord {
    f16x2 x[4];
    template <int CBITS>
    __device__ __forceinline__ void extract(uint32_t w, int sh0) {
        const uint32_t w0 = CBITS == 4 ? w : w >> sh0, w8 = w >> 8;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t mask = CBITS == 4 ? ((p & 1) ? 0x00F000F0u : 0x000F000Fu) : 0x00030003u << (2 * p);
            x[p] = __builtin_bit_cast(f16x2, and_or(CBITS == 4 && p >= 2 ? w8 : w0, mask, 0x64006400u));
        }
    }
    template <int CBITS>
    __device__ __forceinline__ void center(f16x2 zz, const f16x2* zo) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            constexpr _Float16 kInv[4] = {1.0f16, 0.25f16, 0.0625f16, 0.015625f16};
            const int h = CBITS == 4 ? 2 * (p & 1) : p;         // half the pair's bit offset in its byte
            x[p] = h == 0 ? x[p] - zz : __builtin_elementwise_fma(x[p], f16x2{kInv[h], kInv[h]}, zo[h - 1]);
        }
    }
    __device__ __forceinline__ f16x8 scaled(f16x2 ss) const {
        uint32_t o[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) o[p] = __builtin_bit_cast(uint32_t, x[p] * ss);
        return __builtin_bit_cast(f16x8, make_uint4(o[0], o[1], o[2], o[3]));
    }
};

// zo[k] = -(1024 / 2^o + zero) for o = 2 (k + 1), from zz = 1024 + zero
// (exact: integers and quarters below 1024).
__device__ __forceinline__ void zero_offsets(f16x2 zz, f16x2* zo) {
    zo[0] = f16x2{768.0f16, 768.0f16} - zz;
    zo[1] = f16x2{960.0f16, 960.0f16} - zz;
    zo[2] = f16x2{1008.0f16, 1008.0f16} - zz;
}

// In-launch append (the writer of mla_lowbit_quant_append / mla_bf16_append,
// and under protection of mla_lowbit_quant_append_protected, for the step's
// new tokens), as in decode_attn.hip: the wave that reads a new token
// (`reads(p)`: its part of the key range, or under protection of the key list,
// holds position p; every row block writes the same bytes itself) writes it
// before it loads any tile -- the packed copy (BF16:
// the row), and under protection, for a token protected after the step, its
// bf16 row into ring row p or sink + (p - sink) mod recent of the sequence's
// buffer (skipped for a buffer index outside [0, num_prot)).  One 16-byte
// piece per lane and round (72 per token; a group's 8 lanes stay together,
// as the quantizer needs); the wave's stores land before its first tile's
// loads.  The token's bytes enter no other wave's products, masked or not (the
// first tile leaves out the places below the sink).
template <int KIND, bool kProt, class Reads>
__device__ __forceinline__ void narrow_append(const DecodeArgs& a, int b, int L, Reads reads, int lane) {
    using C = NCfg<KIND>;
    bool any = false;
    for (int i = 0; i < a.s_q; ++i) {
        const int pos = L - a.s_q + i;
        if (pos >= 0 && reads(pos)) any = true;
    }
    if (!any) return;
    const int64_t num_slots = a.num_pages * a.g.page_size;
    for (int piece = lane; piece < 72 * a.s_q; piece += 64) {
        const int i = piece / 72, r = piece % 72;
        const int pos = L - a.s_q + i;
        if (pos < 0 || !reads(pos)) continue;
        const int64_t tok = static_cast<int64_t>(b) * a.s_q + i;
        const int64_t slot = a.new_slots[tok];
        if (slot < 0 || slot >= num_slots) continue;
        const wc::SlotPos at = wc::split_slot(slot, num_slots, a.g);
        uint8_t* base = const_cast<uint8_t*>(a.cache) + at.page * a.g.page_bytes;
        const int64_t off = at.off;
        const bool rope = r >= 64;
        const uint16_t* src = rope ? a.new_k + tok * a.new_k_stride + (r - 64) * 8
                                   : a.new_c + tok * a.new_c_stride + r * 8;
        const uint4 raw = *reinterpret_cast<const uint4*>(src);
        if constexpr (C::lowbit) {
            wc::quantize_store<C::cbits, C::pmeta>(raw, rope, r >> 3, r & 7, base, off, a.g);
            if constexpr (kProt) {
                const int64_t ps = a.prot_slot[b];
                if ((pos < a.sink || pos >= L - a.recent) && ps >= 0 && ps < a.num_prot) {
                    const int prow = pos < a.sink ? pos : a.sink + (pos - a.sink) % a.recent;
                    uint8_t* dst = const_cast<uint8_t*>(a.prot) + (ps * (a.sink + a.recent) + prow) * 1152 + 16 * r;
                    *reinterpret_cast<uint4*>(dst) = raw;
                }
            }
        } else {
            *reinterpret_cast<uint4*>(base + off * 1152 + r * 16) = raw;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A load of the packed cache: base + 32-bit lane offset, marked non-temporal
// (the cache bytes are read once per step).
template <class T>
__device__ __forceinline__ T load_nt(const uint8_t* base, uint32_t off) {
    return __builtin_nontemporal_load(reinterpret_cast<const T*>(base + off));
}

// table[index], waited for on the spot.  Inline assembly, so that the compiler
// does not count it among the loads in flight: a load on one side of a branch
// makes it wait for all of them at the loop's start.
__device__ __forceinline__ int load_waited(const int32_t* table, int index) {
    int v;
    asm volatile("global_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(v)
                 : "v"(index * 4), "s"(table)
                 : "memory");
    return v;
}

// ---------------------------------------------------------------------------
template <int KIND, bool kProt, int kR, int kW>
__global__ __launch_bounds__(64 * kW) __attribute__((amdgpu_waves_per_eu(1, 1)))
void narrow_kernel(DecodeArgs a) {
    static_assert(kR == 16 || kR == kMaxRows, "rows per wave");
    constexpr int kLds = narrow_lds<KIND, kProt, kR, kW>();
    static_assert(kLds * kW <= 160 * 1024 && (kW > 1 || 4 * kLds <= 160 * 1024), "one wave per SIMD fits the LDS");
    __shared__ __attribute__((aligned(1024))) uint8_t smem_all[kLds * kW];

    const int lane = threadIdx.x & 63;
    const int wave = kW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* smem = smem_all + wave * kLds;
    const int g = lane >> 4;            // lane group
    const int li = lane & 15;           // index in the group: token of the score A operand, row of its B operand
    const int half = lane >> 5;
    const int rows_total = a.s_q * a.H;
    const int RB = (rows_total + kR - 1) / kR;

    // Block -> (work item, row block): contiguous work items per XCD (block
    // id mod 8), as in decode_attn.hip.
    const int per_xcd = (a.num_work + 7) / 8;
    const int slot = blockIdx.x >> 3;
    const int w = (blockIdx.x & 7) * per_xcd + slot / RB;
    const int rb = slot % RB;
    if (w >= a.num_work) return;

    const int P = a.g.page_size;
    int b, split = 0;
    int Lraw;
    if (a.split_tokens == 0) {
        b = w;
        Lraw = a.seq_lens[b];
    } else {
        // the last b with split_indptr[b] <= w, counted 64 entries at a time
        // with the lengths loaded alongside: one round of loads instead of a
        // chain of dependent ones (as in decode_attn.hip)
        int cnt = 0, start = 0;
        Lraw = 0;
        for (int base = 0; base <= a.B; base += 64) {
            const int idx = base + lane;
            const int ip = idx <= a.B ? a.split_indptr[idx] : 0x7FFFFFFF;
            const int sl = idx < a.B ? a.seq_lens[idx] : 0;
            const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(ip <= w));
            const int last = cnt + c - 1 - base;     // lane of the last such entry in this chunk
            if (c > 0 && last >= 0 && last < 64) {
                start = __builtin_amdgcn_readlane(ip, last);
                Lraw = __builtin_amdgcn_readlane(sl, last);
            }
            cnt += c;
        }
        b = min(cnt - 1, a.B - 1);
        split = w - start;
    }
    const int L = min(max(Lraw, 0), a.max_pages * P);
    const int32_t* bt = a.block_table + static_cast<int64_t>(b) * a.max_pages;

    // this lane's query row in the softmax and the output (li, or l % 32)
    const int lrow = kR == 16 ? li : (lane & 31);
    const int row = rb * kR + lrow;
    const bool row_ok = row < rows_total;
    const int qi = row_ok ? row / a.H : 0;

    float m_ref = -INFINITY, m_true = -INFINITY, l_run = 0.0f;
    // output accumulators.  16 rows: acc[m], channels 16 m + 4 g + v of row li;
    // 32 rows: acc[m], channels out_channel(m, 8 (v / 4) + 4 half + v % 4) of row l % 32
    constexpr int kAccs = kR == 16 ? 32 : 16;
    using AccT = std::conditional_t<kR == 16, f32x4, f32x16>;
    constexpr int kAccLen = kR == 16 ? 4 : 16;
    AccT acc[kAccs];
#pragma unroll
    for (int m = 0; m < kAccs; ++m) acc[m] = AccT{};

    const uint8_t* ring_base = nullptr;
    int ring_rows = 1, ring_nsink = 0, ring_q0 = 0;

    // Transposing reads of V^T from a tile with row starts `rowf` (in units):
    // 16 rows: product m takes channels 16 m ..; lane group g's first read
    // covers tokens 4 g .. of the tile (the second, K = 32, 16 tokens on).
    // 32 rows: product m takes channels 16 x .. (lanes with l / 16 even) and
    // 16 (x + 4) .. (odd), x = 8 (m / 4) + m % 4, tokens 8 half .. + 3, then + 4 .. + 7.
    auto tr_lane_off = [&](auto rowf) {
        return kR == 16 ? 16 * rowf(4 * g + (li >> 2)) + 8 * (li & 3)
                        : 16 * rowf(8 * half + (li >> 2)) + 128 * (g & 1) + 8 * (li & 3);
    };
    auto tr_imm = [](int m) { return kR == 16 ? 32 * m : 32 * (8 * (m >> 2) + (m & 3)); };
    auto tr_read = [](const uint8_t* p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p); };

    // One phase over keys [t_begin, t_end) in one representation (see
    // decode_attn.hip): PK is the cache kind whose pipeline runs; kRing reads
    // bf16 rows of the protection buffer.  This lane's row sees keys
    // t_lo <= t < lim; every valid row sees t < full_lim.
    auto run = [&](auto kind_c, auto ring_c, const int t_begin, const int t_end, const int t_lo, const int lim,
                   const int full_lim) __attribute__((always_inline)) {
        constexpr int PK = decltype(kind_c)::value;
        constexpr bool kRing = decltype(ring_c)::value;
        using C = NCfg<PK>;
        using OpT = std::conditional_t<C::lowbit, f16x8, bf16x8>;
        constexpr int kTok = C::lowbit ? narrow_tok(kR) : kBfTok;
        constexpr int kNB = kTok / 16;          // 16-token blocks per tile
        constexpr int kNR = kR / 16;            // 16-row blocks
        constexpr int kScores = 4 * kNB * kNR;  // scores per lane and tile
        const int n_tiles = t_end > t_begin ? (t_end - t_begin + kTok - 1) / kTok : 0;
        (void)t_lo;
        if (n_tiles == 0) return;

        // queries: B operand of the scores.  BF16 rows: k-step kk of row block r
        // holds channels 32 kk + 8 g .. +8 of row 16 r + li.  Low-bit tiles take the
        // order of the code loads: k-step 4 j + w holds channels 128 j + 32 g + 8 w
        // .. +8.  Read in that order each load would touch 64 separate pieces; they
        // are read in the plain order (64 bytes of a row per load) and the four
        // loads of a slice transposed across the lane groups.
        OpT qf[kNR][kQSteps];
        uint4 rawq[kNR][kQSteps];
        auto read_q = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < kNR; ++r) {
                // rows past the end read row 0 of the sequence; their results are never stored
                const int rr = rb * kR + 16 * r + li;
                const int64_t qrow = static_cast<int64_t>(b) * rows_total + (rr < rows_total ? rr : 0);
                const uint16_t* ql = a.q_lat + qrow * kDc + 8 * g;
                const uint16_t* qr = a.q_rope + qrow * 64 + (C::lowbit ? 16 : 8) * g;
#pragma unroll
                for (int kk = 0; kk < kQSteps; ++kk)
                    rawq[r][kk] = *reinterpret_cast<const uint4*>(kk < 16 ? ql + 32 * kk : qr + (C::lowbit ? 8 : 32) * (kk - 16));
            }
        };
        auto set_q = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < kNR; ++r) {
                if constexpr (C::lowbit) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        group_transpose(rawq[r][4 * j].x, rawq[r][4 * j + 1].x, rawq[r][4 * j + 2].x, rawq[r][4 * j + 3].x);
                        group_transpose(rawq[r][4 * j].y, rawq[r][4 * j + 1].y, rawq[r][4 * j + 2].y, rawq[r][4 * j + 3].y);
                        group_transpose(rawq[r][4 * j].z, rawq[r][4 * j + 1].z, rawq[r][4 * j + 2].z, rawq[r][4 * j + 3].z);
                        group_transpose(rawq[r][4 * j].w, rawq[r][4 * j + 1].w, rawq[r][4 * j + 2].w, rawq[r][4 * j + 3].w);
                    }
                }
#pragma unroll
                for (int kk = 0; kk < kQSteps; ++kk) {
                    const uint4 v = rawq[r][kk];
                    if constexpr (C::lowbit)
                        qf[r][kk] = __builtin_bit_cast(f16x8, make_uint4(bf16x2_to_f16x2(v.x), bf16x2_to_f16x2(v.y),
                                                                         bf16x2_to_f16x2(v.z), bf16x2_to_f16x2(v.w)));
                    else
                        qf[r][kk] = __builtin_bit_cast(bf16x8, v);
                    // 16 rows: kept in accumulation registers, which the score
                    // products read directly as their B operand
                    if constexpr (kR == 16) asm volatile("" : "+a"(qf[r][kk]));
                }
            }
        };

        // online softmax of one tile's scores s: masks, moves the reference
        // (rescaling the accumulators, which hold every earlier tile) when
        // needed, returns the weights.  Score v of a lane is token tok_of(v).
        auto tok_of = [&](int v) {
            return kR == 16 ? 16 * (v >> 2) + 4 * g + (v & 3) : 8 * half + v;
        };
        auto softmax = [&](int it, float (&s)[kScores], float (&p)[kScores]) __attribute__((always_inline)) {
            const int t0 = t_begin + it * kTok;
            // rows see every key of the tile except in the last tile of the range,
            // the tile holding the newest key, or the one with the last sink token
            // (wave-uniform test)
            bool edge = t0 + kTok > full_lim;
            if constexpr (kProt) edge = edge || t0 < t_lo;
            if (edge) {
#pragma unroll
                for (int v = 0; v < kScores; ++v) {
                    const int t = t0 + tok_of(v);
                    bool ok = t < lim;
                    if constexpr (kProt) ok = ok && t >= t_lo;
                    s[v] = ok ? s[v] : -INFINITY;
                }
            }
            float mr = s[0];
#pragma unroll
            for (int v = 1; v < kScores; ++v) mr = fmaxf(mr, s[v]);
            mr = kR == 16 ? max4(mr) : max2(mr);
            const float mt = mr * a.scale_log2;
            m_true = fmaxf(m_true, mt);
            if (m_ref == -INFINITY) m_ref = mt;
            const bool move = __builtin_amdgcn_ballot_w64(mt > m_ref + kRefSlack) != 0;
            if (move) {
                const float m_new = fmaxf(m_ref, mt);
                const float alpha = m_new == m_ref ? 1.0f : __builtin_amdgcn_exp2f(m_ref - m_new);
                m_ref = m_new;
                l_run *= alpha;
                if constexpr (kR == 16) {
#pragma unroll
                    for (int m = 0; m < kAccs; ++m) acc[m] *= alpha;
                } else {
                    // in place: the accumulators fill the accumulation registers (the
                    // score products between them and here cover their latency)
#pragma unroll
                    for (int m = 0; m < kAccs; ++m)
#pragma unroll
                        for (int v = 0; v < kAccLen; ++v) {
                            float t;
                            asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                                         : "+a"(acc[m][v]), "=&v"(t)
                                         : "v"(alpha));
                        }
                }
            }
            const float nref = m_ref == -INFINITY ? 0.0f : -m_ref;
#pragma unroll
            for (int v = 0; v < kScores; ++v) p[v] = __builtin_amdgcn_exp2f(fmaf(s[v], a.scale_log2, nref));
        };

        if constexpr (C::lowbit) {
            // Software pipeline: step it computes the scores of tile it (its
            // operands dequantized in registers) interleaved with the aggregation
            // of tile it-1 (read transposed from the fp16 tile).
            int pg = t_begin / P, po = t_begin % P;     // page and offset of the tile to load next
            int pid_base = pg;                          // lane l holds the id of page pid_base + l
            int pids = bt[min(pid_base + lane, a.max_pages - 1)];

            // One tile's packed bytes in registers, per 16-token block: content
            // codes (slice j: channels 128 j + 32 g .. +32), RoPE codes (channels
            // 16 g .. +16) and the metadata of the lane's groups 2 j + g / 2 (paper
            // storage: the token's whole record).
            using CodeT = std::conditional_t<C::cbits == 4, u32x4, u32x2>;
            CodeT cw[kNB][4];
            u32x2 rw[kNB];
            uint32_t mw[kNB][4], rmw[kNB];
            u32x4 pm0[kNB], pm1[kNB];
            const uint8_t* page = nullptr;
            uint32_t oc[kNB], orc[kNB], om[kNB], orm[kNB];
            // page and lane offsets of tile j, and the cursor's move to the next
            // tile (past the end it stays on the last, which is then read again for
            // nothing).  Tokens of the tile below `first` read token `first`.
            auto locate = [&](int j, int first) __attribute__((always_inline)) {
                const int t0 = t_begin + min(j, n_tiles - 1) * kTok;
                const int last = min(t_end - t0, kTok) - 1;     // tokens past it re-read it
                if (pg - pid_base == 64) {
                    pid_base = pg;
                    pids = load_waited(bt, min(pid_base + lane, a.max_pages - 1));
                }
                int pid = __builtin_amdgcn_readlane(pids, pg - pid_base);
                pid = min(max(pid, 0), static_cast<int>(a.num_pages - 1));
                page = a.cache + static_cast<uint64_t>(static_cast<uint32_t>(pid)) * static_cast<uint32_t>(a.g.page_bytes);
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    const uint32_t t = static_cast<uint32_t>(po + min(max(16 * nb + li, first), last));
                    oc[nb] = t * C::cc + (C::cbits == 4 ? 16 : 8) * g;
                    orc[nb] = static_cast<uint32_t>(a.g.off_cr) + t * 32 + 8 * g;
                    om[nb] = static_cast<uint32_t>(a.g.off_mc) + t * 32 + (C::pmeta ? 0 : 4 * (g >> 1));
                    orm[nb] = static_cast<uint32_t>(a.g.off_mr) + t * 4;
                }
                if (j < n_tiles - 1) {
                    po += kTok;
                    if (po == P) {
                        po = 0;
                        ++pg;
                    }
                }
            };
            auto load_slice = [&](int j) __attribute__((always_inline)) {
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    cw[nb][j] = load_nt<CodeT>(page, oc[nb] + (C::cbits == 4 ? 64 : 32) * j);
                    if constexpr (!C::pmeta) mw[nb][j] = load_nt<uint32_t>(page, om[nb] + 8 * j);
                }
            };
            auto load_rope = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    rw[nb] = load_nt<u32x2>(page, orc[nb]);
                    if constexpr (C::pmeta) {
                        pm0[nb] = load_nt<u32x4>(page, om[nb]);
                        pm1[nb] = load_nt<u32x4>(page, om[nb] + 16);
                    } else {
                        rmw[nb] = load_nt<uint32_t>(page, orm[nb]);
                    }
                }
            };

            // dequantization constants of slice j (j = 4: the RoPE group) of a
            // block's token: scale, 1024 + zero, and the zero offsets of the
            // in-place extraction
            struct Gm { f16x2 zz, ss, zo[3]; };
            auto group_meta = [&](int nb, int j) __attribute__((always_inline)) {
                Gm m;
                if constexpr (C::pmeta) {
                    if (j == 4) {
                        pmeta_to_f16(__uint_as_float(pm1[nb][2]), pm1[nb][3] & 0xFFu, m.zz, m.ss);
                    } else {
                        // group 2 j + g / 2: scale in half g / 2 of word j, zero in byte 2 j + g / 2
                        const uint32_t sbits = (pm0[nb][j] >> (16 * (g >> 1))) << 16;
                        const uint32_t z = ((j < 2 ? pm1[nb][0] : pm1[nb][1]) >> (16 * (j & 1) + 8 * (g >> 1))) & 0xFFu;
                        pmeta_to_f16(__uint_as_float(sbits), z, m.zz, m.ss);
                    }
                } else {
                    meta_to_f16(j == 4 ? rmw[nb] : mw[nb][j], m.zz, m.ss);
                }
                zero_offsets(m.zz, m.zo);
                return m;
            };
            // k-step kk's channels of every block (the three operations per pair,
            // operation by operation over all blocks: a packed operation that
            // reads the one just before it costs a wait state)
            auto dq = [&](int kk, const Gm (&m)[kNB], f16x8 (&o)[kNB]) __attribute__((always_inline)) {
                DqWord x[kNB];
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    const int j = (kk >> 2) & 3, wd = kk & 3;
                    if (kk >= 16) x[nb].template extract<4>(rw[nb][kk & 1], 0);
                    else if constexpr (C::cbits == 4) x[nb].template extract<4>(cw[nb][j][wd], 0);
                    else x[nb].template extract<2>(cw[nb][j][wd >> 1], 8 * (wd & 1));
                }
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) {
                    if (kk >= 16 || C::cbits == 4) x[nb].template center<4>(m[nb].zz, m[nb].zo);
                    else x[nb].template center<2>(m[nb].zz, m[nb].zo);
                }
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb) o[nb] = x[nb].scaled(m[nb].ss);
            };

            // the page ids' round trip overlaps the query loads' issue
            read_q();
            __builtin_amdgcn_sched_barrier(0);
            // Masked tokens below t_lo (the sink, in the first tile) are not loaded:
            // they enter the aggregation with weight 0, and one that is new in this
            // launch is written by the wave of the protected rows, which nothing
            // orders with this wave's loads (0 x the stale bytes can be NaN).
            locate(0, kProt ? max(t_lo - t_begin, 0) : 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) load_slice(j);
            load_rope();
            __builtin_amdgcn_sched_barrier(0);
            set_q();

            uint8_t* tile = smem;
            const uint8_t* vbase = tile + tr_lane_off(f16_row);
            constexpr int kVOff = kR == 16 ? 16 * (f16_row(16) - f16_row(0)) : 16 * (f16_row(4) - f16_row(0));
            static_assert(f16_row(31) - f16_row(15) == f16_row(16) - f16_row(0) && f16_row(15) - f16_row(11) == f16_row(4),
                          "second transposing read at a fixed offset");
            f16x8 pb{};                                  // weights of the previous tile (P^T operand)
            // k-steps of slice j store channels of the slice's eight 16-channel
            // blocks, so their transposing reads come 8 blocks ahead
            constexpr int kVAhead = kAccs / 4;
            f16x8 vb[kVAhead];
            auto vread = [&](int m) __attribute__((always_inline)) {
                const i16x4 v0 = tr_read(vbase + tr_imm(m));
                const i16x4 v1 = tr_read(vbase + tr_imm(m) + kVOff);
                return __builtin_bit_cast(f16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            auto pv = [&](int m) __attribute__((always_inline)) {
                if constexpr (kR == 16)
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vb[m % kVAhead], pb, acc[m], 0, 0, 0);
                else
                    acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vb[m % kVAhead], pb, acc[m], 0, 0, 0);
                if (m + kVAhead < kAccs) vb[m % kVAhead] = vread(m + kVAhead);
            };
            // one step: scores of tile it (QK), the loads of tile it+1, and the
            // aggregation of tile it-1 (PV).  Tile it's content channels replace
            // tile it-1's as soon as they are dequantized: the transposing reads of
            // those blocks were issued before, and LDS serves one wave's accesses
            // in the order they are issued.
            auto step = [&](int it, auto QK, auto PV) __attribute__((always_inline)) {
                constexpr bool kQK = decltype(QK)::value, kPV = decltype(PV)::value;
                f32x4 s[kNB][kNR];
#pragma unroll
                for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
                    for (int r = 0; r < kNR; ++r) s[nb][r] = f32x4{};
                if constexpr (kQK) locate(it + 1, 0);
                if constexpr (kPV) {
#pragma unroll
                    for (int m = 0; m < kVAhead; ++m) vb[m] = vread(m);
                }
                __builtin_amdgcn_sched_barrier(0);
                // the dequantization runs one k-step ahead of the score products,
                // so that vector work separates the products
                Gm gm[kNB];
                f16x8 kv_next[kNB];
                if constexpr (kQK) {
#pragma unroll
                    for (int nb = 0; nb < kNB; ++nb) gm[nb] = group_meta(nb, 0);
                    dq(0, gm, kv_next);
                }
#pragma unroll
                for (int kk = 0; kk < kQSteps; ++kk) {
                    f16x8 kv[kNB];
                    if constexpr (kQK) {
#pragma unroll
                        for (int nb = 0; nb < kNB; ++nb) {
                            kv[nb] = kv_next[nb];
#pragma unroll
                            for (int r = 0; r < kNR; ++r) {
                                if constexpr (kR == 16)
                                    s[nb][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kv[nb], qf[r][kk], s[nb][r], 0, 0, 0);
                                else
                                    score_mfma(s[nb][r], kv[nb], qf[r][kk], kk == 0);
                            }
                        }
                    }
                    if constexpr (kPV) {
                        if (kk < 16) {
                            pv(kAccs / 16 * kk);
                            if constexpr (kAccs == 32) pv(2 * kk + 1);
                        }
                    }
                    if constexpr (kQK) {
                        if (kk + 1 < kQSteps) {
#pragma unroll
                            for (int nb = 0; nb < kNB; ++nb)
                                if (((kk + 1) & 3) == 0) gm[nb] = group_meta(nb, (kk + 1) >> 2);
                            dq(kk + 1, gm, kv_next);
                        }
                        // slice (kk + 1) / 4 is used up: its registers take the next tile's
                        if (kk < 16 && ((kk + 1) & 3) == 3) load_slice((kk + 1) >> 2);
                        if (kk + 1 == kQSteps - 1) load_rope();
#pragma unroll
                        for (int nb = 0; nb < kNB; ++nb)
                            if (kk < 16)
                                *reinterpret_cast<f16x8*>(tile + 16 * (f16_row(16 * nb + li) + 16 * (kk >> 2) + 4 * g + (kk & 3))) = kv[nb];
                    }
                    if constexpr (kQK && kPV) {
                        if (kk < 16) {
                            // products spread over the k-step's vector work
                            constexpr int kProducts = kNB * kNR + kAccs / 16;
                            constexpr int kGap = kR == 16 ? 7 : 5;
#pragma unroll
                            for (int i = 0; i < kProducts; ++i) {
                                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                                __builtin_amdgcn_sched_group_barrier(0x002, kGap, 0);
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (kQK) {
                    float sc[kScores], p[kScores];
                    if constexpr (kR == 16) {
#pragma unroll
                        for (int v = 0; v < kScores; ++v) {
                            sc[v] = s[(v >> 2) % kNB][0][v & 3];
                            // out of the accumulation registers once, before the branches
                            asm volatile("" : "+v"(sc[v]));
                        }
                    } else {
                        score_ready(s[0][0], s[0][kNR - 1]);
                        // lanes of row block 0 and 1 exchange, so that lane l holds row
                        // l % 32: {a0 b0 a2 b2} tokens 8 half + v, {a1 b1 a3 b3} + 4
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[0][0][v]),
                                                                            __float_as_uint(s[0][kNR - 1][v]), false, false);
                            sc[v] = __uint_as_float(x[0]);
                            sc[4 + v] = __uint_as_float(x[1]);
                        }
                    }
                    softmax(it, sc, p);
                    uint32_t pw[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // the normalizer sums the fp16 weights the aggregation uses
                        pw[q] = pack_f16x2(p[2 * q], p[2 * q + 1]);
                        l_run = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, pw[q]), f16x2{1.0f16, 1.0f16}, l_run, false);
                    }
                    pb = __builtin_bit_cast(f16x8, make_uint4(pw[0], pw[1], pw[2], pw[3]));
                }
            };
            step(0, std::true_type{}, std::false_type{});
            for (int it = 1; it < n_tiles; ++it) step(it, std::true_type{}, std::true_type{});
            step(n_tiles, std::false_type{}, std::true_type{});
        } else {
            // raw bf16 rows: both products read the staged tile directly.  Each weight
            // enters the aggregation to 16 significant bits, bf16(w) and the bf16
            // rounding of the exact residual w - bf16(w) in two products per block,
            // over protected rows and wherever several waves share a work item
            // (launches bound by latency, which the second product hardly lengthens);
            // else the weights are bf16 alone and the normalizer sums them rounded.
            constexpr bool kPairW = kRing || kW > 1;
            read_q();
            int st_pg = t_begin / P, st_po = t_begin % P, pid_pg = -1, pid = 0;   // next tile to stage
            auto slot_base = [&](int j) { return smem + slot_offset(j, kBfSlots, kBfTileBytes); };
            auto issue_tile = [&](int j) __attribute__((always_inline)) {
                const int t0 = t_begin + min(j, n_tiles - 1) * kTok;   // past the end: the last tile again
                const int nvalid = min(t_end - t0, kTok);
                const uint32_t lds = lds_addr(slot_base(j));
                if constexpr (kRing) {
                    auto row_start = [&](int tok) {
                        const int v = t0 + tok;
                        const int x = ring_q0 + (v - ring_nsink);       // < 2 * recent
                        const int r = v < ring_nsink ? v : a.sink + (x >= a.recent ? x - a.recent : x);
                        return min(r, ring_rows - 1) * 1152;
                    };
#pragma unroll
                    for (int k = 0; k < kBfLoads; ++k) stage_narrow_bf16(k, ring_base, row_start, nvalid, lds, lane);
                } else {
                    // tiles are issued in order; a 16-token tile never crosses a page
                    // (t_begin and the page size are multiples of 32), and the page
                    // id is fetched once per page
                    if (st_pg != pid_pg) {
                        pid = load_page_id(bt, st_pg);
                        pid = min(max(pid, 0), static_cast<int>(a.num_pages - 1));
                        pid_pg = st_pg;
                    }
                    const uint8_t* page = a.cache + static_cast<int64_t>(pid) * a.g.page_bytes;
                    const int po = st_po;
                    if (j < n_tiles - 1) {
                        st_po += kTok;
                        if (st_po == P) {
                            st_po = 0;
                            ++st_pg;
                        }
                    }
                    auto row_start = [&](int tok) { return (po + tok) * 1152; };
#pragma unroll
                    for (int k = 0; k < kBfLoads; ++k) stage_narrow_bf16(k, page, row_start, nvalid, lds, lane);
                }
            };
            issue_tile(0);
            set_q();
            for (int it = 0; it < n_tiles; ++it) {
                // tile it has landed and every LDS access of the previous step is
                // done; then stage tile it+1 into the slot tile it-1 used
                wait_loads<0>();
                issue_tile(it + 1);
                const uint8_t* st = slot_base(it);
                f32x4 s[kNR];
#pragma unroll
                for (int r = 0; r < kNR; ++r) s[r] = f32x4{};
                constexpr int kKAhead = kR == 16 ? kQSteps : 6;
                bf16x8 kv[kKAhead];
                auto kread = [&](int kk) __attribute__((always_inline)) {
                    return *reinterpret_cast<const bf16x8*>(st + 16 * (bf_row(li) + 4 * kk + g));
                };
#pragma unroll
                for (int kk = 0; kk < kKAhead; ++kk) kv[kk] = kread(kk);
#pragma unroll
                for (int kk = 0; kk < kQSteps; ++kk) {
#pragma unroll
                    for (int r = 0; r < kNR; ++r) {
                        if constexpr (kR == 16)
                            s[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kv[kk % kKAhead], qf[r][kk], s[r], 0, 0, 0);
                        else
                            score_mfma(s[r], kv[kk % kKAhead], qf[r][kk], kk == 0);
                    }
                    if (kk + kKAhead < kQSteps) kv[kk % kKAhead] = kread(kk + kKAhead);
                }
                float sc[kScores], p[kScores];
                if constexpr (kR == 16) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) sc[v] = s[0][v];
                } else {
                    score_ready(s[0], s[kNR - 1]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[0][v]),
                                                                        __float_as_uint(s[kNR - 1][v]), false, false);
                        sc[v] = __uint_as_float(x[0]);
                        sc[4 + v] = __uint_as_float(x[1]);
                    }
                }
                softmax(it, sc, p);
                uint32_t ph[kScores / 2], pl[kScores / 2];
#pragma unroll
                for (int q = 0; q < kScores / 2; ++q) {
                    ph[q] = pack_bf16x2(p[2 * q], p[2 * q + 1]);
                    const float h0 = __uint_as_float(ph[q] << 16), h1 = __uint_as_float(ph[q] & 0xFFFF0000u);
                    pl[q] = pack_bf16x2(p[2 * q] - h0, p[2 * q + 1] - h1);
                    l_run += kPairW ? p[2 * q] : h0;
                    l_run += kPairW ? p[2 * q + 1] : h1;
                }
                // aggregation, transposing reads eight (16 rows) or four blocks
                // ahead of the products
                const uint8_t* vbase = st + tr_lane_off(bf_row);
                constexpr int kVAhead = kR == 16 ? 8 : 4;
                if constexpr (kR == 16) {
                    s16x4 vb[kVAhead];
                    const s16x4 pbh = __builtin_bit_cast(s16x4, make_uint2(ph[0], ph[1]));
                    const s16x4 pbl = __builtin_bit_cast(s16x4, make_uint2(pl[0], pl[1]));
#pragma unroll
                    for (int m = 0; m < kVAhead; ++m) vb[m] = tr_read(vbase + tr_imm(m));
#pragma unroll
                    for (int m = 0; m < kAccs; ++m) {
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vb[m % kVAhead], pbh, acc[m], 0, 0, 0);
                        if constexpr (kPairW)
                            acc[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vb[m % kVAhead], pbl, acc[m], 0, 0, 0);
                        if (m + kVAhead < kAccs) vb[m % kVAhead] = tr_read(vbase + tr_imm(m + kVAhead));
                    }
                } else {
                    constexpr int kVOff = 16 * (bf_row(4) - bf_row(0));
                    static_assert(bf_row(15) - bf_row(11) == bf_row(4), "second transposing read at a fixed offset");
                    auto vread = [&](int m) __attribute__((always_inline)) {
                        const i16x4 v0 = tr_read(vbase + tr_imm(m));
                        const i16x4 v1 = tr_read(vbase + tr_imm(m) + kVOff);
                        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                    };
                    bf16x8 vb[kVAhead];
                    constexpr int n = kScores / 2;
                    const bf16x8 pbh = __builtin_bit_cast(bf16x8, make_uint4(ph[0], ph[1], ph[2 % n], ph[3 % n]));
                    const bf16x8 pbl = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2 % n], pl[3 % n]));
#pragma unroll
                    for (int m = 0; m < kVAhead; ++m) vb[m] = vread(m);
#pragma unroll
                    for (int m = 0; m < kAccs; ++m) {
                        acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[m % kVAhead], pbh, acc[m], 0, 0, 0);
                        if constexpr (kPairW)
                            acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[m % kVAhead], pbl, acc[m], 0, 0, 0);
                        if (m + kVAhead < kAccs) vb[m % kVAhead] = vread(m + kVAhead);
                    }
                }
            }
            // no direct-to-LDS load may outlive the wave's LDS
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    };

    // Part `wave` of kW of n list entries from u0: an equal share, rounded up.
    auto part = [&](int& u0, int& u1) {
        if constexpr (kW > 1) {
            const int n = max(u1 - u0, 0), per = (n + kW - 1) / kW;
            u1 = min(u0 + (wave + 1) * per, u0 + n);
            u0 = min(u0 + wave * per, u1);
        }
    };
    if constexpr (!kProt) {
        int t_begin = 0, t_end = L;
        if (a.split_tokens != 0) {
            t_begin = max(split * a.split_tokens, 0);
            t_end = min(split * a.split_tokens + a.split_tokens, L);
        }
        if constexpr (kW > 1) {
            // 32-token units (t_begin is a multiple of 32)
            int u0 = t_begin / 32, u1 = max((t_end + 31) / 32, u0);
            part(u0, u1);
            t_begin = 32 * u0;
            t_end = min(32 * u1, t_end);
        }
        const int lim = row_ok ? min(L - a.s_q + qi + 1, t_end) : t_begin;
        const int full_lim = min(L - a.s_q + 1, t_end);
        if (a.new_c != nullptr)
            narrow_append<KIND, false>(a, b, L, [&](int pos) { return pos >= t_begin && pos < t_end; }, lane);
        run(std::integral_constant<int, KIND>{}, std::false_type{}, t_begin, t_end, t_begin, lim, full_lim);
    } else {
        // the tile list of mla_plan_splits_protected (32-key list tiles)
        const int sink = a.sink, recent = a.recent;
        const bool has_packed = L - recent > sink;
        const int pk0 = has_packed ? sink / 32 : 0;
        const int n_pk = has_packed ? (L - recent + 31) / 32 - pk0 : 0;
        const int n_prot = has_packed ? sink + recent : L;
        const int n_list = n_pk + (n_prot + 31) / 32;
        int u0 = 0, u1 = n_list;
        if (a.split_tokens != 0) {
            u0 = split_tile(split, a.split_tokens, n_list);
            u1 = min(u0 + a.split_tokens / 32, n_list);
        }
        part(u0, u1);
        if constexpr (NCfg<KIND>::lowbit) {
            if (a.new_c != nullptr) {
                // list tile of position p: a packed position by its tile (from the
                // tile holding token `sink`), a protected one by its index among
                // the protected rows
                const int nsink = min(sink, L), r0 = max(sink, L - recent);
                auto reads = [&](int pos) {
                    const bool prot = pos < sink || pos >= L - recent;
                    const int u = prot ? n_pk + (min(pos, nsink) + max(0, pos - r0)) / 32 : pos / 32 - pk0;
                    return u >= u0 && u < u1;
                };
                narrow_append<KIND, true>(a, b, L, reads, lane);
            }
        }
        if (u0 < min(u1, n_pk)) {
            const int tb = 32 * (pk0 + u0);
            const int te = min(32 * (pk0 + min(u1, n_pk)), L - recent);
            const int lim = row_ok ? min(L - a.s_q + qi + 1, te) : tb;
            const int full_lim = min(L - a.s_q + 1, te);
            run(std::integral_constant<int, KIND>{}, std::false_type{}, tb, te, sink, lim, full_lim);
        }
        if (u1 > max(u0, n_pk)) {
            ring_rows = sink + recent;
            ring_nsink = min(sink, L);
            const int r0 = max(sink, L - recent);
            ring_q0 = recent > 0 ? (r0 - sink) % recent : 0;
            int64_t pslot = a.prot_slot[b];
            pslot = pslot < 0 ? 0 : (pslot >= a.num_prot ? a.num_prot - 1 : pslot);
            ring_base = a.prot + pslot * ring_rows * 1152;
            auto below = [&](int x) { return min(max(x, 0), ring_nsink) + max(0, x - r0); };
            const int vb = 32 * (max(u0, n_pk) - n_pk);
            const int ve = min(32 * (u1 - n_pk), n_prot);
            const int lim = row_ok ? min(below(L - a.s_q + qi + 1), ve) : vb;
            const int full_lim = min(below(L - a.s_q + 1), ve);
            run(std::integral_constant<int, KIND_BF16>{}, std::true_type{}, vb, ve, 0, lim, full_lim);
        }
    }

    // ---- epilogue
    const bool split_out = a.split_tokens != 0;
    const int row0 = rb * kR;
    const int last = min(kR, rows_total - row0) - 1;        // the block's last row
    uint16_t* dst = split_out ? a.part_o + (static_cast<int64_t>(w) * rows_total + row0) * kDc
                              : a.out + (static_cast<int64_t>(b) * rows_total + row0) * kDc;
    float l_tot = kR == 16 ? sum4(l_run) : sum2(l_run);
    float f_own = 1.0f;                 // this wave's share of the row is acc * f_own
    if constexpr (kW > 1) {
        // one reference for the row's kW parts: m_ref = max over the waves, the
        // sums and accumulators of each moved to it (a part with no visible key
        // has m_ref = -inf and weighs 0)
        __shared__ float sh[3][kW][kR];
        if (lane < kR) {
            sh[0][wave][lane] = m_ref;
            sh[1][wave][lane] = l_tot;
            sh[2][wave][lane] = m_true;
        }
        __syncthreads();
        const float own = m_ref;
#pragma unroll
        for (int x = 0; x < kW; ++x) {
            m_ref = fmaxf(m_ref, sh[0][x][lrow]);
            m_true = fmaxf(m_true, sh[2][x][lrow]);
        }
        const float nref = m_ref == -INFINITY ? 0.0f : m_ref;
        f_own = __builtin_amdgcn_exp2f(own - nref);
        l_tot = 0.0f;
#pragma unroll
        for (int x = 0; x < kW; ++x) {
            const float fx = __builtin_amdgcn_exp2f(sh[0][x][lrow] - nref);
            l_tot += fx * sh[1][x][lrow];
        }
    }
    const float inv = (l_tot > 0.0f ? 1.0f / l_tot : 0.0f) * f_own;
    // channels of accumulator m, values 4 q .. 4 q + 3
    auto channel = [&](int m, int q) {
        if constexpr (kR == 16) return 16 * m + 4 * g;
        const int x = 8 * (m >> 2) + (m & 3) + (q >= 2 ? 4 : 0);       // 16-channel block
        return 16 * x + 8 * (q & 1) + 4 * half;
    };
    auto pack4 = [&](float x0, float x1, float x2, float x3) {
        return split_out ? make_uint2(pack_f16x2(x0, x1), pack_f16x2(x2, x3))
                         : make_uint2(pack_bf16x2(x0, x1), pack_bf16x2(x2, x3));
    };
    if constexpr (kW == 1) {
        // the rows go out through LDS, one whole row (1 KiB) per store
#pragma unroll
        for (int m = 0; m < kAccs; ++m)
#pragma unroll
            for (int q = 0; q < kAccLen / 4; ++q)
                *reinterpret_cast<uint2*>(smem + lrow * kOutPitch + 2 * channel(m, q)) =
                    pack4(acc[m][4 * q] * inv, acc[m][4 * q + 1] * inv, acc[m][4 * q + 2] * inv, acc[m][4 * q + 3] * inv);
        // (H is a multiple of 16, so at 16 rows every row exists; at 32 rows those
        // past the end repeat the last one: a test per row would leave each row's
        // LDS read waiting alone before its store)
#pragma unroll
        for (int i0 = 0; i0 < kR; i0 += 8) {
            uint4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                v[i] = *reinterpret_cast<const uint4*>(smem + min(i0 + i, last) * kOutPitch + 16 * lane);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                *reinterpret_cast<uint4*>(dst + min(i0 + i, last) * kDc + 8 * lane) = v[i];
        }
    } else {
        // fp32 rows of every wave in LDS, summed and stored by rows: wave x takes
        // rows kR / kW x ..; 16 rows: all 512 channels at once, 32 rows: 256 at a time
        constexpr int kRounds = kR == 16 ? 1 : 2;
        constexpr int kPitch = merge_pitch(kR);
        constexpr int kPer = 8 / kRounds;               // channels per lane
#pragma unroll
        for (int rd = 0; rd < kRounds; ++rd) {
            if (rd > 0) __syncthreads();
#pragma unroll
            for (int m = 0; m < kAccs / kRounds; ++m)
#pragma unroll
                for (int q = 0; q < kAccLen / 4; ++q) {
                    const AccT& x = acc[m + rd * kAccs / kRounds];
                    *reinterpret_cast<float4*>(smem + lrow * kPitch + 4 * channel(m, q)) =
                        make_float4(x[4 * q] * inv, x[4 * q + 1] * inv, x[4 * q + 2] * inv, x[4 * q + 3] * inv);
                }
            __syncthreads();
            // kBatch rows' reads in flight together
            constexpr int kBatch = 16 / (kW * kPer / 4);
            static_assert(kR / kW % kBatch == 0, "whole batches");
#pragma unroll
            for (int i0 = 0; i0 < kR / kW; i0 += kBatch) {
                float4 v[kBatch][kW][kPer / 4];
#pragma unroll
                for (int i = 0; i < kBatch; ++i)
#pragma unroll
                    for (int x = 0; x < kW; ++x)
#pragma unroll
                        for (int c = 0; c < kPer / 4; ++c)
                            v[i][x][c] = *reinterpret_cast<const float4*>(
                                smem_all + x * kLds + min(wave * (kR / kW) + i0 + i, last) * kPitch + 4 * (kPer * lane + 4 * c));
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    uint16_t* op = dst + min(wave * (kR / kW) + i0 + i, last) * kDc + rd * (kDc / kRounds) + kPer * lane;
#pragma unroll
                    for (int c = 0; c < kPer / 4; ++c) {
                        float4 o = v[i][0][c];
#pragma unroll
                        for (int x = 1; x < kW; ++x) {
                            o.x += v[i][x][c].x;
                            o.y += v[i][x][c].y;
                            o.z += v[i][x][c].z;
                            o.w += v[i][x][c].w;
                        }
                        *reinterpret_cast<uint2*>(op + 4 * c) = pack4(o.x, o.y, o.z, o.w);
                    }
                }
            }
        }
        if (wave != 0) return;
    }
    if (!row_ok || lane >= kR) return;
    if (!split_out) {
        if (a.lse != nullptr)
            a.lse[static_cast<int64_t>(b) * rows_total + row] = l_tot > 0.0f ? (m_ref + log2f(l_tot)) * kLn2 : -INFINITY;
    } else {
        const int64_t prow = static_cast<int64_t>(w) * rows_total + row;
        const float f = m_true == -INFINITY ? 0.0f : exp2f(m_ref - m_true);
        a.part_m[prow] = m_true * kLn2;
        a.part_s[prow] = l_tot * f;
    }
}

template <int KIND, bool kProt, int kR>
bool launch_rows(const DecodeArgs& a, hipStream_t stream, const LaunchEvents& ev) {
    const dim3 grid(static_cast<unsigned>(decode_workgroups(a.num_work, static_cast<int64_t>(a.s_q) * a.H, kR)));
    switch (a.shape.waves) {
        case 4: dispatch_decode(narrow_kernel<KIND, kProt, kR, 4>, grid, dim3(256), stream, ev, a); return true;
        case 2: dispatch_decode(narrow_kernel<KIND, kProt, kR, 2>, grid, dim3(128), stream, ev, a); return true;
        case 1: dispatch_decode(narrow_kernel<KIND, kProt, kR, 1>, grid, dim3(64), stream, ev, a); return true;
        default: return false;
    }
}

template <int KIND, bool kProt>
bool launch_kind(const DecodeArgs& a, hipStream_t stream, const LaunchEvents& ev) {
    switch (a.shape.rows) {
        case 16: return launch_rows<KIND, kProt, 16>(a, stream, ev);
        case 32: return launch_rows<KIND, kProt, 32>(a, stream, ev);
        default: return false;
    }
}

template <bool kProt>
hipError_t launch(CacheKind kind, const DecodeArgs& a, hipStream_t stream) {
    if (a.num_work == 0) return hipSuccess;
    const LaunchEvents ev = take_launch_events();
    static_assert(kNarrowThreads == kWaveThreads && kNarrowRowsPerBlock == 16, "the host checks the largest launch");
    bool ok = false;
    switch (kind) {
        case KIND_C4R4: ok = launch_kind<KIND_C4R4, kProt>(a, stream, ev); break;
        case KIND_C2R4: ok = launch_kind<KIND_C2R4, kProt>(a, stream, ev); break;
        case KIND_C4R4P: ok = launch_kind<KIND_C4R4P, kProt>(a, stream, ev); break;
        case KIND_C2R4P: ok = launch_kind<KIND_C2R4P, kProt>(a, stream, ev); break;
        case KIND_BF16:
            if constexpr (!kProt) ok = launch_kind<KIND_BF16, false>(a, stream, ev);
            break;
    }
    return ok ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_decode_narrow(CacheKind kind, const DecodeArgs& a, hipStream_t stream) {
    return launch<false>(kind, a, stream);
}

hipError_t launch_decode_narrow_protected(CacheKind kind, const DecodeArgs& a, hipStream_t stream) {
    return launch<true>(kind, a, stream);
}

}  // namespace mla
