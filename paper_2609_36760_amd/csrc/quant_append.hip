// Quantize-and-append writer for the packed dual-path cache, and the plain
// BF16 append used by the unquantized comparison cache.  The quantizer, the
// code layout and the metadata storage are in writer_common.h (shared with the
// decode kernel's in-launch append); one group of 64 channels per 8 lanes.
//
// With BF16 protection (Sec. 3.3; Appendix C.5, "BF16 protection and cache
// lifecycle") the same lanes also store the bf16 values they loaded into the
// token's row of its sequence's protection buffer when the token is protected
// once the append is done: position p < sink (row p) or p >= L - recent
// (row sink + (p - sink) mod recent, a ring), L the sequence's new length.
// Tokens leaving the window keep the packed copy written here at insertion.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "writer_common.h"

namespace mla {
namespace {

using wc::kGroup;
using wc::kGroupsPerToken;
using wc::kLanesPerGroup;
constexpr int kThreads = 256;
static_assert(kGroupsPerToken * kLanesPerGroup == kAppendThreadsPerToken, "launch shape the host checks");

// A lane's piece of a token (8 channels of group g) and what decides where it
// goes, loaded before anything is tested (a skipped token's row is read for
// nothing), so that the memory round trips overlap: one for the row, its slot,
// sequence and position, and under protection a second one for the sequence's
// length and buffer.
struct Piece {
    uint4 raw;
    int64_t slot, ps;
    int bseq, p, L, g;
};

// kPer pieces per thread, half the launch apart: with one, a wave waits for its
// two round trips with 1 KiB in flight, and 32 waves per unit do not cover them.
template <int CBITS, bool kProt, bool kPaper, int kPer>
__global__ __launch_bounds__(kThreads) void lowbit_append_kernel(AppendArgs a) {
    // the launch's work items fit 32 bits (the host refuses more tokens)
    const int lig = static_cast<int>(threadIdx.x % kLanesPerGroup);
    const uint32_t gid0 = (blockIdx.x * kThreads + threadIdx.x) / kLanesPerGroup;   // shared by a group's 8 lanes
    const uint32_t step = gridDim.x * (kThreads / kLanesPerGroup);
    const uint32_t total = static_cast<uint32_t>(a.n) * kGroupsPerToken;
    Piece x[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t gid = gid0 + i * step;
        const uint32_t tok32 = min(gid, total - 1) / kGroupsPerToken;
        const int64_t token = tok32;
        x[i].g = static_cast<int>(min(gid, total - 1) - tok32 * kGroupsPerToken);
        const uint16_t* src = x[i].g == kGroupsPerToken - 1 ? a.k_rope + token * a.k_rope_stride + lig * 8
                                                             : a.c_kv + token * a.c_kv_stride + x[i].g * kGroup + lig * 8;
        x[i].raw = *reinterpret_cast<const uint4*>(src);
        x[i].slot = gid < total ? a.slot_mapping[token] : -1;
        if constexpr (kProt) {
            x[i].bseq = a.token_seq[token];
            x[i].p = a.positions[token];
        }
    }
    if constexpr (kProt) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int bs = min(max(x[i].bseq, 0), a.B - 1);      // B >= 1
            x[i].L = a.seq_lens[bs];
            x[i].ps = a.prot_slot[bs];
        }
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (x[i].slot < 0 || x[i].slot >= a.num_slots) continue;        // skipped token
        const bool rope = x[i].g == kGroupsPerToken - 1;
        if constexpr (kProt) {
            // p >= L - recent with p < L implies recent >= 1
            const int p = x[i].p, L = x[i].L;
            if (x[i].bseq >= 0 && x[i].bseq < a.B && p >= 0 && p < L && (p < a.sink || p >= L - a.recent) &&
                x[i].ps >= 0 && x[i].ps < a.num_prot) {
                const int prow = p < a.sink ? p : a.sink + (p - a.sink) % a.recent;
                uint8_t* dst = a.prot + (x[i].ps * (a.sink + a.recent) + prow) * 1152 +
                               (rope ? 1024 + lig * 16 : (x[i].g * kGroup + lig * 8) * 2);
                *reinterpret_cast<uint4*>(dst) = x[i].raw;
            }
        }
        const wc::SlotPos at = wc::split_slot(x[i].slot, a.num_slots, a.g);
        wc::quantize_store<CBITS, kPaper>(x[i].raw, rope, x[i].g, lig, a.cache + at.page * a.g.page_bytes, at.off, a.g);
    }
}

// BF16 comparison cache: row = [c_kv (512) | k_rope (64)] bf16; 72 lanes per
// token, 16 bytes each.
__global__ __launch_bounds__(kThreads) void bf16_append_kernel(AppendArgs a) {
    constexpr int kLanesPerToken = 72;     // 64 content + 8 RoPE pieces of 16 bytes
    static_assert(kLanesPerToken == kAppendThreadsPerToken, "launch shape the host checks");
    const uint32_t tid = blockIdx.x * kThreads + threadIdx.x;      // fits 32 bits, as above
    const uint32_t tok32 = tid / kLanesPerToken;
    const int lane = static_cast<int>(tid - tok32 * kLanesPerToken);
    if (tok32 >= static_cast<uint32_t>(a.n)) return;
    const int64_t token = tok32;
    const int64_t slot = a.slot_mapping[token];
    if (slot < 0 || slot >= a.num_slots) return;
    const uint16_t* src = lane < 64 ? a.c_kv + token * a.c_kv_stride + lane * 8
                                    : a.k_rope + token * a.k_rope_stride + (lane - 64) * 8;
    const wc::SlotPos at = wc::split_slot(slot, a.num_slots, a.g);
    uint8_t* dst = a.cache + at.page * a.g.page_bytes + at.off * 1152 + lane * 16;
    *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
}

}  // namespace

namespace {

template <bool kProt, int kPer>
hipError_t launch_append_per(const AppendArgs& a, hipStream_t stream) {
    const int64_t threads = (static_cast<int64_t>(a.n) * kGroupsPerToken * kLanesPerGroup + kPer - 1) / kPer;
    const dim3 grid(static_cast<unsigned>((threads + kThreads - 1) / kThreads));
    const bool paper = a.g.paper_meta != 0;
    if (a.g.c_bits == 4) {
        if (paper) hipLaunchKernelGGL((lowbit_append_kernel<4, kProt, true, kPer>), grid, dim3(kThreads), 0, stream, a);
        else hipLaunchKernelGGL((lowbit_append_kernel<4, kProt, false, kPer>), grid, dim3(kThreads), 0, stream, a);
    } else {
        if (paper) hipLaunchKernelGGL((lowbit_append_kernel<2, kProt, true, kPer>), grid, dim3(kThreads), 0, stream, a);
        else hipLaunchKernelGGL((lowbit_append_kernel<2, kProt, false, kPer>), grid, dim3(kThreads), 0, stream, a);
    }
    return hipGetLastError();
}

// Under protection a thread takes two pieces from this many tokens: its second
// round trip leaves one-piece waves waiting (65 536 tokens, INT4: 26.6 us against
// 29.9), while smaller launches need the threads (32 768: 15.6 against 15.0).
// Without protection one piece is the faster (65 536 tokens: 23.6 us against 25.3).
constexpr int kTwoPieces = 49152;
template <bool kProt>
hipError_t launch_append(const AppendArgs& a, hipStream_t stream) {
    if (a.n == 0) return hipSuccess;
    if constexpr (kProt) {
        if (a.n >= kTwoPieces) return launch_append_per<kProt, 2>(a, stream);
    }
    return launch_append_per<kProt, 1>(a, stream);
}

}  // namespace

hipError_t launch_lowbit_append(const AppendArgs& a, hipStream_t stream) { return launch_append<false>(a, stream); }

hipError_t launch_lowbit_append_protected(const AppendArgs& a, hipStream_t stream) {
    return launch_append<true>(a, stream);
}

hipError_t launch_bf16_append(const AppendArgs& a, hipStream_t stream) {
    if (a.n == 0) return hipSuccess;
    const int64_t threads = static_cast<int64_t>(a.n) * kAppendThreadsPerToken;
    const dim3 grid(static_cast<unsigned>((threads + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(bf16_append_kernel, grid, dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace mla
