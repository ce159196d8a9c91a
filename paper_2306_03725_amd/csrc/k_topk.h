// Device code that the kernels of a prediction share: a (score, label) pair as one key, the largest key of a wavefront.
#pragma once
#include "usl_internal.h"

constexpr int TOPK_SHORT_MERGE = 8 * 256;   // candidates that a merge of 256 lanes holds in registers; more take it 1024
constexpr int TOPK_SHORT_SEGMENT = 8 * 256;  // scores of a workgroup of the pass over them where rows are few

// The upper word ranks scores (-0 as +0), the lower one equal scores by label (below 2^31, so ~label's top bit says nothing); its last bit says
// that the score is not -0, so that a key holds the score's own bits and no kernel that merges keys waits for the scores themselves.
__device__ __forceinline__ uint64_t score_key(float z, uint32_t label) {
    uint32_t u = __float_as_uint(z);
    const uint32_t minus_zero = u == 0x80000000u;
    if (minus_zero) u = 0u;
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((uint64_t)u << 32) | (uint64_t)(uint32_t)(~label << 1 | (minus_zero ^ 1u));
}
__device__ __forceinline__ int32_t key_label(uint64_t key) { return (int32_t)~((uint32_t)key >> 1 | 0x80000000u); }
__device__ __forceinline__ float key_score(uint64_t key) {
    const uint32_t u = (uint32_t)(key >> 32), bits = (u & 0x80000000u) ? u ^ 0x80000000u : ~u;
    return __uint_as_float(bits == 0u && !(key & 1u) ? 0x80000000u : bits);
}

// Largest v of the wavefront, the same register for all lanes: the upper words, then the lower ones of those that have the largest.
// What bounds these kernels is the chain of 2 kk such maxima; lane shifts within the vector unit (rows of 16 lanes, then the last lane
// of a row into the next ones) do not wait for LDS as shuffles do, and a 32-bit maximum takes its shifted operand in the same instruction,
// where 64-bit keys take five (one row of 500k scores, 5 labels: segments 6.7 and 6.2 us, merge 4.0 and 3.8; usl_predict of 4 instances at m = 300k, d = 8k, k = 16 29.4 and 24.3).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t max_with(uint32_t v) {   // a lane without a source keeps its own
    const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
    return t > v ? t : v;
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    v = max_with<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8: lane 15 of a row has the row's largest
    v = max_with<0x112, 0xF>(v);
    v = max_with<0x114, 0xF>(v);
    v = max_with<0x118, 0xF>(v);
    v = max_with<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
    v = max_with<0x143, 0xC>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint64_t wave_max(uint64_t v) {
    const uint32_t hi = wave_max((uint32_t)(v >> 32)), lo = wave_max((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
    return (uint64_t)hi << 32 | lo;
}
