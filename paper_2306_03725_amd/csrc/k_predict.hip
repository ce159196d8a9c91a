// Prediction (Section 2): the kk highest-scoring labels of every instance, and the hit counts that
// precision-at-k is made of.
//
// A (score, label) pair is packed into one 64-bit key whose unsigned order is the ranking: the upper
// word is the score's bit pattern made monotone (negative values complemented, the sign bit set on the
// rest; -0 folded onto +0 first), the lower word is ~label (and whether the score is -0, below it), so equal scores rank
// the smaller label higher and no two keys of a row are equal.  Key 0 never occurs for a real pair and means "nothing".
#include "k_topk.h"

namespace {

constexpr int TK_NT = 256;             // lanes per workgroup
// scores a lane holds in registers: 64, or 8 where that would leave most of the chip without a workgroup
constexpr int TK_EPT = 64, TK_EPT_FEW = 8;
static_assert(TK_NT * TK_EPT_FEW == TOPK_SHORT_SEGMENT, "what the choice of a prediction's path counts with");
constexpr int TK_MAX = 32;             // largest kk

// Largest v of the workgroup, returned to every lane.  red: two sets used in turn, so one barrier is enough.
template <int NT>
struct BlockMax {
    uint64_t (*red)[NT / 64];
    int turn;
    __device__ __forceinline__ uint64_t operator()(uint64_t v) {
        v = wave_max(v);
        uint64_t* set = red[turn];
        turn ^= 1;
        if ((threadIdx.x & 63) == 0) set[threadIdx.x >> 6] = v;
        __syncthreads();
        uint64_t r = set[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) r = set[w] > r ? set[w] : r;
        return r;
    }
};

// The kk best keys of one segment of 256 * TK_EPT labels of one row, best first, into cand[row][segment][kk]
// (0 where the segment has fewer than kk labels).
//   1. every lane loads its TK_EPT scores (all loads in flight at once) and finds its own best key;
//   2. tau = the kk-th best of the 256 lane maxima: at least kk keys of the segment are >= tau, and
//      every key >= tau belongs to one of the kk lanes whose maximum is >= tau, so at most kk*TK_EPT keys pass;
//   3. those keys are collected in LDS and the best kk are peeled off one by one ("largest key below the
//      previous winner": keys are distinct, so nothing has to be removed).
// VEC: rows are 16-byte aligned and m % 4 == 0, so a lane reads groups of 4 consecutive labels.
template <bool VEC, int TK_EPT>
__global__ void __launch_bounds__(TK_NT)
k_topk_segments(const float* __restrict__ out, int64_t m, int kk, int nseg, uint64_t* __restrict__ cand) {
    __shared__ uint64_t red[2][TK_NT / 64];
    BlockMax<TK_NT> block_max = {red, 0};
    __shared__ uint64_t list[TK_MAX * TK_EPT];
    __shared__ uint32_t count;
    constexpr int TK_SEG = TK_NT * TK_EPT;   // labels per workgroup
    const int64_t seg0 = (int64_t)blockIdx.x * TK_SEG;
    const float* row = out + (int64_t)blockIdx.y * m + seg0;
    const int lim = (int)min((int64_t)TK_SEG, m - seg0);   // labels of this segment that exist
    const int tid = (int)threadIdx.x;
    // label of register e of this lane, counted from the segment's first (32-bit arithmetic throughout)
    auto local_of = [&](int e) -> int {
        return VEC ? ((e >> 2) * TK_NT + tid) * 4 + (e & 3) : e * TK_NT + tid;
    };
    float v[TK_EPT];
    if (VEC) {
#pragma unroll
        for (int e = 0; e < TK_EPT; e += 4) {
            const int j = local_of(e);
            const float4 q = j < lim ? *reinterpret_cast<const float4*>(row + j) : make_float4(0.f, 0.f, 0.f, 0.f);
            v[e] = q.x; v[e + 1] = q.y; v[e + 2] = q.z; v[e + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < TK_EPT; ++e) {
            const int j = local_of(e);
            v[e] = j < lim ? row[j] : 0.f;
        }
    }
    // the lane's best score; labels grow with e, so the first of equal scores is the smaller label
    float top = 0.f;
    int top_j = -1;
#pragma unroll
    for (int e = 0; e < TK_EPT; ++e) {
        const int j = local_of(e);
        const bool better = j < lim && (top_j < 0 || v[e] > top);
        top = better ? v[e] : top;
        top_j = better ? j : top_j;
    }
    const uint64_t mine = top_j >= 0 ? score_key(top, (uint32_t)(seg0 + top_j)) : 0ull;
    uint64_t tau = ~0ull;
    for (int r = 0; r < kk && tau != 0; ++r) tau = block_max(mine < tau ? mine : 0ull);
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    // keys are built only for scores that reach tau's score (a cheap float test first)
    const uint32_t tu = (uint32_t)(tau >> 32);
    const float tau_score = tau == 0 ? -INFINITY : __uint_as_float((tu & 0x80000000u) ? (tu & 0x7FFFFFFFu) : ~tu);
#pragma unroll
    for (int e = 0; e < TK_EPT; ++e) {
        const int j = local_of(e);
        if (j < lim && v[e] >= tau_score) {
            const uint64_t key = score_key(v[e], (uint32_t)(seg0 + j));
            if (key >= tau) list[atomicAdd(&count, 1u)] = key;
        }
    }
    __syncthreads();
    const uint32_t n = count;
    uint64_t* dst = cand + ((size_t)blockIdx.y * nseg + blockIdx.x) * kk;
    uint64_t prev = ~0ull;
    for (int r = 0; r < kk; ++r) {
        uint64_t best = 0;
        for (uint32_t q = threadIdx.x; q < n; q += TK_NT) {
            const uint64_t key = list[q];
            if (key < prev && key > best) best = key;
        }
        prev = block_max(best);
        if (threadIdx.x == 0) dst[r] = prev;
    }
}

// One workgroup per row: the best kk of the row's nseg*kk candidate keys, unpacked.  A launch of its own: merged by the workgroup
// that finishes a row's last segment, behind fences, one row of 500k scores took 14.6 us when the two launches took 7.5 + 5.2.  (Without fences it
// pays for one instance: k_forward_few.)
template <int NT>
__global__ void __launch_bounds__(NT)
k_topk_merge(const uint64_t* __restrict__ cand, int n, int kk, int32_t* __restrict__ top_lab, float* __restrict__ top_val) {
    __shared__ uint64_t red[2][NT / 64];
    BlockMax<NT> block_max = {red, 0};
    const uint64_t* c = cand + (size_t)blockIdx.x * n;
    constexpr int HELD = 8;   // candidates a lane keeps in registers; only very wide rows have more
    uint64_t mine[HELD];
#pragma unroll
    for (int e = 0; e < HELD; ++e) mine[e] = e * NT + (int)threadIdx.x < n ? c[e * NT + threadIdx.x] : 0ull;
    uint64_t prev = ~0ull;
    for (int r = 0; r < kk; ++r) {
        uint64_t best = 0;
#pragma unroll
        for (int e = 0; e < HELD; ++e)
            if (mine[e] < prev && mine[e] > best) best = mine[e];
        for (int q = HELD * NT + (int)threadIdx.x; q < n; q += NT) {
            const uint64_t key = c[q];
            if (key < prev && key > best) best = key;
        }
        prev = block_max(best);
        if ((int)threadIdx.x == r) {
            top_lab[(size_t)blockIdx.x * kk + r] = key_label(prev);
            top_val[(size_t)blockIdx.x * kk + r] = key_score(prev);
        }
    }
}

__global__ void k_zero_hits(unsigned long long* hits, int kk) {
    if ((int)threadIdx.x < kk) hits[threadIdx.x] = 0ull;
}

// hits[r] += 1 for every instance whose rank-r prediction is one of its targets
__global__ void __launch_bounds__(256)
k_precision_hits(const int32_t* __restrict__ top_lab, const int64_t* __restrict__ tgt_off,
                 const int32_t* __restrict__ tgt_lab, int b, int kk, unsigned long long* __restrict__ hits) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= b * kk) return;
    const int i = q / kk, r = q % kk;
    const int32_t label = top_lab[q];
    bool hit = false;
    for (int64_t p = tgt_off[i]; p < tgt_off[i + 1]; ++p) hit |= tgt_lab[p] == label;
    if (hit) atomicAdd(&hits[r], 1ull);
}

}  // namespace

int usl_topk_max(void) { return TK_MAX; }

static int topk_segments(const usl_ctx* c, int ept) { return (int)((c->m + TK_NT * ept - 1) / (TK_NT * ept)); }

// Sized once for the largest batch and the largest kk, so that no later call has to grow it (growing waits for the stream).  Behind the candidates lies
// the word that counts finished workgroups of k_forward_few, in the same allocation and cleared by the same first call, whatever its batch and kk: a later
// call finds both.  A capture only records the clearing, and a plain call may come before the first replay: a context whose first calls are
// captured has no such word until a plain call (topk_done_clear), and its merges are launches of their own.
usl_status usl_reserve_topk(usl_ctx* c) {
    const size_t most = (size_t)topk_segments(c, TK_EPT) * c->max_b, most_few = (size_t)topk_segments(c, TK_EPT_FEW) * (c->num_cu / topk_segments(c, TK_EPT) + 1);
    const size_t by_forward = (size_t)usl_forward_few_blocks(c);
    const size_t two = most > most_few ? most : most_few;
    const size_t bytes = (two > by_forward ? two : by_forward) * TK_MAX * 8, had = c->topk_cand_cap;
    USL_TRY(usl_reserve(c, (void**)&c->topk_cand, &c->topk_cand_cap, bytes + 64));
    if (had != c->topk_cand_cap) c->topk_done_clear = false;
    c->topk_done = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(c->topk_cand) + bytes);
    if (c->topk_done_clear) return USL_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess) {   // (the null stream beside a capture elsewhere)
        (void)hipGetLastError();
        return USL_OK;
    }
    if (capture != hipStreamCaptureStatusNone) return USL_OK;
    hipLaunchKernelGGL(k_zero_hits, dim3(1), dim3(64), 0, c->stream, (unsigned long long*)c->topk_done, 8);
    USL_TRY(usl_check_launch(c, "counter of workgroups"));
    c->topk_done_clear = true;   // behind a launch that was taken
    return USL_OK;
}

// The best kk of every row from nseg sets of kk candidates each (usl_ctx::topk_cand).
usl_status usl_launch_topk_merge(usl_ctx* c, int nseg, int32_t b, int32_t kk, int32_t* top_lab, float* top_val) {
    const int n = nseg * kk;
    if (n <= TOPK_SHORT_MERGE)
        hipLaunchKernelGGL(k_topk_merge<TK_NT>, dim3((unsigned)b), dim3(TK_NT), 0, c->stream, c->topk_cand, n, (int)kk, top_lab, top_val);
    else
        hipLaunchKernelGGL(k_topk_merge<1024>, dim3((unsigned)b), dim3(1024), 0, c->stream, c->topk_cand, n, (int)kk, top_lab, top_val);
    return usl_check_launch(c, "topk");
}

usl_status usl_launch_topk(usl_ctx* c, const float* out, int32_t b, int32_t kk, int32_t* top_lab,
                           float* top_val) {
    // short segments where long ones would not give every compute unit a workgroup (one row of 500k scores: 31 of 256
    // busy, 11 us; 7.5 with short ones)
    const bool few = (int64_t)topk_segments(c, TK_EPT) * b < c->num_cu;
    const int nseg = topk_segments(c, few ? TK_EPT_FEW : TK_EPT);
    USL_TRY(usl_reserve_topk(c));
    const bool vec = c->m % 4 == 0 && (uintptr_t)out % 16 == 0;
#define USL_TOPK(VEC, EPT)                                                                                                   \
    hipLaunchKernelGGL((k_topk_segments<VEC, EPT>), dim3((unsigned)nseg, (unsigned)b), dim3(TK_NT), 0, c->stream, out, c->m, \
                       (int)kk, nseg, c->topk_cand)
    if (few) { if (vec) USL_TOPK(true, TK_EPT_FEW); else USL_TOPK(false, TK_EPT_FEW); }
    else { if (vec) USL_TOPK(true, TK_EPT); else USL_TOPK(false, TK_EPT); }
#undef USL_TOPK
    return usl_launch_topk_merge(c, nseg, b, kk, top_lab, top_val);
}

usl_status usl_launch_precision_hits(usl_ctx* c, const int32_t* top_lab, const int64_t* tgt_off,
                                     const int32_t* tgt_lab, int32_t b, int32_t kk, int64_t* hits) {
    hipLaunchKernelGGL(k_zero_hits, dim3(1), dim3(64), 0, c->stream, (unsigned long long*)hits, (int)kk);
    hipLaunchKernelGGL(k_precision_hits, dim3((unsigned)((b * kk + 255) / 256)), dim3(256), 0, c->stream,
                       top_lab, tgt_off, tgt_lab, (int)b, (int)kk, (unsigned long long*)hits);
    return usl_check_launch(c, "precision_hits");
}
