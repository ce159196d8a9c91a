// Bank-aware slot order for the LDS gathers of forward / backward-weight.
//
// In those kernels the lanes of a wavefront own consecutive labels and, at step s, all read slot
// order[s] of their own label from the activation row in LDS: one unit of 4, 8 or 16 bytes, from bank
// column mod 32 of 32 (of twice the width where units are 8 bytes), or column mod 16 of 16 (16 bytes).
// With the slots in their natural order the addresses of a pass are random and collide (a step then
// costs as many cycles as the fullest bank, 3.5 on average for 32 labels and 32 banks).  The sum over a label's slots may be taken in
// any order, so each label gets a private permutation of its slots, chosen so that the lanes of a
// half-wavefront hit different banks at the same step as far as possible.
//
// A step costs as many LDS cycles as its fullest bank holds lanes, so what counts is the number of steps with
// a collision, not the number of collisions: banks that the group's 32*k slots over-subscribe must collide
// somewhere, and the aim is to gather those collisions in few steps.  The order is therefore built step by
// step as a sequence of bipartite matchings between the 32 labels and the 32 banks over the slots not used yet
// (k_matching.h); the labels that cannot be matched -- their banks are all taken -- double up.  One half-wavefront
// works on one group: lane i is label i and also bank i.  Any outcome is a valid permutation: it changes speed, never
// results.  (A local search on the sum of squared bank counts, used before, spread the unavoidable collisions over all
// steps: 2.0 cycles per step against 1.5 now.)
#include <stdlib.h>

#include "k_matching.h"

namespace {

constexpr int SCHED_NT = 256;

// K = padded fan-in, GS = labels and banks of a group (32, or 16 where a read is 16 bytes wide); k real slots.
template <int K, int GS>
__global__ void __launch_bounds__(SCHED_NT)
k_schedule(const int32_t* __restrict__ idx, int64_t m, int k, int shift, int rounds, uint8_t* __restrict__ perm) {
    constexpr int G = SCHED_NT / GS;
    typedef usl_bank_lists<GS, K> Lists;
    __shared__ typename Lists::Lane lists[G][GS];
    __shared__ __align__(16) uint8_t ord[G][GS][K + 4];     // first the bank of every slot, then the slot read at step s
    __shared__ int deg0[G][GS];                             // slots of the group that read a bank and are not used yet
    __shared__ uint32_t win[G][GS];
    const int gl = threadIdx.x / GS, lane = threadIdx.x & (GS - 1);
    const int label = usl_order_label<GS>((int)threadIdx.x);   // of the workgroup's
    const int64_t j0 = (int64_t)blockIdx.x * SCHED_NT, j = j0 + label;
    const bool valid = j < m;
    deg0[gl][lane] = 0;
    // The banks of all the workgroup's slots, in the order of memory (a lane reading its own row of idx fetched every line several
    // times: 651 MB instead of 64 at m = 500k, k = 32), each into the row of the lane that has its label: behind the barrier a
    // lane reads and writes its own row only, whatever the order in which the lanes of a wavefront run.
    uint8_t(*row)[K + 4] = &ord[0][0];
    const uint32_t n = (uint32_t)(min((int64_t)SCHED_NT, m - j0) * k), inv = k > 1 ? 0xFFFFFFFFu / (uint32_t)k + 1u : 0u;   // exact: n < 2^15
    // Loads of a lane in flight: with 8 and a check behind every one a small layer waited longer than for its own rows (m = 61k, d = 63k,
    // k = 32, b = 29, slots and forward: 132 us, now 127; k = 64, m = 670k: 1085 and 1010); 32 take a workgroup off the compute unit
    // (m = 200k, d = 8k, k = 32, b = 64: 187 and 143).
    constexpr int AT_ONCE = K % 16 == 0 ? 16 : 8;
#pragma unroll 1
    for (uint32_t q0 = threadIdx.x; q0 < n; q0 += AT_ONCE * SCHED_NT) {
        int32_t col[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) col[u] = idx[j0 * k + min(q0 + u * SCHED_NT, n - 1)];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            const uint32_t q = q0 + u * SCHED_NT, r = k > 1 ? __umulhi(q, inv) : q;   // label of the workgroup's
            if (q < n) row[usl_order_row<GS>((int)r)][q - r * (uint32_t)k] = (uint8_t)((col[u] >> shift) & (GS - 1));
        }
    }
    __syncthreads();
    uint32_t avail = Lists::build(lists[gl][lane], ord[gl][lane], k, deg0[gl],
                                  [&](int t) { return valid ? (int)ord[gl][lane][t] : ((lane + t) & (GS - 1)); });
    __syncthreads();
    usl_matching<GS> match(win[gl], lane);
    for (int s = 0; s < k; ++s) {
        match.run(avail, rounds);
        const int mb = match.double_up(avail, match.mb < 0, deg0[gl], k - s);
        ord[gl][lane][s] = (uint8_t)Lists::take(lists[gl][lane], mb, avail);
        atomicSub(&deg0[gl][mb], 1);
    }
    if (valid) {   // steps past k: the padding slots
        for (int s = k; s < K; ++s) ord[gl][lane][s] = (uint8_t)s;
        const uint32_t* from = reinterpret_cast<const uint32_t*>(ord[gl][lane]);
        uint32_t* to = reinterpret_cast<uint32_t*>(perm + j * K);
#pragma unroll
        for (int q = 0; q < K / 4; ++q) to[q] = from[q];
    }
}

// slots in stored order (tuning aid: what the gathers cost without a bank-aware order)
__global__ void k_identity_order(int64_t n, int K, uint8_t* __restrict__ perm) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        perm[e] = (uint8_t)(e % K);
}

}  // namespace

// Fills ctx->slot_order for the connectivity in idx.
usl_status usl_build_slot_order(usl_ctx* c, const int32_t* idx, int K, int unit) {
    USL_TRY(usl_reserve(c, (void**)&c->slot_order, &c->slot_order_cap, (size_t)c->m * K));
    const int shift = unit == 2 ? 1 : 0;  // two single bfloat16 columns share a bank word
    // A layer whose step is k_step_small's gathers too little for an order to pay: over 22 such layers of m * k * max_b >= 2^21 forward and weight gradient
    // take as long with it as without, and a forward on new connectivity 10 to 14 us instead of 26 to 79.  (And the scores have the step's bits.)
    const int rounds = usl_step_small_applies(c) && !getenv("USL_TUNE_ROUNDS") ? 0 : usl_order_rounds(c);
    const unsigned grid = (unsigned)((c->m + SCHED_NT - 1) / SCHED_NT);
    if (rounds <= 0) {
        hipLaunchKernelGGL(k_identity_order, dim3(c->num_cu * 4), dim3(256), 0, c->stream, c->m * K, K, c->slot_order);
    } else {
#define USL_SCHED(KK)                                                                                                          \
    case KK:                                                                                                                   \
        if (unit == 16)                                                                                                        \
            hipLaunchKernelGGL((k_schedule<KK, 16>), dim3(grid), dim3(SCHED_NT), 0, c->stream, idx, c->m, c->k, shift, rounds, c->slot_order); \
        else                                                                                                                   \
            hipLaunchKernelGGL((k_schedule<KK, 32>), dim3(grid), dim3(SCHED_NT), 0, c->stream, idx, c->m, c->k, shift, rounds, c->slot_order); \
        break
        switch (K) {
            USL_SCHED(8);
            USL_SCHED(16);
            USL_SCHED(24);
            USL_SCHED(32);
            USL_SCHED(48);
            USL_SCHED(64);
            default: USL_FAIL(c, USL_EUNSUPPORTED, "no slot order for a padded fan-in of %d", K);
        }
#undef USL_SCHED
    }
    USL_TRY(usl_check_launch(c, "slot order"));
    c->slot_order_for = idx;
    return USL_OK;
}
