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
// step as a sequence of bipartite matchings between the 32 labels and the 32 banks (over the slots not used
// yet): a few rounds of proposals match most labels, augmenting paths (breadth-first, one per bank still
// free) complete the matching, and the labels that cannot be matched -- their banks are all taken -- double
// up on the least loaded bank they can reach.  One half-wavefront works on one group: lane i is label i and
// also bank i, all state is in registers and moves by ballots and shuffles; only a label's own bank list and
// the proposal slots live in LDS.  The result is a deterministic function of idx.  Any outcome is a valid
// permutation: it changes speed, never results.  (A local search on the sum of squared bank counts, used
// before, spread the unavoidable collisions over all steps: 2.0 cycles per step against 1.5 now.)
#include <stdlib.h>

#include "usl_internal.h"

namespace {

constexpr int SCHED_NT = 256;

// K = padded fan-in, GS = labels and banks of a group (32, or 16 where a read is 16 bytes wide); k real slots.
template <int K, int GS>
__global__ void __launch_bounds__(SCHED_NT)
k_schedule(const int32_t* __restrict__ idx, int64_t m, int k, int shift, int rounds, uint8_t* __restrict__ perm) {
    constexpr int G = SCHED_NT / GS;
    constexpr uint32_t ALL = GS == 32 ? 0xFFFFFFFFu : (1u << (GS & 31)) - 1u;
    // per label (rows padded by 4 bytes: lanes of a group then hit different LDS banks)
    __shared__ uint8_t slots[G][GS][K + 4];   // first the bank of every slot, then my slots sorted by bank
    __shared__ __align__(16) uint8_t ord[G][GS][K + 4];     // slot read at step s
    __shared__ uint8_t left_in[G][GS][GS + 4];    // unused slots of mine per bank
    __shared__ uint8_t end_of[G][GS][GS + 4];     // where bank b's slots end in the sorted list
    __shared__ int deg0[G][GS];
    __shared__ int win[G][GS];
    const int gl = threadIdx.x / GS, lane = threadIdx.x & (GS - 1);
    const int hs = threadIdx.x & 63 & ~(GS - 1);        // where my group's bits sit in a wavefront ballot
    const int64_t j = (int64_t)blockIdx.x * SCHED_NT + (threadIdx.x & ~31) + usl_lane_of_position<GS>(threadIdx.x & 31);
    const bool valid = j < m;
    deg0[gl][lane] = 0;
    for (int b = 0; b < GS; ++b) left_in[gl][lane][b] = 0;
    __syncthreads();
    uint8_t* mine = slots[gl][lane];
    uint8_t* cnt = left_in[gl][lane];
    uint8_t* ends = end_of[gl][lane];
    for (int t = 0; t < k; ++t) {
        const int b = valid ? ((idx[j * k + t] >> shift) & (GS - 1)) : ((lane + t) & (GS - 1));
        mine[t] = (uint8_t)b;
        ++cnt[b];
        atomicAdd(&deg0[gl][b], 1);
    }
    uint32_t avail = 0;           // banks my unused slots read
    {   // counting sort of my slots by bank, in place through ord (free until the first step)
        int run = 0;
        for (int b = 0; b < GS; ++b) { run += cnt[b]; ends[b] = (uint8_t)run; if (cnt[b]) avail |= 1u << b; }
        uint8_t* tmp = ord[gl][lane];
        for (int t = 0; t < k; ++t) tmp[t] = mine[t];
        for (int t = k - 1; t >= 0; --t) { const int b = tmp[t]; ends[b] = (uint8_t)(ends[b] - 1); mine[ends[b]] = (uint8_t)t; }
        for (int b = 0; b < GS; ++b) ends[b] = (uint8_t)(ends[b] + cnt[b]);   // back from starts to ends
    }
    __syncthreads();
    auto gballot = [&](bool p) -> uint32_t { return (uint32_t)(__ballot(p) >> hs) & ALL; };
    volatile int* gwin = win[gl];
    // bank role
    int mydeg = deg0[gl][lane];   // slots of the group that read bank `lane` and are not used yet
    for (int s = 0; s < k; ++s) {
        int mb = -1;              // label role: my bank at this step
        int ml = -1;              // bank role: the label that reads me at this step
        for (int r = 0; r < rounds; ++r) {
            const uint32_t freeb = gballot(ml < 0);
            gwin[lane] = 255;
            int prop = -1;
            const uint32_t cand = mb < 0 ? (avail & freeb) : 0u;
            if (cand) {           // first candidate bank at or after a lane- and round-dependent start
                const int sh = (lane + 7 * r) & (GS - 1);
                const uint32_t rc = ((cand >> sh) | (cand << ((GS - sh) & (GS - 1)))) & ALL;
                prop = (__ffs(rc) - 1 + sh) & (GS - 1);
                atomicMin(&win[gl][prop], lane);
            }
            const int w = gwin[lane];
            if (ml < 0 && w < GS) ml = w;
            if (prop >= 0 && gwin[prop] == lane) mb = prop;
        }
        // augmenting paths from the banks still free
        uint32_t todo = gballot(ml < 0 && mydeg > 0);
        while (__any(todo != 0)) {
            const bool act = todo != 0;
            const int b0 = act ? __ffs(todo) - 1 : 0;
            todo &= todo - 1;
            uint32_t front = act ? (1u << b0) : 0u, seen = 0;
            int par = -1, found = -1;
            bool searching = act;
            while (__any(searching)) {
                const bool reach = searching && !((seen >> lane) & 1u) && (avail & front) != 0;
                if (reach) par = __ffs(avail & front) - 1;
                const uint32_t fresh = gballot(reach);
                const uint32_t fresh_free = gballot(reach && mb < 0);
                const uint32_t next = gballot(ml >= 0 && ((fresh >> (ml & (GS - 1))) & 1u));
                seen |= fresh;
                if (searching) {
                    if (fresh_free) { found = __ffs(fresh_free) - 1; searching = false; }
                    else if (next == 0) searching = false;
                    else front = next;
                }
            }
            int cur = found;      // walk back: every label on the path takes the bank it was reached through
            while (__any(cur >= 0)) {
                const bool a = cur >= 0;
                const int cl = a ? cur : 0;
                const int b = __shfl(par, cl, GS) & (GS - 1);
                const int prev = __shfl(ml, b, GS);
                if (a) {
                    if (lane == cl) mb = b;
                    if (lane == b) ml = cl;
                    cur = b == b0 ? -1 : prev;
                }
            }
        }
        // labels without a bank of their own double up: least loaded reachable bank, then the fullest
        int myload = ml >= 0 ? 1 : 0;
        uint32_t left = gballot(mb < 0);
        while (__any(left != 0)) {
            const bool a = left != 0;
            const int l = a ? __ffs(left) - 1 : 0;
            left &= left - 1;
            const uint32_t av = (uint32_t)__shfl((int)avail, l, GS);
            int key = (a && ((av >> lane) & 1u)) ? (((255 - myload) << 17) | (mydeg << 5) | lane) : -1;
#pragma unroll
            for (int o = GS / 2; o > 0; o >>= 1) key = max(key, __shfl_xor(key, o, GS));
            if (a && key >= 0) {
                const int bb = key & (GS - 1);
                if (lane == l) mb = bb;
                if (lane == bb) ++myload;
            }
        }
        // my next unused slot in that bank (slots of a bank are used in rising slot number)
        const int pick = mine[ends[mb] - cnt[mb]];
        if (--cnt[mb] == 0) avail &= ~(1u << mb);
        ord[gl][lane][s] = (uint8_t)pick;
        mydeg -= myload;
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
    int rounds = 3;
    if (const char* e = getenv("USL_TUNE_ROUNDS")) rounds = atoi(e);   // 0 = slots in stored order
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
