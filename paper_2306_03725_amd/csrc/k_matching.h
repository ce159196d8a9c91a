// One step of a bank-aware slot order: a matching between the GS lists (lane i holds list i) and the GS banks of a group
// (lane i is also bank i).  Used by the slot order of the products and by the register lists of the backward product; a
// group is GS neighbouring lanes, all groups of a wavefront go through the same code side by side.
//
// What bounds it is latency: a step is a chain of a few dozen LDS accesses and ballots, and a small layer has no more
// wavefronts than compute units.  Hence no loop over single lists or banks: every list acts at once in rounds, a round
// being one write and one read of LDS.  A proposal round lets every list without a bank write its number to a bank that
// is free and that it has a slot for; the number that stays there has the bank.  A move round lets lists that have a
// bank that a list without one could use move on to a free one, so that the next proposal round finds theirs free: an
// augmenting path of length three, for all lists at once.  Exact augmenting paths, one bank at a time, and doubling up on
// the exactly fullest bank took 360 us for the slots of m = 500k, k = 32 (then 225) and 200 for m = 200k (then 125), for
// gathers that were 2 % faster.
#pragma once
#include "usl_internal.h"

template <int GS>
struct usl_matching {
    static constexpr uint32_t ALL = GS == 32 ? 0xFFFFFFFFu : (1u << (GS & 31)) - 1u;
    typedef volatile __attribute__((address_space(3))) uint32_t lds_word;   // (a generic pointer would mean flat accesses)
    lds_word* win;            // GS words of LDS
    uint32_t tag;             // of the current round: a word with another tag is of an earlier one
    int lane, shift;          // lane of the group; where the group's bits sit in a ballot
    int mb, ml;               // list role: my bank in this step, bank role: the list that reads me (-1: none)

    __device__ __forceinline__ usl_matching(uint32_t* words, int lane_) : win((lds_word*)words), tag(64), lane(lane_), shift((int)(threadIdx.x & 63) & ~(GS - 1)) {
        win[lane] = 0;
    }
    __device__ __forceinline__ uint32_t ballot(bool p) const { return (uint32_t)(__ballot(p) >> shift) & ALL; }
    // OR over the group
    static __device__ __forceinline__ uint32_t any_of(uint32_t v) {
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);   // rotations within 16 lanes
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, false);
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, false);
        if (GS == 32) v |= (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);          // the other 16 of 32
        return v;
    }
    // every list with cand != 0 asks for one of these banks; returns the bank if it got it, else -1; asked: the list that
    // got bank `lane`, else -1
    __device__ __forceinline__ int ask(uint32_t cand, int turn, int* asked) {
        const int sh = (lane + 7 * turn) & (GS - 1);   // first candidate at or after a start of the list's and round's own
        const uint32_t rc = ((cand >> sh) | (cand << ((GS - sh) & (GS - 1)))) & ALL;
        const int bank = (__ffs((int)rc) - 1 + sh) & (GS - 1);
        tag += 64;
        if (cand) win[bank] = tag | (uint32_t)lane;
        const uint32_t got = win[bank], mine = win[lane];
        *asked = (mine & ~63u) == tag ? (int)(mine & 63u) : -1;
        return cand && got == (tag | (uint32_t)lane) ? bank : -1;
    }
    __device__ __forceinline__ void propose(uint32_t avail, int turn) {
        const uint32_t freeb = ballot(ml < 0);
        int asked;
        const int got = ask(mb < 0 ? avail & freeb : 0u, turn, &asked);
        if (got >= 0) mb = got;
        if (asked >= 0) ml = asked;
    }
    // the matching of one step; avail: banks that my slots not used yet read
    __device__ __forceinline__ void run(uint32_t avail, int rounds) {
        mb = ml = -1;
        for (int r = 0; r < rounds; ++r) propose(avail, r);
        for (int r = 0; r < 4; ++r) {
            const bool lacks = mb < 0 && avail != 0;
            if (!__any(lacks)) break;
            const uint32_t wanted = any_of(lacks ? avail : 0u), freeb = ballot(ml < 0);
            const uint32_t cand = mb >= 0 && ((wanted >> mb) & 1u) ? avail & freeb : 0u;
            if (!__any(cand != 0)) break;
            int asked;
            const int got = ask(cand, r, &asked);
            const uint32_t moved = ballot(got >= 0);
            if (ml >= 0 && ((moved >> ml) & 1u)) ml = -1;
            if (asked >= 0) ml = asked;
            if (got >= 0) mb = got;
            propose(avail, r + 1);
        }
    }
    // Lists that found none (left) double up, on banks that two lists do not read yet if they can; preferred: banks that many
    // more slots are left of (degree) than steps, which have to be doubled up some time.  Returns the bank.
    __device__ __forceinline__ int double_up(uint32_t avail, bool left, const int* degree, int steps_left) {
        if (!__any(left)) return mb;
        const int over = degree[lane] - steps_left;
        const uint32_t full = ballot(over > 0), fuller = ballot(over > 2), fullest = ballot(over > 6);
        uint32_t twice = 0;   // banks that two lists read
        for (int r = 0; r < 3; ++r) {
            if (!__any(left && mb < 0)) break;
            uint32_t cand = left && mb < 0 ? avail & ~twice : 0u;
            if (cand & fullest) cand &= fullest;
            else if (cand & fuller) cand &= fuller;
            else if (cand & full) cand &= full;
            int asked;
            const int got = ask(cand, r, &asked);
            twice |= ballot(asked >= 0);
            if (got >= 0) mb = got;
        }
        return mb >= 0 || !left ? mb : __ffs((int)avail) - 1;
    }
};

// A list's entries sorted by bank, one list per lane: N entries at most (128), everything in the lane's own bytes of LDS.  Where
// the banks' entries end are bytes, four to a word: updates are atomics on words that nobody waits for (a chain of reads
// and writes of single bytes took most of the time of these kernels), and the running sums of four bytes are one product.
// The entries of a bank are taken from the end; the first one carries a mark (FIRST), so there is no count beside the end: a
// fifth workgroup fits a compute unit (m = 500k, d = 32k, k = 32: slots of the labels 213 and 187 us, register lists 285 and 266).
template <int GS, int N>
struct usl_bank_lists {
    static constexpr int Q = GS / 4;
    static constexpr uint32_t FIRST = 0x80u;
    static constexpr int WORDS = Q + (N + 3) / 4;
    struct Lane {              // an odd number of words: neighbours' are in different LDS banks
        uint32_t end[Q];       // where bank b's entries end in `sorted`
        uint8_t sorted[(N + 3) / 4 * 4 + (WORDS % 2 ? 0 : 4)];
    };
    // bank[p] (bytes of LDS too) for p < n; returns the banks that occur.  degree: counts of the group.
    template <typename BANK>
    static __device__ __forceinline__ uint32_t build(Lane& me, uint8_t* bank, int n, int* degree, BANK bank_of) {
#pragma unroll
        for (int q = 0; q < Q; ++q) me.end[q] = 0u;
#pragma unroll 4
        for (int p = 0; p < n; ++p) {
            const int b = bank_of(p), sh = 8 * (b & 3);
            const uint32_t old = atomicAdd(&me.end[b >> 2], 1u << sh);
            bank[p] = (uint8_t)((uint32_t)b | (((old >> sh) & 0xFFu) ? 0u : FIRST));
            atomicAdd(&degree[b], 1);
        }
        uint32_t avail = 0, run = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t w = me.end[q], ends = (w + run) * 0x01010101u;   // run: in the lowest byte
            run = ends >> 24;
            me.end[q] = ends - w;   // where they begin: moves to the end as they are filled in
#pragma unroll
            for (int u = 0; u < 4; ++u) avail |= ((w >> (8 * u)) & 0xFFu) ? 1u << (4 * q + u) : 0u;
        }
#pragma unroll 4
        for (int p = 0; p < n; ++p) {
            const uint32_t b = bank[p], sh = 8 * (b & 3u);
            const uint32_t old = atomicAdd(&me.end[(b & ~FIRST) >> 2], 1u << sh);
            me.sorted[(old >> sh) & 0xFFu] = (uint8_t)((uint32_t)p | (b & FIRST));
        }
        return avail;
    }
    // takes an entry of a bank that has one left
    static __device__ __forceinline__ int take(Lane& me, int b, uint32_t& avail) {
        uint8_t& end = reinterpret_cast<uint8_t*>(me.end)[b];
        const int at = end - 1;
        const uint32_t e = me.sorted[at];
        end = (uint8_t)at;
        if (e & FIRST) avail &= ~(1u << b);
        return (int)(e & ~FIRST);
    }
};
