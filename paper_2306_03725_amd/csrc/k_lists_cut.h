// How a layer is cut up for the kernels that keep the connections of a window of labels in registers
// (k_backward_input_lds.hip), and the turns of the workgroups that walk column lists (k_backward_input.hip).  Plain arithmetic on the layer's sizes: no GPU is needed to check it.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace usl_lists {

constexpr int WL = 32768;      // most labels a window has: one float32 row of 128 KiB in LDS.  A layer's windows are of equal
                               // size wl <= WL (a multiple of 4): no short last window whose workgroups idle
constexpr int NF = 2048;       // features per workgroup (two per lane)
constexpr int NT = 1024;
// most labels of a window whose rows LDS holds two at a time; four; four, and the activations in a place of their own
constexpr int BOTH2_LABELS = 15968, BOTH4_LABELS = 7232, BOTH4_OWN_LABELS = 4672;

// A workgroup owns a window of wl labels and a block of NF features.  Where the layer is narrower
// than a block, the window consists of S runs of `run` labels, and the features count S times over, once for every run
// ("virtual" features run * d + c, vd = S * d of them): the lists stay of the length that the registers are made for.
// The sums of the runs are added up on their way out of the workgroup.
// fpb: features of a block, a multiple of 32 (whole lines of x), at most NF.
// Every window has labels: (nwin - 1) * wl < m <= nwin * wl.
struct Cut {
    int run, S, wl, nwin, vd, nfb, fpb;
    __host__ __device__ __forceinline__ uint32_t vfeat(uint32_t col, uint32_t label_in_window, int d) const {
        return S == 1 ? col : col + label_in_window / (uint32_t)run * (uint32_t)d;
    }
};

// (window, feature block) workgroups run in rounds of one per compute unit: a last round that is not full takes as
// long as a full one, so the windows are made a little shorter until the rounds are full (up to a quarter more
// windows: more than that and the extra partial sums cost what the shorter lists save).
inline int64_t full_rounds(int64_t num_cu, int64_t nwin, int64_t nfb) {
    const int64_t cu = num_cu > 0 ? num_cu : 1;
    const int64_t rounds = (nwin * nfb + cu - 1) / cu, full = rounds * cu / nfb;
    return full > nwin && full * 4 <= nwin * 5 ? full : nwin;
}

// Windows of equal size for m labels, about nwin of them: rounding the size up to a multiple of 4 can leave fewer.
inline void equal_windows(Cut* cut, int64_t m, int64_t nwin) {
    const int64_t wl = ((m + nwin - 1) / nwin + 3) / 4 * 4;
    cut->run = cut->wl = (int)wl;
    cut->nwin = (int)((m + wl - 1) / wl);
}

// usl_backward_input's form: windows of as many labels as send about 32 connections into a feature (the registers of a
// lane hold two such lists), at most WL (the LDS row), a multiple of 4 (16-byte copies), all of equal size.
inline Cut bwi_cut(int64_t m, int d, int k, int num_cu) {
    const int64_t by_lists = (int64_t)32 * d / k, cap = (by_lists < WL ? by_lists : WL) / 4 * 4;
    Cut cut;
    cut.S = 1;
    cut.vd = d;
    cut.nfb = (d + NF - 1) / NF;
    cut.fpb = NF;
    equal_windows(&cut, m, full_rounds(num_cu, (m + cap - 1) / cap, cut.nfb));
    return cut;
}

// Do the activations of the block have a place of their own, beside that of the sums (a barrier less per pass)?  Where a row
// leaves room for it, and where runs share activations (the places of the sums are then other ones).
inline bool both_own(int Q, const Cut& cut) { return Q == 4 && (cut.wl <= BOTH4_OWN_LABELS || cut.S > 1); }

// Chains of windows: as many as the compute units have room for, where there are more windows than that.
inline int both_chains(const Cut& cut, int num_cu) {
    const int at_once = num_cu > cut.nfb ? num_cu / cut.nfb : 1;
    const int rounds = (cut.nwin + at_once - 1) / at_once;
    return (cut.nwin + rounds - 1) / rounds;
}

// ... and the rounds of workgroups that they go through, one after the other on a compute unit
inline int both_rounds(const Cut& cut, int num_cu) { const int chains = both_chains(cut, num_cu); return (cut.nwin + chains - 1) / chains; }

// The form for both products: lists of 16 connections (half the registers go to the weight-gradient sums; with four
// instances a lane has 32 slots instead of 36, hence 14), longer where the features do not fill the lanes twice over;
// blocks of equal size; S runs where the layer is narrower than half a block.
// Q: instances of a pass, 2 or 4 (both_q, below).
inline Cut both_cut(int64_t m, int d, int k, int num_cu, int Q) {
    auto cut_of = [&](int labels) {   // with windows of that many at most
        Cut cut;
        cut.S = d <= NT ? NF / d : 1;
        if (cut.S > labels / 4) cut.S = labels / 4;   // a run has at least four labels, and the window has to fit LDS (d = 1)
        cut.vd = cut.S * d;
        cut.nfb = (cut.vd + NF - 1) / NF;
        cut.fpb = ((cut.vd + cut.nfb - 1) / cut.nfb + 31) / 32 * 32;
        const int64_t mean = Q == 4 ? 14 : 16, longest = Q == 4 ? 21 : 24;
        const int64_t lists = mean * NF / cut.fpb < longest ? mean * NF / cut.fpb : longest;
        const int64_t most = labels / cut.S;
        int64_t run = lists * d / k;
        run = run < most ? run : most;
        run = run >= 4 ? run / 4 * 4 : 4;
        if (cut.S == 1) {
            equal_windows(&cut, m, full_rounds(num_cu, (m + run - 1) / run, cut.nfb));
        } else {
            cut.run = (int)run;
            cut.wl = cut.run * cut.S;
            cut.nwin = (int)((m + cut.wl - 1) / cut.wl);
        }
        return cut;
    };
    if (Q != 4) return cut_of(BOTH2_LABELS);
    const Cut own = cut_of(BOTH4_OWN_LABELS);
    if (d <= NT) return own;
    // Windows that leave the activations a place of their own, unless their lists would be short (fewer than 11 connections) or they
    // make more rounds than longer ones.  usl_backward with windows of up to 4672 and of up to 7232 labels: m = 154k, d = 2762, k = 8,
    // b = 64: 70 and 77 us; m = 6k, d = 3094, k = 8, b = 24: 29 and 33; m = 22k, d = 6747, k = 16, b = 64: 44 and 47; m = 41k, d = 13k,
    // k = 32, b = 400: 185 and 179; two rounds and one, m = 200k, d = 12k, k = 32, b = 64: 250 and 169.
    const Cut wide = cut_of(BOTH4_LABELS);
    return (int64_t)11 * d / k <= (int64_t)BOTH4_OWN_LABELS && both_rounds(own, num_cu) <= both_rounds(wide, num_cu) ? own : wide;
}

// Parts of the batch in the kernel for both products: more than one where the (window, feature block) workgroups leave
// compute units idle.  A workgroup loads its lists and weights and hands out its sums in about 20 us, a pass of its loop
// takes about 4.4 (m = 31k, d = 1k, k = 32, b = 128: 179 us with 1 part, 116 with 2, 83 with 4, 77 with 6, 103 with 8, which
// are two rounds); every part writes a weight gradient of its own, which the reader adds up.  Of 16 layers measured
// (profiles/rules_measured.txt) the best number or within 6 % of it.  forced > 0: that many, if the batch has them.
inline int both_parts(const Cut& cut, int64_t m, int k, int num_cu, int rows, int Q, int forced) {
    const int64_t wgs = (int64_t)cut.nwin * cut.nfb, passes = (rows + Q - 1) / Q, cu = num_cu;
    if (forced > 0) return (int)(forced < passes ? forced : passes);
    int best = 1;
    double best_t = 0.0;
    for (int P = 1; P <= 32 && P <= passes; ++P) {
        if ((size_t)P * m * k * 4 > ((size_t)1 << 28) && P > 1) break;
        const double rounds = (double)((wgs * P + cu - 1) / cu);
        const double t = rounds * (20.0 + 4.4 * (double)((passes + P - 1) / P)) + (double)P * m * k * 8 / 4e6;
        if (P == 1 || t < best_t) { best = P; best_t = t; }
    }
    return best;
}

// Instances that a pass of the kernel for both products takes together.  A pass is a chain of waits, so the fewer the better:
// four, where windows that send 11 connections into a feature leave four rows room in LDS beside the activations (usl_backward with
// four and two, float32: m = 200k, d = 12k, k = 32, b = 64: 171 and 187 us; m = 400k, d = 27k, k = 64, b = 64: 617 and 698); two, where even
// windows of 7232 labels send fewer than 14 (too many windows; m = 700k, d = 32k, k = 64, b = 256: 3312 and 2800).
// In between the rounds of workgroups decide, one after the other on a compute unit: four where there are more workgroups than compute
// units, in no more rounds than two and in five at most.  With six the chains' sums come from memory in every pass (m = 670k, d = 30k,
// k = 64, bfloat16, b = 512: 5419 us with two, 5985 with four).  m = 670k, d = 16k, k = 32, b = 32, three rounds each: 348 and
// 322; m = 300k, d = 24k, k = 48, b = 64, two and three rounds: 362 and 409; m = 130k, d = 15 360, k = 32, b = 128, less than one round of
// windows: 202 (in two parts of the batch that fit a round) and 225.
// The rule does not see the batch, which can decide it the other way: the six rounds above at b = 64 take 938 and 887, and
// m = 130k, d = 15 000, where two parts of the windows of two do not fit a round, 169 and 141 at b = 64.
inline int both_q(int64_t m, int d, int k, int num_cu) {
    if (d <= NT || (int64_t)11 * d / k <= (int64_t)BOTH4_OWN_LABELS) return 4;
    if ((int64_t)14 * d / k > (int64_t)BOTH4_LABELS) return 2;
    const Cut two = both_cut(m, d, k, num_cu, 2), four = both_cut(m, d, k, num_cu, 4);
    const int rounds = both_rounds(four, num_cu);
    return (int64_t)four.nwin * four.nfb > num_cu && rounds <= both_rounds(two, num_cu) && rounds <= 5 ? 4 : 2;
}

// How a batch of `rows` instances goes through: in passes of at most G, one part each, or at once in several parts.
// sets: sums of the input gradient that are kept beside each other.
struct BothPlan { int parts, sets; };
inline BothPlan both_plan(const Cut& cut, int64_t m, int k, int num_cu, int rows, int G, int Q, int forced) {
    BothPlan p;
    p.parts = rows <= G ? both_parts(cut, m, k, num_cu, rows, Q, forced) : 1;
    p.sets = p.parts > 1 ? cut.nwin : both_chains(cut, num_cu);
    return p;
}
// The most that any batch of up to max_b instances takes, of parts and of rows of input-gradient sums (sets times
// instances): neither grows with the batch (m = 13 330, d = 5000, k = 32: 12 parts at 96 instances, 11 at 128).
struct BothMost { int parts; size_t rows; };
inline BothMost both_most(const Cut& cut, int64_t m, int k, int num_cu, int max_b, int G, int Q, int forced) {
    BothMost most = {1, (size_t)both_chains(cut, num_cu) * (size_t)(G < max_b ? G : max_b)};
    for (int b = max_b < G ? max_b : G; b >= 1; b = (b - 1) / Q * Q) {   // the largest batch of every number of passes
        const BothPlan p = both_plan(cut, m, k, num_cu, b, G, Q, forced);
        if (p.parts > most.parts) most.parts = p.parts;
        if ((size_t)p.sets * (size_t)b > most.rows) most.rows = (size_t)p.sets * (size_t)b;
    }
    return most;
}

// The column lists' features lie chunk by chunk, each in the order of falling list length.  Their workgroups go through all
// chunks at once, so that those of the long lists start first and a launch ends with short ones: the pos-th workgroup of every
// chunk before the (pos + 1)-th of any (`whole` chunks of `per_chunk` workgroups, and one of `rest`).  Chunk after chunk, a
// launch ended on a chunk of which the long lists had just begun: usl_backward_input 223 us at m = 200k, d = 70k, k = 32, b = 32,
// now 199; m = 791k, d = 51k, k = 16, b = 14: 409 and 359; m = 100k, d = 16k, k = 64, b = 300: 727 and 694.
struct ChunkTurns {
    int per_chunk, whole, rest;
    // which workgroup of the features' order the turn-th one is
    __host__ __device__ __forceinline__ int operator()(int turn) const {
        const int all = rest * (whole + 1);
        if (turn < all) return turn % (whole + 1) * per_chunk + turn / (whole + 1);
        turn -= all;
        return turn % whole * per_chunk + rest + turn / whole;
    }
};
// d features in chunks of `chunk`, `per` of them to a workgroup (chunk is a multiple of per)
inline ChunkTurns chunk_turns(int d, int chunk, int per) { return ChunkTurns{chunk / per, d / chunk, (d % chunk + per - 1) / per}; }

}  // namespace usl_lists
