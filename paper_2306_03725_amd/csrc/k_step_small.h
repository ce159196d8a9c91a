// Which layers take the training step in two launches (k_step_small.hip), and where things lie in LDS there.
#pragma once

#include <stdint.h>

namespace usl_small {

constexpr int NL = 64;                              // labels of a workgroup
constexpr int MOST_K = 32, SLOT_BITS = 11;          // NL * MOST_K slots; a key: column above, slot below
static_assert(NL * MOST_K == 1 << SLOT_BITS, "a slot fits its bits");
constexpr int LDS_MOST = 144 * 1024;   // (m = 2746, d = 1636, k = 8, b = 19, 144 KB: 33 and 39 us; m = 2065, d = 878, k = 32, b = 26, 143 KB: 42 and 38)

// Byte offsets in LDS
struct SmallLds {
    int x, red, g, rows, keys, ent, first, bits, off, bytes;
};
__host__ __device__ inline SmallLds small_lds(int d, int k, int b, int waves) {
    const int G = (b + 3) / 4, x = G * d * 16, red = waves * NL * (k + 1) * 4;
    SmallLds L;
    L.x = 0;                                  // [G][d] units of four instances; then
    L.red = 0;                                // [waves][NL][k + 1] sums of the weight gradient
    L.g = (x > red ? x : red);                // [G][NL] of the gradient
    L.rows = L.g + G * NL * 16;               // [NL][k + 1] {byte of the column's unit, weight}
    L.keys = L.rows + NL * (k + 1) * 8;
    int n2 = 64;
    while (n2 < NL * k) n2 *= 2;
    L.ent = L.keys + (n2 + 1) * 4 / 16 * 16 + 16;   // [NL * k] {byte of the label's unit, weight} in the order of the columns
    L.first = L.ent + NL * k * 8;             // [d] first entry of a column, and behind it the last one + 1, 16 bits each
    L.bits = L.first + (d * 4 + 15) / 16 * 16;   // [b] which of the labels are targets
    L.off = L.bits + b * 8;                   // [b + 1] where the instances' targets begin
    L.bytes = (L.off + (b + 1) * 4 + 15) / 16 * 16;
    return L;
}

// Wavefronts of a workgroup: eight where four would have more than two groups of instances each
static inline int small_waves(int b) { return b > 32 ? 8 : 4; }

static inline bool small_step_fits(int64_t m, int d, int k, int b) {
    if (k > MOST_K || d > 65536 || b > 1024 || (int64_t)(b + 3) / 4 * 16 * d > LDS_MOST) return false;
    return small_lds(d, k, b, small_waves(b)).bytes <= LDS_MOST && (m + NL - 1) / NL <= 65535;
}

// By the largest batch, so that every batch of a layer takes the same path and finds its scratch sized.  A workgroup is bound by its own chain, so the path pays
// where few workgroups follow one another on a compute unit: as many as LDS holds at once (registers leave room for 28 wavefronts of up to 8
// slots a label, 16 of up to 16, 8 of more, so some of these are two rounds: still ahead).  Both paths, us:
// m = 1024, d = 64, k = 8, b = 16: 30.2 and 10.8; m = 4096, d = 256, k = 16, b = 32: 37.9 and 19.8; m = 16 000, d = 64, k = 32, b = 64: 65.6 and 29.1;
// m = 36 551, d = 140, k = 16, b = 9: 47.2 and 25.0; two rounds by registers: m = 76 770, d = 62, k = 12, b = 4: 54 and 36; m = 61 269, d = 79, k = 6, b = 52: 57 and 45;
// two rounds by LDS: m = 31 147, d = 211, k = 31, b = 43: 70 and 88; m = 31 974, d = 843, k = 16, b = 19: 49 and 74.
// Not where the general path has little to do for a label, or a wavefront brings in long rows of several groups of instances, one column a lane after the other:
// k <= 4, seven workgroups a compute unit and more: m = 113 303, d = 265, k = 4, b = 5 32 and 45; m = 200 000, d = 64, k = 3, b = 8 38 and 60; m = 72 586, d = 181, k = 3, b = 11
// 31.5 and 31.2; with hardly a feature it is the other way round: m = 137 886, d = 16, k = 4, b = 4 60 and 43.
// 25 columns a lane and more: m = 15 555, d = 1658, k = 24, b = 9 35 and 51; m = 9551, d = 778, k = 28, b = 28 41 and 49; m = 3782, d = 747, k = 16, b = 17 (24) 34 and 31.
static inline bool small_step_pays(int64_t m, int d, int k, int b, int cus) {
    const int waves = small_waves(b), groups = (b + 3) / 4;
    const int64_t wgs = (m + NL - 1) / NL;
    if (wgs > (int64_t)cus * (160 * 1024 / small_lds(d, k, b, waves).bytes)) return false;
    if (k <= 4 && d > 24 && wgs > (int64_t)cus * 6) return false;
    return groups < 3 || (groups + waves - 1) / waves * ((d + 63) / 64) <= 24;
}

}  // namespace usl_small
