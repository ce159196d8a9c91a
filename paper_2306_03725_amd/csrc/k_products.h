// Kernels of the two products, handed out by the files that instantiate them.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace usl_products {

// FORWARD_CACHED: the scores go through the caches where FORWARD's go past them (K = 24 and four instances a read; others: FORWARD's kernel); FORWARD_LOSS: the scores become
// the gradient of the loss; FORWARD_MARKS: of the squared hinge, and its nonzeros are marked
enum ProductKind { FORWARD, FORWARD_CACHED, FORWARD_LOSS, FORWARD_MARKS, WEIGHT_GRADIENT };

struct ProductKernel {
    const void* fn;        // nullptr: no such kernel
    const void* even;      // the same for blocks of fewer labels than its lanes take
    int K, LPT, NT;        // padded fan-in, labels per lane, lanes
    int transpose_bytes;   // LDS its prologue and epilogue need
};

ProductKernel kernel_f32_q4(ProductKind kind, int K, int shape);
ProductKernel kernel_f32_q2(ProductKind kind, int K, int shape);
ProductKernel kernel_f32_q1(ProductKind kind, int K, int shape);
ProductKernel kernel_f32_halves(ProductKind kind, int K, int shape);
ProductKernel kernel_bf16_q4(ProductKind kind, int K, int shape);
ProductKernel kernel_bf16_q2(ProductKind kind, int K, int shape);
ProductKernel kernel_bf16_q1(ProductKind kind, int K, int shape);

// Workgroups of NT lanes with `regs` registers each and `lds` bytes that a compute unit holds.
static inline int resident_workgroups(int NT, int regs, size_t lds) {
    const int by_regs = regs < 64 ? 8 : 512 / ((regs + 7) / 8 * 8);   // wavefronts on a SIMD
    const int waves = by_regs * 4 / (NT / 64), by_lds = (int)((size_t)(160 * 1024) / lds), n = waves < by_lds ? waves : by_lds;
    return n < 1 ? 1 : n;
}

// Blocks of equal size: where not every compute unit has as many workgroups as the busiest, so many fewer labels to a block that it has (its
// share of the row copies stays what it was).  nblk full blocks, the batch in `parts`; `resident` workgroups to a compute unit.
// m = 200k, d = 8k, k = 32, b = 64, bfloat16 (196 blocks of 1024 labels or 250 of 800): forward 56 and 49 us; weight gradient of m = 300k,
// d = 24k, k = 48, b = 64: 255 and 227.  Where lanes have several labels, and so fewer of them in a smaller block, the blocks fill all places of a
// round of workgroups (m = 404k, d = 1331, k = 8, b = 115: a step 266 us with 506 blocks, 294 with 253); where they have one, smaller blocks leave
// lanes idle, and filled up that way 3 in 5 launches took longer (m = 67k, d = 498, k = 16, b = 12: 9.0 and, in 1053 blocks, 12.4).
static inline int even_block_labels(int64_t m, const ProductKernel& kern, int64_t nblk, int parts, int cus, int resident) {
    const int64_t unit = kern.LPT > 1 ? (int64_t)cus * resident : cus, most = (nblk * parts + unit - 1) / unit * unit / parts;   // nblk at least
    return (int)(((m + most - 1) / most + 31) / 32 * 32);   // (the slot order goes by 32 labels)
}

// Not where the form for them spills more than the one of full blocks (bfloat16 with two labels of 32 slots on 1024 lanes: m = 150k, d = 15k,
// b = 64: 65 and 74).  Nor, with the batch in more than 8 parts, where x is more than an L2 holds beside the rest: more blocks then bring it in
// more often (m = 1399, d = 52k, k = 8, b = 54: 9.4 and 20.6; of 1250 such launches of up to 4000 labels half are slower by more than 3 %).
static inline bool even_blocks_allowed(int parts, int64_t x_bytes, size_t scratch_full, size_t scratch_even) {
    return scratch_even <= scratch_full && (parts <= 8 || x_bytes <= (int64_t)2 << 20);
}

}  // namespace usl_products
