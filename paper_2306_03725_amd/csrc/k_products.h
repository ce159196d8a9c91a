// Kernels of the two products, handed out by the files that instantiate them.
#pragma once

namespace usl_products {

// FORWARD_LOSS: the scores become the gradient of the loss; FORWARD_MARKS: of the squared hinge, and its nonzeros are marked
enum ProductKind { FORWARD, FORWARD_LOSS, FORWARD_MARKS, WEIGHT_GRADIENT };

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

}  // namespace usl_products
