// Forward and weight-gradient kernels: bfloat16 activations, 2 instances per group.
#include "k_products_inst.h"

usl_products::ProductKernel usl_products::kernel_bf16_q2(ProductKind kind, int K, int shape) {
    return pick_k<uint16_t, 2, false>(kind, K, shape);
}
