// Forward and weight-gradient kernels: float32 activations, 2 instances per group.
#include "k_products_inst.h"

usl_products::ProductKernel usl_products::kernel_f32_q2(ProductKind kind, int K, int shape) {
    return pick_k<float, 2, false>(kind, K, shape);
}
