// Forward and weight-gradient kernels: float32 activations, 4 instances per group.
#include "k_products_inst.h"

usl_products::ProductKernel usl_products::kernel_f32_q4(ProductKind kind, int K, int shape) {
    return pick_k<float, 4, false>(kind, K, shape);
}
