// Forward and weight-gradient kernels: float32 activations, 1 instance per group.
#include "k_products_inst.h"

usl_products::ProductKernel usl_products::kernel_f32_q1(ProductKind kind, int K, int shape) {
    return pick_k<float, 1, false>(kind, K, shape);
}
