// Forward and weight-gradient kernels: float32 activations, rows in two halves.
#include "k_products_inst.h"

usl_products::ProductKernel usl_products::kernel_f32_halves(ProductKind kind, int K, int shape) {
    return pick_k<float, 1, true>(kind, K, shape);
}
