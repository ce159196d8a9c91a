// Instances of the forward and weight-gradient kernels for one (storage type, instances per group), included by one
// source file each so that they compile side by side.  Defines a function that hands out the kernels by fan-in and
// workgroup shape:  shape 0 = 256 lanes x 1 label,  1 = 512 x 64 / K,  2 = 1024 x 64 / K (64 slots of 6 bytes take 96 of
// the 128 registers a lane of a full compute unit has; twice the slots in 512 lanes of 256 registers was slower
// everywhere but in the forward product at K = 64).
// Rows that leave room for one workgroup per compute unit (Q = 1) come in the wide shapes only.
// bfloat16 with K = 64 in such rows (Q <= 2) also as 1024 lanes with one label each in the forward product: sixteen
// wavefronts wait for their reads instead of eight.  64 slots of 4 bytes and what the loop needs are more than the 128
// registers: 53 to 59 are spilled with Q = 2 and 33 to 35 with Q = 1, as many as 512 lanes with two labels spill of 256
// (47 to 64), and the scratch they are read back from stays in the caches.  m = 670k, d = 32k, k = 64, b = 512: 512 lanes
// with two labels 2362 us, this 2310; a step of 8 ms gains less than its own runs differ by (1 to 3 %).  Not in shorter
// rows, where smaller workgroups share a compute unit (m = 300k, d = 4k, k = 60, b = 64: 512 lanes with one 121, this 151).
#pragma once
#include "k_products_common.h"
#include "k_products.h"

namespace usl_products {

constexpr int labels_per_lane(int K, int slots) { return slots / K < 1 ? 1 : slots / K > 8 ? 8 : slots / K; }

template <int K, typename TS, int Q, bool HALVES>
ProductKernel pick(ProductKind kind, int shape) {
    constexpr int L = K == 8 ? 4 : labels_per_lane(K, 64), L2 = labels_per_lane(K, 128);
    constexpr bool WIDE_PAIRS = K == 64 && sizeof(TS) == 2 && Q <= 2;
#define USL_FORWARD_KIND(LPT, NT, EVEN)                                                                        \
    (kind == FORWARD_MARKS    ? (const void*)k_forward<K, LPT, NT, TS, Q, HALVES, 2, EVEN, false>               \
     : kind == FORWARD_LOSS   ? (const void*)k_forward<K, LPT, NT, TS, Q, HALVES, 1, EVEN, false>               \
     : kind == FORWARD_CACHED ? (const void*)k_forward<K, LPT, NT, TS, Q, HALVES, 0, EVEN, (K <= 16 || (K == 24 && Q == 4))> \
                              : (const void*)k_forward<K, LPT, NT, TS, Q, HALVES, 0, EVEN, (K <= 16)>)
#define USL_FORWARD(LPT, NT) ProductKernel{USL_FORWARD_KIND(LPT, NT, false), USL_FORWARD_KIND(LPT, NT, true), K, LPT, NT, transpose_bytes<K, NT>()}
#define USL_GRADIENT(LPT, NT)                                                                                  \
    ProductKernel{(const void*)k_backward_weight<K, LPT, NT, TS, Q, HALVES, false>, (const void*)k_backward_weight<K, LPT, NT, TS, Q, HALVES, true>, \
                  K, LPT, NT, transpose_bytes<K, NT>()}
#define USL_PICK(LPT, NT) (gradient ? USL_GRADIENT(LPT, NT) : USL_FORWARD(LPT, NT))
    const bool gradient = kind == WEIGHT_GRADIENT;
    if constexpr (Q > 1) {
        if (shape == 0) return USL_PICK(1, 256);
        if (shape == 1) return USL_PICK(L, 512);
        if constexpr (K == 64) {
            if (shape == 2) return gradient ? USL_GRADIENT(L, 1024) : USL_FORWARD(L2, 512);
        } else {
            if (shape == 2) return USL_PICK(L, 1024);
        }
        if constexpr (L > 1 && K >= 16) {
            if (shape == 3) return USL_PICK(1, 1024);
        } else if constexpr (WIDE_PAIRS) {
            if (shape == 3 && !gradient) return USL_FORWARD(1, 1024);
        }
    } else if constexpr (K < 64) {
        if (shape == 1) return USL_PICK(1, 1024);
        if constexpr (L > 1) {
            if (shape == 2) return USL_PICK(L, 1024);
        }
    } else {   // 64 slots in 128 registers would spill
        if (shape == 1) return USL_PICK(1, 512);
        if (shape == 2) return USL_PICK(L2, 512);
        if constexpr (WIDE_PAIRS) {
            if (shape == 3 && !gradient) return USL_FORWARD(1, 1024);
        }
    }
#undef USL_PICK
#undef USL_GRADIENT
#undef USL_FORWARD
#undef USL_FORWARD_KIND
    return ProductKernel{nullptr, nullptr, 0, 0, 0, 0};
}

template <typename TS, int Q, bool HALVES>
ProductKernel pick_k(ProductKind kind, int K, int shape) {
    switch (K) {
        case 8: return pick<8, TS, Q, HALVES>(kind, shape);
        case 16: return pick<16, TS, Q, HALVES>(kind, shape);
        case 24: return pick<24, TS, Q, HALVES>(kind, shape);
        case 32: return pick<32, TS, Q, HALVES>(kind, shape);
        case 48: return pick<48, TS, Q, HALVES>(kind, shape);
        case 64: return pick<64, TS, Q, HALVES>(kind, shape);
        default: return ProductKernel{nullptr, nullptr, 0, 0, 0, 0};
    }
}

}  // namespace usl_products
