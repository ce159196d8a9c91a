// Device code that the kernels which end a training step share: the sum of the loss, Adam on one weight.
#pragma once
#include "usl_internal.h"

// One block adds the per-block sums in a fixed order: the loss is reproducible run to run.
template <int NT_>
__device__ __forceinline__ void sum_loss(const usl_loss_sum& sum) {
    __shared__ double red[NT_ / 64];
    double s = 0.0;
    for (size_t q = threadIdx.x; q < sum.n; q += NT_) s += sum.partials[q];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < NT_ / 64; ++q) t += red[q];
        *sum.loss = (float)((double)sum.scale * t);
    }
}

template <typename TS> struct WIo;
template <> struct WIo<float> {
    static __device__ __forceinline__ float get(const float* W, size_t f) { return W[f]; }
    static __device__ __forceinline__ void put(float* W, size_t f, float v) { W[f] = v; }
};
template <> struct WIo<uint16_t> {
    static __device__ __forceinline__ float get(const uint16_t* W, size_t f) { return usl_bf16_to_f32(W[f]); }
    static __device__ __forceinline__ void put(uint16_t* W, size_t f, float v) { W[f] = usl_f32_to_bf16(v); }
};

__device__ __forceinline__ float adam_one(float w, float gw, float& a, float& v, float lr, float b1,
                                          float b2, float eps, float ic1, float ic2) {
    a = fmaf(b1, a, (1.f - b1) * gw);
    v = fmaf(b2, v, (1.f - b2) * gw * gw);
    return w - lr * (a * ic1) / (sqrtf(v * ic2) + eps);
}
