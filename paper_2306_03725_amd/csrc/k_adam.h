// Device code that the kernels which end a training step share: the sum of the loss, Adam on one weight.
#pragma once
#include "usl_internal.h"

// One block adds the per-block sums in a fixed order: the loss is reproducible run to run.  Sixteen loads of a lane in flight: what
// bounds it is their latency (31 500 sums by 1024 lanes: 13.5 and 7.3 us).
template <int NT_>
__device__ __forceinline__ void sum_loss(const usl_loss_sum& sum) {
    __shared__ double red[NT_ / 64];
    double s = 0.0;
    constexpr int AT_ONCE = 16;
    for (size_t q0 = threadIdx.x; q0 < sum.n; q0 += (size_t)NT_ * AT_ONCE) {
        double v[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) v[u] = q0 + (size_t)u * NT_ < sum.n ? sum.partials[q0 + (size_t)u * NT_] : 0.0;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) s += v[u];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < NT_ / 64; ++q) t += red[q];
        *sum.loss = (float)((double)sum.scale * t);
    }
}

// The first `lead` blocks (of 256 lanes) of the kernel that ends a step whose loss forward computed: the first of them adds up the loss, the
// others take the targets' bits back, four instances to a wavefront.  In front of the others, which are at work by the time these
// wait for the target lists.
static inline unsigned step_end_blocks(const usl_loss_sum& sum) { return sum.partials ? (unsigned)((1 + (sum.targets.b + 15) / 16 + 7) / 8 * 8) : 0u; }   // (a multiple of 8: the others keep their XCDs)
__device__ __forceinline__ void step_end(const usl_loss_sum& sum, unsigned lead) {
    if (blockIdx.x == 0) { sum_loss<256>(sum); return; }
    const usl_targets& t = sum.targets;
    if (!t.off) return;
    const int n = ((int)lead - 1) * 4;
    for (int i = (int)(blockIdx.x - 1) * 4 + (int)(threadIdx.x >> 6); i < t.b; i += n) {
        const int64_t p1 = t.off[i + 1];
        for (int64_t p = t.off[i] + (threadIdx.x & 63); p < p1; p += 64) {
            const int64_t j = t.lab[p];
            if (j >= 0 && j < t.m) t.bits[(size_t)(i >> 5) * t.m + j] = 0u;   // all bits of the word go in this launch; nobody reads them
        }
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
