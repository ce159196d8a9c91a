// Device code that adds up the windows' (or chains of windows') sums of the input gradient.
#pragma once
#include "usl_internal.h"

// out[i][c] = sum over the sets of partial[set][i][c], by block `block` of `blocks` of 256 lanes each.
// Bound by the stream of the partial sums.  Where lanes are few the loads of eight or four windows go out together (AT_ONCE): one
// after the other a lane waits out every window.  Where they are many, one: they cover for one another, and their rows stay
// close together.  In a step, with eight, four, one: m = 31k, d = 1k, b = 128 (128 workgroups): 5.8, 6.4, 11.0 us; m = 200k, d = 8k, b = 64
// (512): 24, 22, 31; m = 60k, d = 8k, b = 128 (1000): 15.1, 13.9, 12.6; m = 130k, d = 32k, b = 64 (2048): 17.8, 16.4, 15.6; m = 500k,
// d = 32k, b = 256, 537 MB: 116, 119, 109 (120 with the rows from the first).
template <int AT_ONCE>
__device__ __forceinline__ void usl_add_up_windows(const usl_window_sums& s, bool poison, unsigned block, unsigned blocks) {
    const size_t step = (size_t)blocks * 256;
    for (size_t u = (size_t)block * 256 + threadIdx.x; u < s.n4; u += step) {
        const size_t v = s.n4 - 1 - u;   // the last rows first: they were written last, and may still be in a cache
        float4 a = s.partial[v];
#pragma unroll AT_ONCE
        for (int q = 1; q < s.sets; ++q) {
            const float4 t = s.partial[(size_t)q * s.n4 + v];
            a.x += t.x; a.y += t.y; a.z += t.z; a.w += t.w;
        }
        if (poison) a.x = a.y = a.z = a.w = __uint_as_float(0x7FC00000u);
        if (s.vec) {
            reinterpret_cast<float4*>(s.out)[v] = a;
        } else {
            const uint32_t row4 = (uint32_t)s.dp / 4, i = (uint32_t)(v / row4), c = (uint32_t)(v % row4) * 4;
            float* to = s.out + (size_t)i * s.d + c;
            const float r[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((int)c + q < s.d) to[q] = r[q];
        }
    }
}
