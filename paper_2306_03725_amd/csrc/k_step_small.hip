// The whole training step of a small layer in two launches (usl_train_step).
//
// What bounds a step that gathers little is the chain of launches and of trips to memory behind one another, whatever the sizes: copy of the
// activations, forward with the loss, the targets, both backward products, Adam took 30 us at m = 1024, d = 64, k = 8, b = 16, of which
// k_both_lds, which brings lists, weights, slices of g and sums one after the other, 16.6.  Here a workgroup has 64 labels and the
// whole batch: their rows and all of x come in, then the targets, and everything else happens in LDS.  Each of its four or eight wavefronts takes all
// 64 labels (a lane each) for its share of the groups of four instances; x lies interleaved by four, so a slot costs one read of 16 bytes.
// The input gradient of the workgroup's labels is gathered from its own connections in the order of their columns and left as a partial sum
// per workgroup, which the second launch adds up in a fixed order.
//
// The order of the connections depends on idx alone.  The workgroup keeps it in scratch of the context and looks at every entry before it uses it: keys
// (column, slot) that rise from entry to entry are all its connections, once each, in order, whatever the scratch held before; anything else is sorted
// anew.  So nothing here can be stale.
//
// Where it is used, and both paths' times: small_step_pays.
#include <stdlib.h>
#include <string.h>

#include "k_adam.h"
#include "k_products_common.h"   // dot2
#include "k_step_small.h"

using namespace usl_small;

namespace {

struct SmallArgs {
    const void* x;
    const int32_t* idx;
    float *m1, *m2;
    const int64_t* off;
    const int32_t* lab;
    float *g, *grad_W;
    float* sums;         // [workgroups][b][d] of the input gradient; nullptr: not asked for
    double* partials;    // [workgroups] of the loss
    uint16_t* order;     // [workgroups][NL * k]
    int64_t m;
    int d, k, b, kind;
    float scale, lr, b1, b2, eps, ic1, ic2;
};

// KP: k, or (FULL = false) the power of two above it.  SHARED: wavefronts share the columns of a group of instances (of four
// wavefronts one or two had long rows to themselves and the others none: m = 2096, d = 5314, k = 2, b = 4 67 and 26 us; m = 1762, d = 6033, k = 6, b = 1 47
// and 20; rows of up to 128 columns 2 to 5 % slower so, and with three groups and more there is nothing to share).
template <typename TS, int KP, bool FULL, int NT, bool SHARED>
__global__ void __launch_bounds__(NT)
k_step_small(SmallArgs a, TS* __restrict__ W) {
    constexpr int PER = NL * KP / NT, WAVES = NT / 64;   // slots of a lane
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = (int)threadIdx.x, label = tid & 63, wave = tid >> 6, k = FULL ? KP : a.k, d = a.d, b = a.b, G = (b + 3) / 4;
    const SmallLds L = small_lds(d, k, b, WAVES);
    float4* xs = reinterpret_cast<float4*>(lds + L.x);
    float4* gs = reinterpret_cast<float4*>(lds + L.g);
    uint2* rows = reinterpret_cast<uint2*>(lds + L.rows);
    float* red = reinterpret_cast<float*>(lds + L.red);
    uint32_t* keys = reinterpret_cast<uint32_t*>(lds + L.keys);
    uint2* ent = reinterpret_cast<uint2*>(lds + L.ent);
    uint16_t* first = reinterpret_cast<uint16_t*>(lds + L.first);
    uint32_t* bits = reinterpret_cast<uint32_t*>(lds + L.bits);
    uint32_t* offs = reinterpret_cast<uint32_t*>(lds + L.off);
    const int64_t j0 = (int64_t)blockIdx.x * NL;
    const int nl = (int)min((int64_t)NL, a.m - j0), n = nl * k;
    const size_t f0 = (size_t)j0 * k;
    const uint32_t inv = k > 1 ? 0xFFFFFFFFu / (uint32_t)k + 1u : 0u;   // e / k by a multiplication; exact: e < 2^11
    auto label_of = [&](int e) { return k > 1 ? (int)__umulhi((uint32_t)e, inv) : e; };
    // of x and its gradient a wavefront has group `group0` and every WAVES-th after it, columns `column0` and every `columns`-th
    static_assert(!SHARED || WAVES == 4, "one group or two");
    const int share = !SHARED ? 0 : G == 1 ? wave : wave >> 1, group0 = !SHARED ? wave : G == 1 ? 0 : wave & 1;
    const int column0 = share * 64 + label, columns = !SHARED ? 64 : G == 1 ? 256 : 128;

    // what has to come from memory: the rows on their way together, behind them the offsets and x, which go to LDS as they come
    uint32_t col[PER];
    float w[PER], a1[PER], a2[PER];
    uint32_t ord[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = tid + q * NT;
        const bool in = e < n;
        col[q] = in ? (uint32_t)a.idx[f0 + e] : 0u;
        w[q] = in ? WIo<TS>::get(W, f0 + e) : 0.f;
        a1[q] = in ? a.m1[f0 + e] : 0.f;
        a2[q] = in ? a.m2[f0 + e] : 0.f;
        ord[q] = in && a.sums ? a.order[f0 + e] : 0u;
    }
    const int64_t t0 = a.off[0];
    for (int i = tid; i <= b; i += NT) offs[i] = (uint32_t)(a.off[i] - t0);
    const TS* x = reinterpret_cast<const TS*>(a.x);
    for (int g = group0; g < G; g += WAVES)
        for (int c = column0; c < d; c += columns) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = 4 * g + q < b ? usl_load_f32<TS>(x, (size_t)(4 * g + q) * d + c) : 0.f;
            xs[g * d + c] = make_float4(v[0], v[1], v[2], v[3]);
        }
    for (int i = tid; i < 2 * b; i += NT) bits[i] = 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = tid + q * NT, l = label_of(e);
        if (e < NL * k) rows[l * (k + 1) + e - l * k] = make_uint2(col[q] * 16u, __float_as_uint(w[q]));   // (labels that do not exist: weight 0)
    }
    __syncthreads();

    // targets: which of the workgroup's labels they are
    const uint32_t n_tgt = offs[b];
    int32_t tgt = (uint32_t)tid < n_tgt ? a.lab[t0 + tid] : -1;
    // forward
    uint32_t at[KP];
    float wr[KP];
#pragma unroll
    for (int t = 0; t < KP; ++t) {
        const uint2 r = t < k ? rows[label * (k + 1) + t] : make_uint2(0u, 0u);
        at[t] = r.x;
        wr[t] = __uint_as_float(r.y);
    }
    auto unit = [&](int g, uint32_t byte) { return *reinterpret_cast<const float4*>(reinterpret_cast<const unsigned char*>(xs + (size_t)g * d) + byte); };
    for (int g = wave; g < G; g += WAVES) {
        // The bits of usl_forward: in the order of the slots (bfloat16 by pairs), or, for up to four instances, by fours of them that are added
        // up pairwise (k_forward_few).
        constexpr int F = KP / 4;
        float4 part[F];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            float4 z = f == 0 || G == 1 ? make_float4(0.f, 0.f, 0.f, 0.f) : part[f == 0 ? 0 : f - 1];
#pragma unroll
            for (int t = 4 * f; t < 4 * f + 4; t += 2)
                if (t < k) {
                    const float4 u = unit(g, at[t]), v = t + 1 < k ? unit(g, at[t + 1]) : make_float4(0.f, 0.f, 0.f, 0.f);
                    if constexpr (sizeof(TS) == 4) {
                        const float w0 = wr[t], w1 = wr[t + 1];
                        z.x = fmaf(w0, u.x, z.x); z.y = fmaf(w0, u.y, z.y); z.z = fmaf(w0, u.z, z.z); z.w = fmaf(w0, u.w, z.w);
                        z.x = fmaf(w1, v.x, z.x); z.y = fmaf(w1, v.y, z.y); z.z = fmaf(w1, v.z, z.z); z.w = fmaf(w1, v.w, z.w);
                    } else {
                        const uint32_t w2 = usl_products::join_hi(__float_as_uint(wr[t]), __float_as_uint(wr[t + 1]));
                        auto both = [&](float p, float q, float acc) { return usl_products::dot2(usl_products::join_hi(__float_as_uint(p), __float_as_uint(q)), w2, acc); };
                        z.x = both(u.x, v.x, z.x); z.y = both(u.y, v.y, z.y); z.z = both(u.z, v.z, z.z); z.w = both(u.w, v.w, z.w);
                    }
                }
            part[f] = z;
        }
        if (G == 1) {
#pragma unroll
            for (int o = 1; o < F; o *= 2)
#pragma unroll
                for (int f = 0; f + o < F; f += 2 * o) { part[f].x += part[f + o].x; part[f].y += part[f + o].y; part[f].z += part[f + o].z; part[f].w += part[f + o].w; }
            part[F - 1] = part[0];
        }
        const float4 z = part[F - 1];
        gs[g * NL + label] = z;
    }
    for (uint32_t p = (uint32_t)tid;;) {
        const int64_t j = (int64_t)tgt - j0;
        if (p < n_tgt && tgt >= 0 && j >= 0 && j < nl) {
            int lo = 0, hi = b;   // the instance: offs[lo] <= p < offs[lo + 1]
            while (hi - lo > 1) {
                const int mid = (lo + hi) / 2;
                if (offs[mid] <= p) lo = mid; else hi = mid;
            }
            atomicOr(&bits[2 * lo + (int)(j >> 5)], 1u << (j & 31));
        }
        p += NT;
        if (p >= n_tgt) break;
        tgt = a.lab[t0 + p];
    }
    __syncthreads();

    // loss, and what the wavefront's instances give to the weight gradient
    double lost = 0.0;
    float gw[KP];
#pragma unroll
    for (int t = 0; t < KP; ++t) gw[t] = 0.f;
    for (int g = wave; g < G; g += WAVES) {
        const float4 z4 = gs[g * NL + label];
        const float z[4] = {z4.x, z4.y, z4.z, z4.w};
        float gv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 4 * g + q;
            gv[q] = 0.f;
            if (i < b && label < nl) {
                const float y = (bits[2 * i + (label >> 5)] >> (label & 31)) & 1u ? 1.f : 0.f;
                const usl_loss_of r = usl_loss_one(a.kind, z[q], y, a.scale);
                gv[q] = r.g;
                lost += (double)r.l;
                a.g[(size_t)i * a.m + j0 + label] = r.g;
            }
        }
        gs[g * NL + label] = make_float4(gv[0], gv[1], gv[2], gv[3]);
#pragma unroll
        for (int t = 0; t < KP; ++t)
            if (t < k) {
                const float4 v = unit(g, at[t]);
                gw[t] = fmaf(gv[0], v.x, gw[t]); gw[t] = fmaf(gv[1], v.y, gw[t]); gw[t] = fmaf(gv[2], v.z, gw[t]); gw[t] = fmaf(gv[3], v.w, gw[t]);
            }
    }
    __syncthreads();   // x has been read
#pragma unroll
    for (int t = 0; t < KP; ++t)
        if (t < k) red[(wave * NL + label) * (k + 1) + t] = gw[t];
    // the connections in the order of their columns
    uint32_t key[PER];
    int n2 = 64;
    while (n2 < n) n2 *= 2;
    if (a.sums) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + q * NT;
            const uint32_t s = min(ord[q], (uint32_t)n - 1u), l = (uint32_t)label_of((int)s);
            key[q] = rows[l * (k + 1) + s - l * k].x / 16u << SLOT_BITS | s;
            if (e < n) keys[e] = key[q];
        }
        for (int c = tid; c < 2 * d; c += NT) first[c] = 0;
    }
    __syncthreads();   // red, gs, keys
    if (a.sums) {
        bool wrong = false;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + q * NT;
            if (e > 0 && e < n && keys[e - 1] >= key[q]) wrong = true;
        }
        if (__syncthreads_or(wrong)) {   // new connectivity
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int e = tid + q * NT;
                if (e < n2) keys[e] = e < n ? col[q] << SLOT_BITS | (uint32_t)e : 0xFFFFFFFFu;
            }
            __syncthreads();
            for (int size = 2; size <= n2; size *= 2)
                for (int step = size / 2; step > 0; step /= 2) {
                    for (int p = tid; p < n2 / 2; p += NT) {
                        const int lo = p / step * 2 * step + p % step, hi = lo + step;
                        const uint32_t u = keys[lo], v = keys[hi];
                        if ((u > v) == ((lo & size) == 0)) { keys[lo] = v; keys[hi] = u; }
                    }
                    __syncthreads();
                }
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int e = tid + q * NT;
                if (e < n) {
                    key[q] = keys[e];
                    a.order[f0 + e] = (uint16_t)(key[q] & ((1u << SLOT_BITS) - 1u));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + q * NT;
            if (e >= n) continue;
            const uint32_t s = key[q] & ((1u << SLOT_BITS) - 1u), c = key[q] >> SLOT_BITS, l = (uint32_t)label_of((int)s);
            ent[e] = make_uint2(l * 16u, rows[l * (k + 1) + s - l * k].y);
            if (e == 0 || keys[e - 1] >> SLOT_BITS != c) first[2 * c] = (uint16_t)e;
            if (e == n - 1 || keys[e + 1] >> SLOT_BITS != c) first[2 * c + 1] = (uint16_t)(e + 1);
        }
    }
    // Adam
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = tid + q * NT, l = label_of(e);
        if (e >= n) continue;
        float gv = red[l * (k + 1) + e - l * k];
#pragma unroll
        for (int v = 1; v < WAVES; ++v) gv += red[(v * NL + l) * (k + 1) + e - l * k];
        a.grad_W[f0 + e] = gv;
        const float wn = adam_one(w[q], gv, a1[q], a2[q], a.lr, a.b1, a.b2, a.eps, a.ic1, a.ic2);
        a.m1[f0 + e] = a1[q];
        a.m2[f0 + e] = a2[q];
        WIo<TS>::put(W, f0 + e, wn);
    }
    __syncthreads();   // ent, first; red has been read
    for (int o = 32; o > 0; o >>= 1) lost += __shfl_down(lost, o);
    if (label == 0) reinterpret_cast<double*>(lds + L.rows)[wave] = lost;   // (rows have been read)
    if (a.sums) {
        for (int g = group0; g < G; g += WAVES) {
            const unsigned char* gg = reinterpret_cast<const unsigned char*>(gs + (size_t)g * NL);
            for (int c = column0; c < d; c += columns) {
                float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
                const uint32_t range = reinterpret_cast<const uint32_t*>(first)[c];
                uint32_t e = range & 0xFFFFu;
                const uint32_t end = range >> 16;
                auto add = [&](uint2 u, float4 v) {
                    const float we = __uint_as_float(u.y);
                    s.x = fmaf(we, v.x, s.x); s.y = fmaf(we, v.y, s.y); s.z = fmaf(we, v.z, s.z); s.w = fmaf(we, v.w, s.w);
                };
                for (; e + 4 <= end; e += 4) {   // four entries' reads together
                    uint2 u[4];
                    float4 v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) u[q] = ent[e + q];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const float4*>(gg + u[q].x);
#pragma unroll
                    for (int q = 0; q < 4; ++q) add(u[q], v[q]);
                }
                for (; e < end; ++e) {
                    const uint2 u = ent[e];
                    add(u, *reinterpret_cast<const float4*>(gg + u.x));
                }
                const float r[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (4 * g + q < b) a.sums[((size_t)blockIdx.x * b + 4 * g + q) * d + c] = r[q];
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        const double* r = reinterpret_cast<const double*>(lds + L.rows);
        double t = 0.0;
        for (int v = 0; v < WAVES; ++v) t += r[v];
        a.partials[blockIdx.x] = t;
    }
}

// grad_x[v] = the workgroups' sums, added up in a fixed order: 64 values and four runs of workgroups to a block.  The last block: the loss.
constexpr int SUMS_NT = 256;
__global__ void __launch_bounds__(SUMS_NT)
k_step_small_sums(const float* __restrict__ sums, int wgs, size_t n, float* __restrict__ grad_x, usl_loss_sum sum) {
    if (blockIdx.x == gridDim.x - 1) {
        sum_loss<SUMS_NT>(sum);
        return;
    }
    constexpr int WAVES = SUMS_NT / 64;
    __shared__ float part[WAVES][64];
    const size_t v = (size_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const int wave = (int)threadIdx.x >> 6, per = (wgs + WAVES - 1) / WAVES, w1 = min(wgs, (wave + 1) * per);
    float s = 0.f;
    if (v < n) {
#pragma unroll 8
        for (int w = wave * per; w < w1; ++w) s += sums[(size_t)w * n + v];
    }
    part[wave][threadIdx.x & 63] = s;
    __syncthreads();
    if (wave == 0 && v < n) grad_x[v] = ((part[0][threadIdx.x] + part[1][threadIdx.x]) + part[2][threadIdx.x]) + part[3][threadIdx.x];
}

}  // namespace

// USL_TUNE_SMALL=on|off: wherever the shape allows it at all, or never.
bool usl_step_small_applies(const usl_ctx* c) {
    const char* e = getenv("USL_TUNE_SMALL");
    const bool on = e && strcmp(e, "on") == 0;
    if (!small_step_fits(c->m, c->d, c->k, c->max_b) || (e && *e && !on) || (!on && getenv("USL_TUNE_BOTH"))) return false;
    return on || small_step_pays(c->m, c->d, c->k, c->max_b, c->num_cu);
}

usl_status usl_launch_step_small(usl_ctx* c, const void* x, const int32_t* idx, void* W, float* m1, float* m2, const int64_t* tgt_off,
                                 const int32_t* tgt_lab, int loss_kind, float scale, float lr, float beta1, float beta2, float eps, float inv_c1,
                                 float inv_c2, float* g, float* grad_W, float* grad_x, float* loss, int32_t b) {
    const int wgs = (int)((c->m + NL - 1) / NL);
    USL_TRY(usl_reserve_loss_partials(c));
    USL_TRY(usl_reserve(c, (void**)&c->bce_partials, &c->bce_partials_cap, (size_t)wgs * sizeof(double)));
    if (grad_x) {
        USL_TRY(usl_reserve(c, (void**)&c->small_sums, &c->small_sums_cap, (size_t)wgs * (size_t)c->max_b * (size_t)c->d * 4));
        USL_TRY(usl_reserve(c, (void**)&c->small_order, &c->small_order_cap, (size_t)c->m * c->k * sizeof(uint16_t)));
    }
    SmallArgs a;
    a.x = x; a.idx = idx; a.m1 = m1; a.m2 = m2; a.off = tgt_off; a.lab = tgt_lab; a.g = g; a.grad_W = grad_W;
    a.sums = grad_x ? c->small_sums : nullptr;
    a.partials = c->bce_partials; a.order = c->small_order;
    a.m = c->m; a.d = c->d; a.k = c->k; a.b = b; a.kind = loss_kind;
    a.scale = scale; a.lr = lr; a.b1 = beta1; a.b2 = beta2; a.eps = eps; a.ic1 = inv_c1; a.ic2 = inv_c2;
    const int waves = small_waves(b);
    const size_t lds = (size_t)small_lds(c->d, c->k, b, waves).bytes;
#define USL_SMALL(TS, KP, FULL, NT, SHARED)                                                                                   \
    do {                                                                                                                      \
        if (lds > 65536)                                                                                                      \
            USL_HIP(c, hipFuncSetAttribute((const void*)k_step_small<TS, KP, FULL, NT, SHARED>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
        hipLaunchKernelGGL((k_step_small<TS, KP, FULL, NT, SHARED>), dim3((unsigned)wgs), dim3(NT), lds, c->stream, a, (TS*)W); \
    } while (0)
#define USL_SMALL_W(TS, KP, FULL)                                                                                             \
    do {                                                                                                                      \
        if (waves == 8) USL_SMALL(TS, KP, FULL, 512, false);                                                                  \
        else if (b <= 8 && c->d > 128) USL_SMALL(TS, KP, FULL, 256, true);   /* see the kernel */                             \
        else USL_SMALL(TS, KP, FULL, 256, false);                                                                             \
    } while (0)
#define USL_SMALL_K(TS)                                                                                                       \
    do {                                                                                                                      \
        if (c->k == 8) USL_SMALL_W(TS, 8, true);                                                                              \
        else if (c->k == 16) USL_SMALL_W(TS, 16, true);                                                                       \
        else if (c->k == 32) USL_SMALL_W(TS, 32, true);                                                                       \
        else if (c->k < 8) USL_SMALL_W(TS, 8, false);                                                                         \
        else if (c->k < 16) USL_SMALL_W(TS, 16, false);                                                                       \
        else USL_SMALL_W(TS, 32, false);                                                                                      \
    } while (0)
    if (c->storage == USL_F32) USL_SMALL_K(float); else USL_SMALL_K(uint16_t);
#undef USL_SMALL_K
#undef USL_SMALL_W
#undef USL_SMALL
    USL_TRY(usl_check_launch(c, "training step of a small layer"));
    const size_t n = grad_x ? (size_t)b * c->d : 0;
    hipLaunchKernelGGL(k_step_small_sums, dim3((unsigned)((n + 63) / 64 + 1)), dim3(SUMS_NT), 0, c->stream, c->small_sums, wgs, n, grad_x,
                       usl_loss_sum{c->bce_partials, (size_t)wgs, scale, loss, {}});
    return usl_check_launch(c, "sums of a small layer's step");
}
