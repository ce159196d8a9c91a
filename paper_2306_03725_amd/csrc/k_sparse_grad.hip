// The two backward products over the nonzero entries of g only (Section 3.3: with the squared hinge loss
// the gradient of every easy negative is exactly zero, "implicit negative mining", and Algorithms 2 and 3
// skip those entries).  The dense kernels walk all b*m*k products and can skip zeros only where a whole
// wavefront group or a whole 32-instance piece is zero; here the work is proportional to the nonzeros:
//   1. k_compact_g reads g once and appends every nonzero (label, value) to a list of its instance;
//      an instance that would exceed its list's capacity (more than 1/32 of the labels) marks the
//      gradient "dense" and the lists are abandoned -- the decision is taken on the device, the host
//      never waits for it;
//   2. if the lists stand: grad_W is cleared and every (entry, slot) adds g * x[i][idx[j][t]] into
//      grad_W[j][t] (float atomics: one 4k-byte row of grad_W per entry, few collisions), and grad_x is
//      built one instance per workgroup in an LDS copy of its row (LDS float atomics are slow, but there
//      are only nnz*k of them) and written out once;
//   3. the dense kernels are launched all the same and leave at their first instruction when the lists
//      stand (and the other way round): `gate` below.
// Results equal the dense sums up to the order of the additions (a skipped term is 0 * finite).
#include <stdlib.h>

#include "usl_internal.h"

namespace {

constexpr int CG_NT = 256, CG_PER = 32, CG_CHUNK = CG_NT * CG_PER;   // labels per block, as 8 x float4 per lane

// The words of nz_state: [0] 1 once the gradient counts as dense, [2], [3] the look in progress (look_done), and the number of
// entries listed for instance i, each in a 128-byte line of its own.  Side by side, 32 instances' counts shared a line with
// one another, and the first of them with the word that every block reads first: what a block waits for is its turn at
// that line (k_compact_g, m = 500k, b = 256, usl_backward_weight on 0.5 % nonzeros 293 us with the first rows first, 312 with the
// last, now 272 with either; on 0.1 % 190, 198 and 166; the squared-hinge step 1029, 1010 and 990).
constexpr size_t STATE_LINE = USL_NZ_STATE_LINE;

// The end of a look at g, by one lane of each of its blocks: `full`, the instance's nonzeros cannot fit a list; `dense`, lists would not be worth
// trying.  The blocks meet in one 64-bit word, a count of blocks for each verdict beside the count of all, so nothing has to be
// made visible before it: a fence among the XCDs writes their L2s back, here with a loss's gradients in them.  The block that
// completes the count decides for all and leaves the word 0 for the next look.  (A batch has at most 65535 instances.)  The host's word, serial and verdict in one, needs no order of stores either.
// m = 500k, b = 256: k_probe_density 17.8 us and 4.9 of a launch that cleared the words, now 9.4.
constexpr int LOOK_BITS = 20;
__device__ __forceinline__ void look_done(uint32_t* state, bool full, bool dense, uint32_t blocks, uint32_t* hint, uint32_t serial) {
    unsigned long long* word = reinterpret_cast<unsigned long long*>(state + 2);
    const unsigned long long mine = 1ull | (unsigned long long)dense << LOOK_BITS | (unsigned long long)full << 2 * LOOK_BITS, all = atomicAdd(word, mine) + mine;
    if ((uint32_t)(all & ((1u << LOOK_BITS) - 1)) != blocks) return;
    atomicExch(word, 0ull);
    state[0] = all >> 2 * LOOK_BITS ? 1u : 0u;
    const uint32_t any_dense = (uint32_t)(all >> LOOK_BITS) & ((1u << LOOK_BITS) - 1) ? 1u : 0u;
    __hip_atomic_store(hint, serial << 1 | any_dense, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A look at a sample of g (four labels in 1024 of every row) before the full pass: a dense gradient, the
// common case after binary cross-entropy, is recognised here and the full pass leaves at its first instruction.
// Also clears the instances' counts for that pass.
__global__ void __launch_bounds__(256)
k_probe_density(const float* __restrict__ g, int64_t m, uint32_t* __restrict__ state,
                uint32_t* __restrict__ hint /* pinned host memory: see look_done */,
                uint32_t serial) {
    __shared__ uint32_t seen, hit;
    if (threadIdx.x == 0) { seen = 0; hit = 0; }
    __syncthreads();
    const float* row = g + (size_t)blockIdx.x * m;
    uint32_t n = 0, nz = 0;
    constexpr int AT_ONCE = 4;
    for (int64_t j0 = 0; j0 < m; j0 += AT_ONCE * 256 * 1024) {   // 4 of every 1024 labels
        float v[AT_ONCE][4];
        bool in[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            const int64_t j = j0 + (u * 256 + (int)threadIdx.x) * 1024;
            in[u] = j + 4 <= m;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[u][q] = in[u] ? row[j + q] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
            n += in[u] ? 4u : 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) nz += v[u][q] != 0.f ? 1u : 0u;
        }
    }
    for (int o = 32; o > 0; o >>= 1) { n += __shfl_down(n, o); nz += __shfl_down(nz, o); }
    if ((threadIdx.x & 63) == 0) { atomicAdd(&seen, n); atomicAdd(&hit, nz); }
    __syncthreads();
    // the lists hold m/32 entries per instance: a sample twice as dense as that cannot fit
    if (threadIdx.x == 0) {
        // what the host reads before its next call: would lists have been worth trying?  (sample at most 1/64 nonzero)
        state[usl_nz_count_at(blockIdx.x)] = 0;
        look_done(state, seen >= 128 && (uint64_t)hit * 16 > seen, (uint64_t)hit * 64 > seen, gridDim.x, hint, serial);
    }
}

__global__ void __launch_bounds__(CG_NT)
k_compact_g(const float* __restrict__ g, int64_t m, uint32_t cap, uint32_t* __restrict__ state,
            int32_t* __restrict__ nz_lab, float* __restrict__ nz_val) {
    __shared__ uint32_t wave_total[CG_NT / 64];
    __shared__ uint32_t block_base;
    if (*reinterpret_cast<volatile uint32_t*>(state) != 0) return;   // the sample, or an earlier block, found g dense
    const int i = (int)(gridDim.y - 1 - blockIdx.y);   // the last rows first: behind a loss they were written last, and may still be in a cache (m = 500k, b = 256, squared-hinge step 1004 and 990 us)
    const int64_t j0 = (int64_t)blockIdx.x * CG_CHUNK;
    const float* row = g + (size_t)i * m;
    const bool vec = (m % 4 == 0) && ((uintptr_t)g % 16 == 0);
    float4 v[CG_PER / 4];
#pragma unroll
    for (int u = 0; u < CG_PER / 4; ++u) {
        const int64_t j = j0 + ((int64_t)u * CG_NT + threadIdx.x) * 4;
        if (vec && j + 4 <= m) {
            v[u] = *reinterpret_cast<const float4*>(row + j);
        } else {
            v[u].x = j < m ? row[j] : 0.f;         v[u].y = j + 1 < m ? row[j + 1] : 0.f;
            v[u].z = j + 2 < m ? row[j + 2] : 0.f; v[u].w = j + 3 < m ? row[j + 3] : 0.f;
        }
    }
    uint32_t cnt = 0;
#pragma unroll
    for (int u = 0; u < CG_PER / 4; ++u)
        cnt += (v[u].x != 0.f ? 1u : 0u) + (v[u].y != 0.f ? 1u : 0u) + (v[u].z != 0.f ? 1u : 0u) + (v[u].w != 0.f ? 1u : 0u);
    // places: prefix over the lanes of a wavefront, then over the wavefronts; one atomic per block reserves them
    uint32_t incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if ((int)(threadIdx.x & 63) >= o) incl += t;
    }
    if ((threadIdx.x & 63) == 63) wave_total[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < CG_NT / 64; ++q) {
        const uint32_t t = wave_total[q];
        if (q < (int)(threadIdx.x >> 6)) before += t;
        total += t;
    }
    if (total == 0) return;   // the same for every lane of the block
    if (threadIdx.x == 0) block_base = atomicAdd(&state[usl_nz_count_at(i)], total);
    __syncthreads();
    const uint32_t base = block_base;
    if (base + total > cap) {
        if (threadIdx.x == 0) atomicOr(&state[0], 1u);
        return;
    }
    uint32_t at = base + before + incl - cnt;
    int32_t* lab = nz_lab + (size_t)i * cap;
    float* val = nz_val + (size_t)i * cap;
#pragma unroll
    for (int u = 0; u < CG_PER / 4; ++u) {
        const int64_t j = j0 + ((int64_t)u * CG_NT + threadIdx.x) * 4;
        if (v[u].x != 0.f) { lab[at] = (int32_t)j; val[at] = v[u].x; ++at; }
        if (v[u].y != 0.f) { lab[at] = (int32_t)(j + 1); val[at] = v[u].y; ++at; }
        if (v[u].z != 0.f) { lab[at] = (int32_t)(j + 2); val[at] = v[u].z; ++at; }
        if (v[u].w != 0.f) { lab[at] = (int32_t)(j + 3); val[at] = v[u].w; ++at; }
    }
}

// The lists from the marks that forward left: a workgroup has 1024 words of an instance, counts and places them, and brings the gradients
// of the listed labels (4 to 64 bytes of memory each instead of the whole row: at m = 500k, b = 256 16 MB of marks for 512 MB of g).  One atomic
// a workgroup, in the instance's own line, reserves the places and counts the workgroups; the instance's last one knows its count, which is
// exact, so this is the look as well (k_probe_density).  k_before_forward or k_interleave cleared the lines.
// What bounds it is the chain of four trips to memory (marks, place, labels, gradients), so it is spread over the chip.  With one workgroup for an instance
// m = 1.5M, k = 16, b = 8, 1.6 % nonzero took 37 us, now 6.7 (the look and the pass over g 27); m = 3M, b = 8 69 and 8.2; m = 500k, k = 32, b = 256, 0.2 % nonzero
// 11.2 and 9.6 (116).
constexpr int LN_NT = 256, LN_PER = 4, LN_WORDS = LN_NT * LN_PER;
__global__ void __launch_bounds__(LN_NT)
k_list_nonzeros(const uint32_t* __restrict__ bits, int64_t words, const float* __restrict__ g, int64_t m, int b, uint32_t cap,
                uint32_t* __restrict__ state, int32_t* __restrict__ nz_lab, float* __restrict__ nz_val, uint32_t* __restrict__ hint, uint32_t serial) {
    typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // an instance's words begin anywhere
    __shared__ uint32_t wave_total[LN_NT / 64];
    __shared__ uint32_t block_base;
    const int i = (int)blockIdx.y, lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const uint32_t* row = bits + (size_t)i * words;
    const int64_t w0 = (int64_t)blockIdx.x * LN_WORDS + (int)threadIdx.x * LN_PER;
    uint32_t v[LN_PER], cnt = 0;
    if (w0 + LN_PER <= words) {
        const u32x4_any t = *reinterpret_cast<const u32x4_any*>(row + w0);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
        for (int u = 0; u < LN_PER; ++u) v[u] = w0 + u < words ? row[w0 + u] : 0u;
    }
#pragma unroll
    for (int u = 0; u < LN_PER; ++u) cnt += (uint32_t)__popc(v[u]);
    uint32_t incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wave_total[wave] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < LN_NT / 64; ++q) {
        const uint32_t t = wave_total[q];
        if (q < wave) before += t;
        total += t;
    }
    if (threadIdx.x == 0) {   // workgroups above, entries below
        const unsigned long long had = atomicAdd(reinterpret_cast<unsigned long long*>(state + usl_nz_count_at(i)), 1ull << 32 | total);
        block_base = (uint32_t)had;
        const uint32_t count = (uint32_t)had + total;
        if ((uint32_t)(had >> 32) + 1 == gridDim.x) look_done(state, count > cap, (uint64_t)count * 64 > (uint64_t)m, (uint32_t)b, hint, serial);
    }
    __syncthreads();
    const uint32_t base = block_base;
    if (base + total > cap) return;   // the same for all lanes; the look finds the count too large
    int32_t* lab = nz_lab + (size_t)i * cap + base;
    float* val = nz_val + (size_t)i * cap + base;
    uint32_t at = before + incl - cnt;
#pragma unroll
    for (int u = 0; u < LN_PER; ++u)
        for (uint32_t rest = v[u]; rest; rest &= rest - 1) lab[at++] = (int32_t)((w0 + u) * 32 + __ffs((int)rest) - 1);
    __syncthreads();   // the labels are written
    constexpr int AT_ONCE = 4;
    for (uint32_t e0 = threadIdx.x; e0 < total; e0 += LN_NT * AT_ONCE) {
        int32_t j[AT_ONCE];
        float z[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) j[u] = e0 + u * LN_NT < total ? lab[e0 + u * LN_NT] : 0;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) z[u] = e0 + u * LN_NT < total ? g[(size_t)i * m + j[u]] : 0.f;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u)
            if (e0 + u * LN_NT < total) val[e0 + u * LN_NT] = z[u];
    }
}

__global__ void k_new_state(uint32_t* state) {
    if (threadIdx.x < STATE_LINE) state[threadIdx.x] = 0;
}

// clears p[0..n) when the lists stand (state[0] == 0)
__global__ void k_zero_if_sparse(float* __restrict__ p, size_t n, const uint32_t* __restrict__ state) {
    if (*state != 0) return;
    const size_t stride = (size_t)gridDim.x * blockDim.x * 4;
    for (size_t f = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4; f < n; f += stride) {
        if (f + 4 <= n && ((uintptr_t)p % 16 == 0)) *reinterpret_cast<float4*>(p + f) = make_float4(0.f, 0.f, 0.f, 0.f);
        else for (size_t q = f; q < n && q < f + 4; ++q) p[q] = 0.f;
    }
}

// grad_W[j][t] += g * x[i][idx[j][t]] for every listed (i, j, g) and slot t.  grid (blocks, b): the blocks of one
// instance stride over its entries; an item is one (entry, slot) pair, so a row of grad_W gets k neighbouring atomics.
template <typename TS>
__global__ void __launch_bounds__(256)
k_bww_sparse(const TS* __restrict__ x, const int32_t* __restrict__ idx, const uint32_t* __restrict__ state,
             const int32_t* __restrict__ nz_lab, const float* __restrict__ nz_val, uint32_t cap,
             float* __restrict__ grad_W, int d, int k) {
    if (state[0] != 0) return;
    const int i = blockIdx.y;
    const uint64_t items = (uint64_t)state[usl_nz_count_at(i)] * (uint32_t)k;
    const int32_t* lab = nz_lab + (size_t)i * cap;
    const float* val = nz_val + (size_t)i * cap;
    const TS* row = x + (size_t)i * d;
    for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < items; e += (uint64_t)gridDim.x * 256) {
        const uint32_t q = (uint32_t)(e / (uint32_t)k);
        const uint32_t t = (uint32_t)(e - (uint64_t)q * (uint32_t)k);
        const size_t slot = (size_t)lab[q] * k + t;
        const float xv = usl_load_f32<TS>(row, (size_t)idx[slot]);
        if (xv != 0.f) unsafeAtomicAdd(grad_W + slot, val[q] * xv);   // activations after a ReLU are half zeros
    }
}

// grad_x[i][c] = sum over listed (j, g) of instance i and slots t with idx[j][t] == c of W[j][t] * g.
// One workgroup per (instance, slice of at most 32768 columns): the slice lives in LDS, starts at zero, takes
// the additions as LDS atomics and is written out once (the row is overwritten, as the dense path does).
constexpr int XS_NT = 1024, XS_COLS = 32768;
template <typename TS>
__global__ void __launch_bounds__(XS_NT)
k_bwi_sparse(const int32_t* __restrict__ idx, const TS* __restrict__ W, const uint32_t* __restrict__ state,
             const int32_t* __restrict__ nz_lab, const float* __restrict__ nz_val, uint32_t cap,
             float* __restrict__ grad_x, int d, int k) {
    extern __shared__ float acc[];
    if (state[0] != 0) return;
    const int i = blockIdx.y;
    const int c0 = blockIdx.x * XS_COLS;
    const int nc = min(XS_COLS, d - c0);
    for (int c = threadIdx.x; c < nc; c += XS_NT) acc[c] = 0.f;
    __syncthreads();
    const uint64_t items = (uint64_t)state[usl_nz_count_at(i)] * (uint32_t)k;
    const int32_t* lab = nz_lab + (size_t)i * cap;
    const float* val = nz_val + (size_t)i * cap;
    for (uint64_t e = threadIdx.x; e < items; e += XS_NT) {
        const uint32_t q = (uint32_t)(e / (uint32_t)k);
        const uint32_t t = (uint32_t)(e - (uint64_t)q * (uint32_t)k);
        const size_t slot = (size_t)lab[q] * k + t;
        const uint32_t c = (uint32_t)(idx[slot] - c0);
        if (c < (uint32_t)nc) unsafeAtomicAdd(&acc[c], val[q] * usl_load_f32<TS>(W, slot));
    }
    __syncthreads();
    float* dst = grad_x + (size_t)i * d + c0;
    for (int c = threadIdx.x; c < nc; c += XS_NT) dst[c] = acc[c];
}

}  // namespace

// Labels a list holds at most: an instance with more nonzeros than 1/32 of the labels makes the gradient "dense".
static uint32_t list_capacity(const usl_ctx* c) {
    const int64_t cap = c->m / 32;
    return (uint32_t)(cap < 64 ? 64 : cap);
}

bool usl_sparse_supported(const usl_ctx* c) {
    // lists of max_b * m/32 entries: not worth their memory for tiny layers, and the dense kernels win there anyway
    return c->m >= 65536 && (size_t)c->max_b * list_capacity(c) * 8 <= ((size_t)4 << 30);
}

// Does the context expect a gradient that is almost all zeros?  Reads, without waiting, what the looks of
// earlier calls reported (whichever of them have finished by now).
bool usl_sparse_expected(usl_ctx* c) {
    if (c->hint_host) {
        const uint32_t h = *(const volatile uint32_t*)c->hint_host, serial = h >> 1, dense = h & 1u;
        if (serial != c->hint_seen) {
            c->hint_seen = serial;
            c->sparse_streak = dense ? 0 : c->sparse_streak + 1;
        }
    }
    bool expected = c->sparse_streak >= 2;
    if (const char* e = getenv("USL_TUNE_SPARSE")) {
        if (!strcmp(e, "always")) expected = true;
        else if (!strcmp(e, "never")) expected = false;
    }
    return expected;
}

static usl_status state_ready(usl_ctx* c) {
    if (!c->hint_host) {
        USL_HIP(c, hipHostMalloc((void**)&c->hint_host, 64, hipHostMallocMapped));
        c->hint_host[0] = 1;
        USL_HIP(c, hipHostGetDevicePointer((void**)&c->hint_dev, c->hint_host, 0));
    }
    if (c->nz_state) return USL_OK;
    USL_TRY(usl_reserve(c, (void**)&c->nz_state, &c->nz_state_cap, usl_nz_count_at(c->max_b) * 4));
    hipLaunchKernelGGL(k_new_state, dim3(1), dim3(64), 0, c->stream, c->nz_state);
    return usl_check_launch(c, "state of the nonzeros' lists");
}
static usl_status lists_ready(usl_ctx* c) {
    const size_t bytes = (size_t)c->max_b * list_capacity(c) * 4;
    USL_TRY(usl_reserve(c, (void**)&c->nz_lab, &c->nz_lab_cap, bytes));
    return usl_reserve(c, (void**)&c->nz_val, &c->nz_val_cap, bytes);
}

// Looks at g[b][m] and, if the context has reason to expect a gradient that is almost all zeros, builds the
// lists of its nonzeros.  Every call enqueues the sample look (a few microseconds), whose verdict reaches the host
// through two pinned words that the NEXT calls read without waiting: after two such looks in a row that found
// the sample sparse the lists are tried, and the first look that finds it dense ends that.  A gradient that turns
// sparse is therefore handled by the dense kernels for two more calls, one that turns dense by the gated dense
// kernels once -- never wrongly, and a steadily dense gradient (binary cross-entropy) pays for the sample only.
// *gate: NULL = only the dense kernels run this time; else the device word that is 0 when the lists stand and 1
// when the dense kernels (which are then enqueued behind the gate) have to do the work.
// USL_TUNE_SPARSE=always / never overrides the expectation (tests, profiling).
usl_status usl_sparse_compact(usl_ctx* c, const float* g, int32_t b, const uint32_t** gate) {
    const uint32_t cap = list_capacity(c);
    *gate = nullptr;
    USL_TRY(state_ready(c));
    const bool try_lists = usl_sparse_expected(c);
    hipLaunchKernelGGL(k_probe_density, dim3((unsigned)b), dim3(256), 0, c->stream, g, c->m, c->nz_state, c->hint_dev,
                       ++c->probe_serial);
    if (!try_lists) return usl_check_launch(c, "gradient sample");
    USL_TRY(lists_ready(c));
    dim3 grid((unsigned)((c->m + CG_CHUNK - 1) / CG_CHUNK), (unsigned)b);
    hipLaunchKernelGGL(k_compact_g, grid, dim3(CG_NT), 0, c->stream, g, c->m, cap, c->nz_state, c->nz_lab, c->nz_val);
    *gate = c->nz_state;
    return usl_check_launch(c, "gradient compaction");
}

usl_status usl_sparse_marks_ready(usl_ctx* c) {
    USL_TRY(state_ready(c));
    return usl_reserve(c, (void**)&c->nz_bits, &c->nz_bits_cap, (size_t)c->max_b * usl_sparse_mark_words(c) * 4);
}

usl_status usl_sparse_lists(usl_ctx* c, const float* g, int32_t b, const uint32_t** gate) {
    USL_TRY(lists_ready(c));
    const int64_t words = (int64_t)usl_sparse_mark_words(c);
    hipLaunchKernelGGL(k_list_nonzeros, dim3((unsigned)((words + LN_WORDS - 1) / LN_WORDS), (unsigned)b), dim3(LN_NT), 0, c->stream, c->nz_bits, words, g,
                       c->m, (int)b, list_capacity(c), c->nz_state, c->nz_lab, c->nz_val, c->hint_dev, ++c->probe_serial);
    *gate = c->nz_state;
    return usl_check_launch(c, "lists of the marked gradients");
}

usl_status usl_sparse_backward_weight(usl_ctx* c, const void* x, const int32_t* idx, float* grad_W, int32_t b, bool cleared) {
    const uint32_t cap = list_capacity(c);
    const size_t N = (size_t)c->m * c->k;
    if (!cleared) hipLaunchKernelGGL(k_zero_if_sparse, dim3(c->num_cu * 8), dim3(256), 0, c->stream, grad_W, N, c->nz_state);
    dim3 grid(64, (unsigned)b);
    if (c->storage == USL_F32)
        hipLaunchKernelGGL(k_bww_sparse<float>, grid, dim3(256), 0, c->stream, (const float*)x, idx, c->nz_state,
                           c->nz_lab, c->nz_val, cap, grad_W, c->d, c->k);
    else
        hipLaunchKernelGGL(k_bww_sparse<uint16_t>, grid, dim3(256), 0, c->stream, (const uint16_t*)x, idx, c->nz_state,
                           c->nz_lab, c->nz_val, cap, grad_W, c->d, c->k);
    return usl_check_launch(c, "backward_weight over the nonzero gradients");
}

usl_status usl_sparse_backward_input(usl_ctx* c, const int32_t* idx, const void* W, float* grad_x, int32_t b) {
    const uint32_t cap = list_capacity(c);
    const size_t lds = (size_t)(c->d < XS_COLS ? c->d : XS_COLS) * 4;
    dim3 grid((unsigned)((c->d + XS_COLS - 1) / XS_COLS), (unsigned)b);
    if (c->storage == USL_F32) {
        USL_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(k_bwi_sparse<float>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(k_bwi_sparse<float>, grid, dim3(XS_NT), lds, c->stream, idx, (const float*)W, c->nz_state,
                           c->nz_lab, c->nz_val, cap, grad_x, c->d, c->k);
    } else {
        USL_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(k_bwi_sparse<uint16_t>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(k_bwi_sparse<uint16_t>, grid, dim3(XS_NT), lds, c->stream, idx, (const uint16_t*)W,
                           c->nz_state, c->nz_lab, c->nz_val, cap, grad_x, c->d, c->k);
    }
    return usl_check_launch(c, "backward_input over the nonzero gradients");
}
