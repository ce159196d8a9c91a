// Forward product (Algorithm 1) and weight gradient (Algorithm 3) of the uniformly-sparse layer: the choice of the
// kernel and its shape, the interleaved copy of the activations, and the kernels for shapes without a register-resident
// form.  The register-resident kernels themselves are in k_products_common.h.
#include <stdlib.h>

#include "k_products.h"
#include "k_products_common.h"
#include "k_count.h"
#include "k_topk.h"

using namespace usl_products;

namespace {

// ---- any k, any d --------------------------------------------------------------------------------------------

struct TileGeom {
    int part_cols;      // columns per slice of a row
    int nparts;         // slices per row
    int inst_per_group; // instances handled by one blockIdx.y
    int vec_ok;         // 16-byte copies allowed
};

// n elements from global memory into LDS, 16 bytes at a time where the alignment allows it
template <typename TS, int NT>
__device__ __forceinline__ void stage(const TS* __restrict__ src, TS* __restrict__ lds, int n, bool vec_ok) {
    if (vec_ok) {
        const int nv = (int)((size_t)n * sizeof(TS) / 16);
        for (int v = threadIdx.x; v < nv; v += NT) reinterpret_cast<uint4*>(lds)[v] = reinterpret_cast<const uint4*>(src)[v];
    } else {
        for (int c = threadIdx.x; c < n; c += NT) lds[c] = src[c];
    }
}
__device__ __forceinline__ float lds_val(const float* row, uint32_t c) { return row[c]; }
__device__ __forceinline__ float lds_val(const uint16_t* row, uint32_t c) { return usl_bf16_to_f32(row[c]); }

// any k, any d: one thread per label, idx / W re-read from global memory for every instance
template <int NT, typename TS>
__global__ void __launch_bounds__(NT)
k_forward_generic(const TS* __restrict__ x, const int32_t* __restrict__ idx,
                  const TS* __restrict__ W, float* __restrict__ out, int64_t m, int d, int k, int b,
                  TileGeom tg) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    TS* lds = reinterpret_cast<TS*>(lds_raw);
    const int64_t j = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t jj = j < m ? j : m - 1;
    const int i_begin = blockIdx.y * tg.inst_per_group;
    const int i_end = min(b, i_begin + tg.inst_per_group);
    for (int i = i_begin; i < i_end; ++i) {
        float acc = 0.f;
        for (int part = 0; part < tg.nparts; ++part) {
            const int c0 = part * tg.part_cols;
            const uint32_t cols = (uint32_t)min(tg.part_cols, d - c0);
            __syncthreads();
            stage<TS, NT>(x + (size_t)i * d + c0, lds, (int)cols, tg.vec_ok);
            __syncthreads();
            for (int t = 0; t < k; ++t) {
                const uint32_t c = (uint32_t)idx[jj * k + t] - (uint32_t)c0;
                if (c < cols) acc = fmaf(usl_load_f32<TS>(W, (size_t)(jj * k + t)), lds_val(lds, c), acc);
            }
        }
        if (j < m) out[(size_t)i * m + j] = acc;
    }
}

// any k, any d: one thread per connection
template <int NT, typename TS, bool ATOMIC>
__global__ void __launch_bounds__(NT)
k_backward_weight_generic(const float* __restrict__ g, const TS* __restrict__ x,
                          const int32_t* __restrict__ idx, float* __restrict__ grad_W, int64_t m,
                          int d, int k, int b, TileGeom tg) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    TS* lds = reinterpret_cast<TS*>(lds_raw);
    const int64_t N = m * k;
    const int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t ee = e < N ? e : N - 1;
    const int64_t j = ee / k;
    const uint32_t col = (uint32_t)idx[ee];
    const int i_begin = blockIdx.y * tg.inst_per_group;
    const int i_end = min(b, i_begin + tg.inst_per_group);
    float acc = 0.f;
    for (int i = i_begin; i < i_end; ++i) {
        const float gv = g[(size_t)i * m + j];
        for (int part = 0; part < tg.nparts; ++part) {
            const int c0 = part * tg.part_cols;
            const uint32_t cols = (uint32_t)min(tg.part_cols, d - c0);
            __syncthreads();
            stage<TS, NT>(x + (size_t)i * d + c0, lds, (int)cols, tg.vec_ok);
            __syncthreads();
            const uint32_t c = col - (uint32_t)c0;
            if (c < cols) acc = fmaf(gv, lds_val(lds, c), acc);
        }
    }
    if (e < N) {
        if (ATOMIC) unsafeAtomicAdd(grad_W + e, acc);
        else grad_W[e] = acc;
    }
}

// out[e] = part[0][e] + part[1][e] + ...: the partial weight gradients of a split batch, added in a fixed order.
// n rounded up to a multiple of 4 elements apart; out 16-byte aligned.
__global__ void k_sum_parts(const float* __restrict__ part, int groups, size_t n, size_t stride, float* __restrict__ out,
                            const uint32_t* __restrict__ gate) {
    if (gate && *gate == 0) return;
    size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x, nv = (n + 3) / 4;
    for (; v < nv; v += step) {
        float4 a = reinterpret_cast<const float4*>(part)[v];
        for (int q = 1; q < groups; ++q) {
            const float4 t = reinterpret_cast<const float4*>(part + (size_t)q * stride)[v];
            a.x += t.x; a.y += t.y; a.z += t.z; a.w += t.w;
        }
        if (v * 4 + 4 <= n) {
            reinterpret_cast<float4*>(out)[v] = a;
        } else {
            const float r[4] = {a.x, a.y, a.z, a.w};
            for (size_t e = v * 4; e < n; ++e) out[e] = r[e - v * 4];
        }
    }
}

__global__ void k_fill_zero(float* __restrict__ p, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t s = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += s) p[i] = 0.f;
}

// Sets the bits of the targets (usl_ctx::tgt_bits).  Wavefront q of n takes instances q, q + n, ...  The kernel that ends the step
// takes them back (step_end).
constexpr int MARK_WAVES = 4;   // of a block of 256 lanes
__device__ __forceinline__ void mark_targets(const usl_targets& t, int q, int n) {
    for (int i = q; i < t.b; i += n) {
        const int64_t p1 = t.off[i + 1];
        for (int64_t p = t.off[i] + (threadIdx.x & 63); p < p1; p += 64) {
            const int64_t j = t.lab[p];
            if (j >= 0 && j < t.m) atomicOr(t.bits + (size_t)(i >> 5) * t.m + j, 1u << (i & 31));
        }
    }
}
// What a step needs before forward: the targets marked, the fingerprint of idx compared for the backward product where lists stand
// (a launch of its own takes 4 to 8 us), the counts of the nonzeros' lists cleared where forward marks the nonzeros.  Done by block `at` of n blocks of 256 lanes.
struct Before {
    usl_targets targets;      // off = nullptr: nothing to do
    const uint32_t* idx;      // nullptr: nothing to compare
    size_t n_words;
    uint64_t* print;
    uint32_t* nz_state;       // nullptr, or whose instances' counts are to be cleared (k_list_nonzeros)
    __host__ __device__ int print_blocks() const { return idx ? USL_PRINT_SUMS / MARK_WAVES : 0; }
    int blocks() const { return print_blocks() + (targets.b + MARK_WAVES - 1) / MARK_WAVES; }
};
__device__ __forceinline__ void before_forward(const Before& w, int at, int n) {
    const int first = w.print_blocks(), wave = (int)(threadIdx.x >> 6);
    if (at < first) usl_idx_fingerprint_sums<1>(w.idx, w.n_words, w.print, USL_PRINT_BOTH_PRODUCTS, 0, at * MARK_WAVES + wave, 0);
    if (at < first) return;
    const int q = (at - first) * MARK_WAVES + wave, waves = (n - first) * MARK_WAVES;
    if (w.nz_state && (threadIdx.x & 63) == 0)
        for (int i = q; i < w.targets.b; i += waves) *reinterpret_cast<uint64_t*>(w.nz_state + usl_nz_count_at(i)) = 0;
    mark_targets(w.targets, q, waves);
}
__global__ void __launch_bounds__(256)
k_before_forward(Before w) { before_forward(w, (int)blockIdx.x, (int)gridDim.x); }

// xi[group][column][Q instances] from x[b][d]; columns past d and instances past b are zeros.
// grid (blocks of 256 columns, groups); in a training step some rows of blocks more, which mark the targets and compare the
// fingerprint (a launch of its own takes 5 us): from row `row0` on
template <typename TS, int Q>
__global__ void __launch_bounds__(256)
k_interleave(const TS* __restrict__ x, TS* __restrict__ xi, int b, int d, int cols, Before before, int row0) {
    const int c = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;
    if (before.targets.off && g >= row0) {
        before_forward(before, (int)((g - row0) * gridDim.x + blockIdx.x), (int)((gridDim.y - row0) * gridDim.x));
        return;
    }
    if (c >= cols) return;
    TS v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = c < d && g * Q + q < b ? x[(size_t)(g * Q + q) * d + c] : (TS)0;
    TS* to = xi + ((size_t)g * cols + c) * Q;
    typedef typename Unit<TS, Q>::T U;
    U u;
    __builtin_memcpy(&u, v, sizeof(U));
    *reinterpret_cast<U*>(to) = u;
}

// v of another lane: a permutation within 16 lanes by the vector unit
template <int CTRL>
__device__ __forceinline__ float moved(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true)); }

// ---- forward of one group of instances (b <= Q) ----------------------------------------------------------------
// With one row of activations nothing is reused, and bringing idx and W into registers label by label only delays them:
// here they stream.  A lane takes four neighbouring slots (16 bytes of idx, 16 or 8 of W, coalesced), gathers their
// activations from the row in LDS, and the LPL lanes of a label add up their sums.  LPL rounds give a wavefront the sums of 64 consecutive labels, one per lane (fewer rounds and labels where a
// small layer would leave wavefronts without any; always an even number).  Bound by the stream of idx
// and W: m = 500k, k = 32, b = 1: 128 MB in 21.6 us, 5.9 TB/s (29.6 us label by label).  Not for rows that exceed LDS (gathers
// from L2 instead took 498 us at m = 3M, d = 65536, where the two halves of the label-by-label form take about 300).
// VEC: k is a multiple of 4.
// AHEAD: rounds in flight, a divisor of `rounds`.  Four where there is one instance (four spill where there are four): with two,
// and the sums of a label's lanes through LDS, the scores of m = 500k took 0.8 us longer.
// BEST, one instance: the kk best labels, by keys (k_topk.h).  Each wavefront finds its own from its lanes' scores (the first few in registers, which then go
// nowhere else; those of more turns read back from out), then the workgroup its own, which go to cand[workgroup][kk] (0 where there are fewer).  With top_lab the workgroup
// that comes last may merge them (last_one_merges): candidates and the count of workgroups go by atomics of the device's scope, so no fence writes back an L2.  What it reads
// is what was written: a store of that scope passes its XCD's L2 and is there when the wait behind it ends, before the workgroup adds to the count; the loads are asked
// for after the addition has returned and a barrier, and pass the L2 too, so that no older line answers them.  (With a launch of its own for the merge and the scores
// read back for it usl_predict took 35.5 us at m = 500k, d = 32k, k = 32, so 33.0; m = 5000, d = 64, k = 8 10.6 and 8.6.)  A kernel of its own:
// it takes 10 more registers, with which a compute unit holds one workgroup of 1024 in the place of two where k is no multiple of 4.  Where it is used:
// best_from_forward.  (Several instances one after the other took longer than a kernel over the scores: m = 31k, d = 1k, k = 32, b = 4 16.2 and 26.6.)
constexpr int FEW_HELD = 4;   // turns whose scores, or candidates, a lane keeps in registers
template <int LPL, typename TS, int Q, bool VEC, int AHEAD, bool BEST>
__global__ void __launch_bounds__(1024)
k_forward_few(const char* __restrict__ xi, const int32_t* __restrict__ idx, const TS* __restrict__ W, float* __restrict__ out,
              int64_t m, int k, int b, int row_bytes, int rounds, int kk, uint64_t* __restrict__ cand, uint32_t* __restrict__ done,
              int32_t* __restrict__ top_lab, float* __restrict__ top_val) {
    typedef typename Unit<TS, Q>::T U;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const uint32_t lds0 = lds_base(lds_raw);
    const int nw = (int)blockDim.x >> 6;
    stage_async(xi, lds0, row_bytes, (int)threadIdx.x, (int)blockDim.x);
    const int lane = threadIdx.x & 63, sub = lane & (LPL - 1), t = sub * 4;
    const int64_t waves = (int64_t)gridDim.x * nw;
    const int64_t w0 = (int64_t)blockIdx.x * nw + (threadIdx.x >> 6);
    struct Piece { uint32_t c[4]; uint32_t w[sizeof(TS) == 4 ? 4 : 2]; };
    // What a slot that does not exist reads: a unit of zeros behind the row.  (Weight 0 times a real activation would turn
    // an infinity into NaN for labels that have no connection to it.)
    const uint32_t nowhere = (uint32_t)row_bytes / (uint32_t)sizeof(U);
    if (threadIdx.x < 4) reinterpret_cast<uint32_t*>(lds_raw)[(uint32_t)row_bytes / 4 + threadIdx.x] = 0u;
    // the four slots of this lane in round r of the wavefront's 64 labels
    auto fetch = [&](int64_t j0, int r, Piece& p) {
        const int64_t j = j0 + r * (64 / LPL) + lane / LPL;
        const bool in = j < m && t < k;
        if (VEC) {
            uint4 c = make_uint4(nowhere, nowhere, nowhere, nowhere);
            if (in) c = *reinterpret_cast<const uint4*>(idx + j * k + t);
            p.c[0] = c.x; p.c[1] = c.y; p.c[2] = c.z; p.c[3] = c.w;
            if constexpr (sizeof(TS) == 4) {
                uint4 w = make_uint4(0, 0, 0, 0);
                if (in) w = *reinterpret_cast<const uint4*>(W + j * k + t);
                p.w[0] = w.x; p.w[1] = w.y; p.w[2] = w.z; p.w[3] = w.w;
            } else {
                uint2 w = make_uint2(0, 0);
                if (in) w = *reinterpret_cast<const uint2*>(W + j * k + t);
                p.w[0] = w.x; p.w[1] = w.y;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool inq = j < m && t + q < k;
                p.c[q] = inq ? (uint32_t)idx[j * k + t + q] : nowhere;
                if constexpr (sizeof(TS) == 4) p.w[q] = inq ? __float_as_uint(W[j * k + t + q]) : 0u;
                else if (q & 1) p.w[q / 2] |= inq ? (uint32_t)W[j * k + t + q] << 16 : 0u;
                else p.w[q / 2] = inq ? (uint32_t)W[j * k + t + q] : 0u;
            }
        }
    };
    auto activation = [&](uint32_t col) -> U { return lds_read<U>(lds0 + col * (uint32_t)sizeof(U)); };
    auto dot4 = [&](const Piece& p, float (&acc)[Q]) {
        U v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = activation(p.c[q]);
        if constexpr (sizeof(TS) == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float w = __uint_as_float(p.w[q]);
                if constexpr (Q == 1) acc[0] = fmaf(w, v[q], acc[0]);
                else {
#pragma unroll
                    for (int i = 0; i < Q; ++i) acc[i] = fmaf(w, v[q][i], acc[i]);
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                if constexpr (Q == 1) acc[0] = dot2((uint32_t)v[q] | ((uint32_t)v[q + 1] << 16), p.w[q / 2], acc[0]);
                else if constexpr (Q == 2) {
                    acc[0] = dot2(join_lo(v[q], v[q + 1]), p.w[q / 2], acc[0]);
                    acc[1] = dot2(join_hi(v[q], v[q + 1]), p.w[q / 2], acc[1]);
                } else {
                    acc[0] = dot2(join_lo(v[q].x, v[q + 1].x), p.w[q / 2], acc[0]);
                    acc[1] = dot2(join_hi(v[q].x, v[q + 1].x), p.w[q / 2], acc[1]);
                    acc[2] = dot2(join_lo(v[q].y, v[q + 1].y), p.w[q / 2], acc[2]);
                    acc[3] = dot2(join_hi(v[q].y, v[q + 1].y), p.w[q / 2], acc[3]);
                }
            }
        }
    };
    Piece p[AHEAD];
    const int per = rounds * (64 / LPL);   // labels of a wavefront's turn
    if (w0 * per < m) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) fetch(w0 * per, a, p[a]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    constexpr int HELD = FEW_HELD;
    const int64_t step = waves * per, turns = w0 * per < m ? (m - w0 * per + step - 1) / step : 0;
    float kept[BEST ? HELD : 1] = {};
    int turn = 0;
    for (int64_t wv = w0; wv * per < m; wv += waves, ++turn) {
        const int64_t j0 = wv * per, jn = (wv + waves) * per;
        float sum[Q] = {};   // of label j0 + (lane % LPL) * (64 / LPL) + lane / LPL
#pragma unroll 1
        for (int r0 = 0; r0 < rounds; r0 += AHEAD) {
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) {
                const int r = r0 + a;
                float acc[Q] = {};
                dot4(p[a], acc);
                if (r + AHEAD < rounds) fetch(j0, r + AHEAD, p[a]);
                else fetch(jn, a, p[a]);
#pragma unroll
                for (int i = 0; i < Q; ++i) {   // (lanes that have been added up are alike: a mirror reaches the others as well)
                    if (LPL > 1) acc[i] += moved<0xB1>(acc[i]);    // quads 1 0 3 2
                    if (LPL > 2) acc[i] += moved<0x4E>(acc[i]);    // quads 2 3 0 1
                    if (LPL > 4) acc[i] += moved<0x141>(acc[i]);   // 8 lanes, mirrored
                    if (LPL > 8) acc[i] += moved<0x140>(acc[i]);   // 16
                }
#pragma unroll
                for (int i = 0; i < Q; ++i) sum[i] = sub == r ? acc[i] : sum[i];
            }
        }
        const int64_t j = j0 + sub * (64 / LPL) + lane / LPL;
        if (sub < rounds && j < m && (!BEST || turns > HELD)) {
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (i < b) out[(size_t)i * m + j] = sum[i];
        }
        if constexpr (BEST) {
#pragma unroll
            for (int q = 0; q < HELD; ++q) kept[q] = turn == q ? sum[0] : kept[q];
        }
    }
    if constexpr (!BEST) return;
    uint64_t* list = reinterpret_cast<uint64_t*>(lds_raw);
    auto label_of = [&](int64_t at) -> int64_t {   // m: none
        const int64_t j = w0 * per + at * step + sub * (64 / LPL) + lane / LPL;
        return at < turns && sub < rounds && j < m ? j : m;
    };
    // the kk largest keys of the workgroup's lanes, the r-th in lane r of wavefront 0; more(prev): a lane's largest below prev beside those held
    auto largest = [&](const uint64_t (&held)[HELD], auto more) -> uint64_t {
        __syncthreads();   // LDS is no longer read
        uint64_t prev = ~0ull, found = 0;
        for (int r = 0; r < kk; ++r) {
            uint64_t best = more(prev);
#pragma unroll
            for (int q = 0; q < HELD; ++q)
                if (held[q] < prev && held[q] > best) best = held[q];
            prev = wave_max(best);
            if (lane == 0) list[(threadIdx.x >> 6) * kk + r] = prev;
        }
        __syncthreads();
        if (threadIdx.x >= 64) return 0;
        const int n = nw * kk;   // at most 16 * 32
        uint64_t mine[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) mine[q] = q * 64 + lane < n ? list[q * 64 + lane] : 0ull;
        prev = ~0ull;
        for (int r = 0; r < kk; ++r) {
            uint64_t best = 0;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (mine[q] < prev && mine[q] > best) best = mine[q];
            prev = wave_max(best);
            if (lane == r) found = prev;
        }
        return found;
    };
    uint64_t held[HELD];
#pragma unroll
    for (int q = 0; q < HELD; ++q) held[q] = label_of(q) < m ? score_key(kept[BEST ? q : 0], (uint32_t)label_of(q)) : 0ull;
    const uint64_t own = largest(held, [&](uint64_t prev) {
        uint64_t best = 0;
        for (int64_t at = HELD; at < turns; ++at) {
            const int64_t j = label_of(at);
            const uint64_t key = j < m ? score_key(out[j], (uint32_t)j) : 0ull;
            if (key < prev && key > best) best = key;
        }
        return best;
    });
    uint64_t* to = cand + (size_t)blockIdx.x * kk + lane;
    if (!top_lab) {
        if ((int)threadIdx.x < kk) *to = own;
        return;
    }
    uint32_t* last = reinterpret_cast<uint32_t*>(lds_raw) + 16 * 32 * 2;   // behind the lists
    if (threadIdx.x < 64) {
        if (lane < kk) __hip_atomic_store(to, own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the candidates are there before the count says so
        const uint32_t share = usl_count_share(blockIdx.x, gridDim.x);
        if (lane == 0) *last = usl_count_is_last(__hip_atomic_fetch_add(done, share, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), share) ? 1u : 0u;
    }
    __syncthreads();
    if (!*last) return;
    const uint32_t n = gridDim.x * (uint32_t)kk;   // HELD to a lane at most
#pragma unroll
    for (int q = 0; q < HELD; ++q) {
        const uint32_t at = (uint32_t)q * blockDim.x + threadIdx.x;
        held[q] = at < n ? __hip_atomic_load(cand + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
    }
    const uint64_t top = largest(held, [](uint64_t) -> uint64_t { return 0; });
    if ((int)threadIdx.x < kk) {
        top_lab[lane] = key_label(top);
        top_val[lane] = key_score(top);
    }
}

// out[i][:] once more, slot by slot, for the instances whose activation 0 is not finite (see pads_with_column_0): nearly
// always none, and a block that finds none leaves.  A lane per label.
template <typename TS>
__global__ void __launch_bounds__(256)
k_forward_again(const TS* __restrict__ x, const int32_t* __restrict__ idx, const TS* __restrict__ W, float* __restrict__ out, int64_t m, int d,
                int k, int b) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    for (int i0 = 0; i0 < b; i0 += 64) {
        const float v = i0 + lane < b ? usl_load_f32<TS>(x, (size_t)(i0 + lane) * d) : 0.f;
        uint64_t todo = __ballot((__float_as_uint(v) & 0x7F800000u) == 0x7F800000u);
        for (; todo; todo &= todo - 1) {
            const int i = i0 + __ffsll((unsigned long long)todo) - 1;
            if (j >= m) continue;
            float acc = 0.f;
            for (int t = 0; t < k; ++t) acc = fmaf(usl_load_f32<TS>(W, (size_t)j * k + t), usl_load_f32<TS>(x, (size_t)i * d + idx[j * k + t]), acc);
            out[(size_t)i * m + j] = acc;
        }
    }
}

inline size_t max_sz(size_t a, size_t b) { return a > b ? a : b; }

template <typename KERNEL>
usl_status allow_lds(usl_ctx* c, KERNEL kern, size_t bytes) {
    if (bytes > 65536)
        USL_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    return USL_OK;
}

TileGeom plan_generic(const usl_ctx* c, int esize, int b, int64_t nblk, const void* x, size_t* lds_bytes, int* groups) {
    TileGeom tg;
    const size_t row_bytes = (size_t)c->d * esize;
    tg.vec_ok = (row_bytes % 16 == 0) && (((uintptr_t)x) % 16 == 0);
    tg.part_cols = row_bytes <= (size_t)USL_ROW_LDS_BYTES ? c->d : USL_ROW_LDS_BYTES / esize;
    tg.nparts = (c->d + tg.part_cols - 1) / tg.part_cols;
    // enough workgroups to fill the chip: split the batch when there are few label blocks
    const int64_t want = (int64_t)c->num_cu * (row_bytes > 40960 ? 1 : 2);
    int G = 1;
    if (nblk * 4 < want * 3) {
        G = (int)((want + nblk - 1) / nblk);
        if (G > b) G = b;
    }
    tg.inst_per_group = (b + G - 1) / G;
    *groups = (b + tg.inst_per_group - 1) / tg.inst_per_group;
    *lds_bytes = ((size_t)tg.part_cols * esize + 15) & ~(size_t)15;
    return tg;
}

template <typename TS>
usl_status run_forward_generic(usl_ctx* c, const void* x, const int32_t* idx, const void* W, float* out, int b) {
    constexpr int NT = 256;
    const int64_t nblk = (c->m + NT - 1) / NT;
    size_t lds;
    int G;
    TileGeom tg = plan_generic(c, (int)sizeof(TS), b, nblk, x, &lds, &G);
    USL_TRY(allow_lds(c, k_forward_generic<NT, TS>, lds));
    hipLaunchKernelGGL((k_forward_generic<NT, TS>), dim3((unsigned)nblk, (unsigned)G), dim3(NT), lds,
                       c->stream, (const TS*)x, idx, (const TS*)W, out, c->m, c->d, c->k, b, tg);
    return usl_check_launch(c, "forward (generic)");
}

template <typename TS>
usl_status run_backward_weight_generic(usl_ctx* c, const float* g, const void* x, const int32_t* idx, float* grad_W, int b) {
    constexpr int NT = 256;
    const int64_t N = c->m * (int64_t)c->k;
    const int64_t nblk = (N + NT - 1) / NT;
    size_t lds;
    int G;
    TileGeom tg = plan_generic(c, (int)sizeof(TS), b, nblk, x, &lds, &G);
    dim3 grid((unsigned)nblk, (unsigned)G);
    if (G > 1) {
        hipLaunchKernelGGL(k_fill_zero, dim3(c->num_cu * 4), dim3(256), 0, c->stream, grad_W, (size_t)N);
        USL_TRY(allow_lds(c, k_backward_weight_generic<NT, TS, true>, lds));
        hipLaunchKernelGGL((k_backward_weight_generic<NT, TS, true>), grid, dim3(NT), lds, c->stream,
                           g, (const TS*)x, idx, grad_W, c->m, c->d, c->k, b, tg);
    } else {
        USL_TRY(allow_lds(c, k_backward_weight_generic<NT, TS, false>, lds));
        hipLaunchKernelGGL((k_backward_weight_generic<NT, TS, false>), grid, dim3(NT), lds, c->stream,
                           g, (const TS*)x, idx, grad_W, c->m, c->d, c->k, b, tg);
    }
    return usl_check_launch(c, "backward_weight (generic)");
}

// ---- the register-resident kernels ---------------------------------------------------------------------------

// tuning and test aids: workgroup shape (0 .. 3) and parts of the batch instead of the estimate's choice; parts of the batch (up to
// as many as it has groups) for the last half of forward's blocks of labels, whatever the rounds
int tune_shape() { const char* e = getenv("USL_TUNE_SHAPE"); return e && *e ? atoi(e) : -1; }
int tune_split() { const char* e = getenv("USL_TUNE_SPLIT"); return e && *e ? atoi(e) : 0; }
// labels of a block (rounded up to 32s, at most what its lanes take)
int tune_labels() { const char* e = getenv("USL_TUNE_LABELS"); return e && *e ? atoi(e) : 0; }
int tune_tail() { const char* e = getenv("USL_TUNE_TAIL"); return e && *e ? atoi(e) : 0; }

// How the activations of this layer are laid out for the kernels (k_products_common.h): instances per group, bytes
// from row to row, whether x itself is that layout.
struct Layout {
    int Q, K, row_bytes, zero_col;
    bool halves, copy;
};

int padded_fan_in(int k) { return k <= 32 ? (k + 7) / 8 * 8 : k <= 48 ? 48 : 64; }

// Q from the width of a row: the largest group whose row of units fits LDS, and no larger than the batch needs.
Layout layout_of(const usl_ctx* c, int b, const void* x) {
    Layout L;
    const int es = c->storage == USL_F32 ? 4 : 2;
    L.K = padded_fan_in(c->k);
    L.zero_col = 0;
    L.halves = L.copy = false;
    for (L.Q = b >= 3 ? 4 : b; L.Q >= 1; L.Q >>= 1) {
        const int unit = L.Q * es, per = 16 / unit;   // columns in 16 bytes
        L.copy = L.Q > 1 || L.K > c->k || (size_t)c->d * es % 16 != 0 || (uintptr_t)x % 16 != 0;
        const int cols = ((c->d + (L.K > c->k ? 1 : 0)) + per - 1) / per * per;   // a column of zeros for padding slots
        L.row_bytes = cols * unit;
        L.zero_col = L.K > c->k ? c->d : 0;
        if (L.row_bytes <= ROW_LDS_MAX && cols <= 65536) return L;
    }
    // a float32 row in two halves, or the widest bfloat16 row with padded fan-in
    const bool zeros = L.K > c->k && c->d < 65536;
    L.Q = 1;
    L.zero_col = zeros ? c->d : 0;
    L.copy = zeros || (size_t)c->d * es % 16 != 0 || (uintptr_t)x % 16 != 0;
    L.row_bytes = ((c->d + (zeros ? 1 : 0)) * es + 15) / 16 * 16;
    L.halves = L.row_bytes > ROW_LDS_MAX;
    return L;
}

// At d = 65536 a column of zeros would be number 65536, which does not fit the 16 bits of a packed index: padding slots read
// column 0 there, with weight 0, and instances whose activation 0 is not finite are done again (k_forward_again).
bool pads_with_column_0(const usl_ctx* c, const Layout& L) { return L.K > c->k && c->d == 65536; }

ProductKernel kernel_for(const usl_ctx* c, const Layout& L, ProductKind kind, int shape) {
    if (c->storage == USL_F32)
        return L.halves ? kernel_f32_halves(kind, L.K, shape) : L.Q == 4 ? kernel_f32_q4(kind, L.K, shape)
             : L.Q == 2 ? kernel_f32_q2(kind, L.K, shape) : kernel_f32_q1(kind, L.K, shape);
    return L.Q == 4 ? kernel_bf16_q4(kind, L.K, shape) : L.Q == 2 ? kernel_bf16_q2(kind, L.K, shape) : kernel_bf16_q1(kind, L.K, shape);
}

struct Launch {
    ProductKernel kern;
    Geom geom;
    Tail tail;
    int64_t nblk;
    int G;              // parts of the batch
    int64_t extra;      // workgroups beyond nblk, of a tail that takes the batch in parts of its own
    int resident;       // workgroups that a compute unit is taken to hold
    size_t lds;
};

// Shape and split of the batch by estimated time, in clocks of a compute unit.  What a compute unit's workgroups share:
// the gathers (lanes * slots at 14, 12 or 8 LDS reads per clock for units of 4, 8, 16 bytes), the row copies (42 bytes
// per clock; half hidden where another buffer or workgroup is at its gathers), idx, W and grad_W on their way (7 bytes
// per clock with every unit at it).  What a workgroup waits for alone: its prologue, a barrier and copy latency per
// tile, and, with few wavefronts, the latency of a batch of reads (200 clocks).  The weight gradient of a split batch
// is written and read once more per part.  Of 40 launches over the range of sizes (profiles/rules_measured.txt) the choice
// is within 10 % of the best shape and split found by hand in 36, the median the best itself; furthest off is the weight
// gradient of a small layer with a large batch (m = 1024, d = 64, k = 8, b = 512: 25.5 us, with 16 parts 15), then
// m = 1e6, d = 2000, k = 16, b = 16 (both products 13 %) and a forward product of b = 200 over m = 5000 (17 %).
Launch choose(const usl_ctx* c, const Layout& L, int b, ProductKind kind, int most_parts = 65535) {
    const bool backward = kind == WEIGHT_GRADIENT, with_loss = kind == FORWARD_LOSS || kind == FORWARD_MARKS;
    const int es = c->storage == USL_F32 ? 4 : 2, unit = L.Q * es;
    const int groups = (b + L.Q - 1) / L.Q;
    const double reads_per_clk = unit == 16 ? 8.0 : unit == 8 ? 12.0 : 14.0;
    const int cus = c->num_cu;
    Launch best = {};
    best.kern.fn = nullptr;
    double best_t = 0.0;
    // clocks of wgs workgroups with gpb groups and `labels` labels each, `res` workgroups to a compute unit
    auto clocks = [&](const ProductKernel& kern, const Geom& tg, int res, int64_t wgs, int gpb, int labels) {
        const int lanes = (labels + 63) / 64 * 64;   // whole wavefronts gather
        const double most = (double)((wgs + cus - 1) / cus);      // workgroups the busiest compute unit runs
        const double per_cu = wgs > cus ? 0.75 * most + 0.25 * wgs / cus : most;
        const double rounds = (double)((wgs + (int64_t)cus * res - 1) / ((int64_t)cus * res));
        const double together = most / rounds;
        const double copy = (double)gpb * L.row_bytes / 42.0;
        // At most two wavefronts on a SIMD: they wait for their reads.  The factors are from workgroups of 512 lanes with two
        // labels each and of 1024 with one: m = 100k, d = 4k, k = 32, b = 128: forward 63 and 54 us, weight gradient 89 and 76;
        // m = 200k, d = 8k, b = 64, bfloat16: 60.4 and 57.3, 83 and 70.  (512 lanes with one label each lose nothing to 1024 in the
        // weight gradient: m = 646k, d = 2k, k = 64, b = 31: 223 and 253.)
        const bool thin = kern.NT / 64 * res <= 8;
        const double waits = !thin ? 1.0 : !backward ? 1.1 : kern.LPT > 1 ? 1.3 : 1.0;
        const double gather = (double)gpb * lanes * kern.K * (L.halves ? 2 : 1) / reads_per_clk * waits;
        const double more = copy > gather ? copy : gather, less = copy > gather ? gather : copy;
        const double load = (double)labels * c->k * (4.0 + (backward ? 4.0 : es)) / 7.0;
        const double tiles = (double)((gpb + tg.tile_rows - 1) / tg.tile_rows) * (L.halves ? 2 : 1);
        const double latency = (double)gpb * ((labels + kern.NT - 1) / kern.NT) * kern.K * (L.halves ? 2 : 1) / (unit == 16 ? 4 : 8) * 200.0;
        double busy = per_cu * (more + (tg.nbuf == 2 || together > 1.5 ? 0.5 : 1.0) * less);
        if (busy < rounds * latency) busy = rounds * latency;
        return busy + per_cu * load + rounds * (6000.0 + tiles * (tg.nbuf == 2 ? 600.0 : 1500.0) / (together > 1.0 ? together : 1.0));
    };
    auto sums_of = [&](int parts) { return backward && parts > 1 ? 6000.0 + (double)(parts + 1) * c->m * c->k * 4 / 4000.0 : 0.0; };
    // parts that there is room for: partial weight gradients of 512 MB at most, and no more of them than most_parts
    const size_t held = backward ? ((size_t)1 << 29) / ((size_t)c->m * c->k * 4) : (size_t)most_parts;
    const int room = held < 1 || most_parts < 1 ? 1 : held < (size_t)most_parts ? (int)held : most_parts;
    const int shape_force = tune_shape(), split_force = tune_split(), tail_force = backward ? 0 : tune_tail(), labels_force = tune_labels();
    auto shared_by = [&](int64_t same) {
        const int64_t resident = (int64_t)best.resident * (cus / 8 > 0 ? cus / 8 : 1);   // workgroups on an XCD; they go round-robin to the 8
        return (int)(same < 1 ? 1 : same < resident ? same : resident);
    };
    // the labels over n blocks of `labels`
    auto deal = [&](int64_t n, int labels) {
        // With the blocks of labels first, an XCD reads an eighth of the labels' rows and all of x; with the parts of the
        // batch first (a multiple of 8 of them) the other way round.
        // m = 16k, d = 32k, k = 32, b = 256 (x 33 MB, labels 4): forward 52 and 49 us, weight gradient 73 and 60; m = 4k,
        // d = 65k: 76 and 31, 94 and 51; m = 30k, d = 16k, b = 128 (8.4 and 7.7): 43 and 47, 52 and 51.
        best.geom.parts_first = best.G % 8 == 0 && n <= 65535 &&
                                (int64_t)groups * L.row_bytes > 2 * c->m * c->k * (backward ? 4 : 4 + es);
        best.geom.share = shared_by(best.geom.parts_first ? n : n / 8);
        best.tail = Tail{0x7FFFFFFF, 1, 1, 1, labels};
        best.extra = 0;
        best.nblk = n;
    };
    // Labels of a block of equal size (k_products.h); 0: full blocks.  By the estimate, with the workgroups that registers and LDS really leave
    // room for (of the 256-lane forms of 32 slots and more a compute unit holds half to three quarters of what the rule below takes them for): of 2212
    // scores and weight gradients over the range of sizes where it is 10 % ahead the blocks of equal size are 6 % faster on average, 38 are slower by
    // more than 3 %.  With the loss 256-lane forms have to win by 20 %: of 96 steps below that 27 are slower by more than 3 %, 5 faster; of 17 with
    // larger forms none and 3 (m = 200k, d = 8k, k = 32, b = 64, bfloat16: 219.5 and 212.4 with them).
    auto even_labels = [&]() -> int {
        const ProductKernel& kern = best.kern;
        const int per_block = kern.NT * kern.LPT, gpb = best.geom.groups_per_block;
        hipFuncAttributes full, even;
        if (hipFuncGetAttributes(&full, kern.fn) != hipSuccess || hipFuncGetAttributes(&even, kern.even) != hipSuccess) { (void)hipGetLastError(); return 0; }
        if (!even_blocks_allowed(best.G, (int64_t)groups * L.row_bytes, full.localSizeBytes, even.localSizeBytes)) return 0;
        const int res = resident_workgroups(kern.NT, full.numRegs, best.lds);
        const int labels = even_block_labels(c->m, kern, best.nblk, best.G, cus, res);
        const int64_t wgs = best.nblk * best.G, n = (c->m + labels - 1) / labels;
        if (labels >= per_block || (with_loss && (size_t)(n * best.G) > usl_forward_blocks(c))) return 0;
        const int64_t tail = best.extra ? best.tail.blocks : 0;
        double t = clocks(kern, best.geom, res, wgs - tail, gpb, per_block) + sums_of(best.G);
        if (tail) t += clocks(kern, best.geom, res, tail + best.extra, best.tail.groups, per_block);
        const double t_even = clocks(kern, best.geom, res, n * best.G, gpb, labels) + sums_of(best.G);
        return t_even * (with_loss && kern.NT == 256 ? 1.2 : 1.1) < t ? labels : 0;
    };
    for (int shape = 0; shape < 4; ++shape) {
        if (shape_force >= 0 && shape != shape_force && kernel_for(c, L, kind, shape_force).fn) continue;
        const ProductKernel kern = kernel_for(c, L, kind, shape);
        if (!kern.fn) continue;
        const int64_t per_block = (int64_t)kern.NT * kern.LPT, nblk = (c->m + per_block - 1) / per_block;
        // tiles of about 16 KB, two of them where they fit beside each other
        Geom tg;
        tg.row_bytes = L.row_bytes;
        tg.zero_col = L.zero_col;
        tg.groups = groups;
        tg.tile_rows = L.halves || L.Q == 1 || L.row_bytes > 16384 ? 1 : 16384 / L.row_bytes;
        if (tg.tile_rows > groups) tg.tile_rows = groups;
        if (with_loss && tg.tile_rows > 32 / L.Q) tg.tile_rows = 32 / L.Q;   // a tile's instances lie in one window of targets
        const size_t tile = L.halves ? (size_t)HALF_COLS * 4 : (size_t)tg.tile_rows * L.row_bytes;
        tg.nbuf = L.Q > 1 && 2 * tile <= (size_t)ROW_LDS_MAX ? 2 : 1;
        tg.buf_bytes = (int)tile;
        size_t lds = max_sz(tile * tg.nbuf, (size_t)kern.transpose_bytes);
        if (L.halves) lds = max_sz(lds, (size_t)HALF_COLS * 4 + 16);
        lds = (lds + 15) & ~(size_t)15;
        tg.dummy = (int)lds;
        lds += 256;
        const int regs = kern.NT == 1024 ? 128 : kern.NT == 256 ? 40 + kern.K * 3 / 2 : 50 + kern.LPT * kern.K * 3 / 2;
        int res = (int)((size_t)(160 * 1024) / lds);   // workgroups a compute unit holds
        const int by_regs = (512 / regs > 8 ? 8 : 512 / regs) * 4 / (kern.NT / 64);
        if (res > by_regs) res = by_regs;
        if (res < 1) res = 1;
        const auto time_of = [&](int64_t wgs, int gpb) { return clocks(kern, tg, res, wgs, gpb, (int)per_block); };
        for (int G = 1; G <= groups; G = G < 8 ? G + 1 : G + (G + 3) / 4) {
            if ((split_force > 0 || tail_force > 0) && G > 1) break;
            const int split = split_force > 0 ? (split_force < room ? split_force : room) : G, gpb = (groups + split - 1) / split;
            const int64_t parts = (groups + gpb - 1) / gpb;   // those that have work
            if (parts > room) break;
            if (with_loss && parts > 1 && (size_t)(nblk * parts) > usl_forward_blocks(c) && split_force <= 0) break;
            const int64_t slots = (int64_t)cus * res;
            double t = time_of(nblk * parts, gpb) + sums_of((int)parts);
            // A last round of workgroups that leaves most of the chip idle: its blocks take the batch in parts, so that there are
            // more and shorter workgroups of them (the scores need no adding up).  m = 670k, d = 16k, k = 32, b = 32 (328 blocks
            // of 2048 labels, 72 in three parts): 187 and 162 us; m = 600k, d = 20k, k = 32, b = 128: 452 and 330; m = 670k, d = 32k,
            // k = 64, b = 256, bfloat16: 1450 and 1305.
            const int64_t last = tail_force > 0 ? (nblk + 1) / 2 : nblk > slots ? nblk % slots : 0;
            const int64_t tail = parts == 1 && !backward ? last : 0;
            int tail_gpb = 0;
            const double whole = t;
            for (int T = tail_force > 0 ? tail_force : 2; tail > 0 && T <= groups && (T <= 16 || T == tail_force); ++T) {
                const int per = (groups + T - 1) / T;
                const int64_t items = tail * ((groups + per - 1) / per);
                if (with_loss && (size_t)(nblk - tail + items) > usl_forward_blocks(c) && tail_force <= 0) break;
                const double with = time_of(nblk - tail, gpb) + time_of(items, per);
                if (with < t || tail_force > 0) { t = with; tail_gpb = per; }
                if (tail_force > 0) break;
            }
            // ... but labels of eight slots with two wavefronts on a SIMD have to win against another shape or split by 8 %: they wait for
            // the stores of the scores, half as many as their reads, which the estimate leaves out (m = 645k, d = 3k, k = 8, b = 125:
            // 512 lanes and a tail 78 us by the estimate, 123 measured; 1024 lanes in three parts 83 and 98).
            if (tail_gpb && kern.K == 8 && kern.NT / 64 * res <= 8) t = t * 1.08 < whole ? t * 1.08 : whole;
            if (best.kern.fn && t >= best_t) continue;
            best_t = t;
            best.kern = kern;
            tg.groups_per_block = gpb;
            best.geom = tg;
            best.resident = res;
            best.lds = lds;
            best.G = (int)parts;
            deal(nblk, (int)per_block);
            if (tail_gpb) {
                best.tail = Tail{(int)(nblk - tail), (int)tail, tail_gpb, shared_by(tail / 8), (int)per_block};
                best.extra = tail * ((groups + tail_gpb - 1) / tail_gpb) - tail;
            }
        }
    }
    if (!best.kern.fn || tail_force > 0) return best;
    const int labels = labels_force > 0 ? (labels_force + 31) / 32 * 32 : even_labels();
    if (labels > 0 && labels < best.kern.NT * best.kern.LPT) {
        best.kern.fn = best.kern.even;
        deal((c->m + labels - 1) / labels, labels);
    }
    return best;
}

usl_status launch(usl_ctx* c, const Launch& p, void** args, const char* what) {
    if (p.lds > 65536)
        USL_HIP(c, hipFuncSetAttribute(p.kern.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds));
    const dim3 grid = p.geom.parts_first ? dim3((unsigned)p.G, (unsigned)p.nblk) : dim3((unsigned)(p.nblk + p.extra), (unsigned)p.G);
    USL_HIP(c, hipLaunchKernel(p.kern.fn, grid, dim3((unsigned)p.kern.NT), args, p.lds, c->stream));
    return usl_check_launch(c, what);
}

usl_status interleave(usl_ctx* c, const void* x, int b, int Q, int row_bytes, void** to, size_t* cap, const Before& before = Before{}) {
    const int es = c->storage == USL_F32 ? 4 : 2, groups = (b + Q - 1) / Q, cols = row_bytes / (Q * es);
    const int qmax = 4;   // sized once, for the largest batch any later call can bring
    const size_t need = (size_t)((c->max_b + qmax - 1) / qmax) * qmax * ((size_t)c->d + 16) * es;
    USL_TRY(usl_reserve(c, to, cap, max_sz(need, (size_t)groups * row_bytes)));
    const int blocks = (cols + 255) / 256, more_rows = before.targets.off ? (before.blocks() + blocks - 1) / blocks : 0;
    const dim3 grid((unsigned)blocks, (unsigned)(groups + more_rows < 65535 ? groups + more_rows : 65535));
#define USL_IL(TS, QQ) hipLaunchKernelGGL((k_interleave<TS, QQ>), grid, dim3(256), 0, c->stream, (const TS*)x, (TS*)*to, b, c->d, cols, before, groups)
    if (es == 4) { if (Q == 4) USL_IL(float, 4); else if (Q == 2) USL_IL(float, 2); else USL_IL(float, 1); }
    else { if (Q == 4) USL_IL(uint16_t, 4); else if (Q == 2) USL_IL(uint16_t, 2); else USL_IL(uint16_t, 1); }
#undef USL_IL
    return usl_check_launch(c, "activations");
}

// The interleaved activations of this call, in scratch of the context (or x itself, if it is laid out that way).
// Inside usl_train_step the copy that forward made serves the backward products too.  before: what else is to be done on the way.
usl_status activations(usl_ctx* c, const Layout& L, const void* x, int b, const void** xi, const Before& before = Before{}) {
    *xi = x;
    const bool copies = L.copy && (c->xi_of != x || c->xi_q != L.Q || c->xi_row_bytes != L.row_bytes);
    const bool along = copies && (b + L.Q - 1) / L.Q < 65535 - 32;   // k_interleave's grid has room for the fingerprint's blocks and more, a row each at worst
    if (before.targets.off && !along) hipLaunchKernelGGL(k_before_forward, dim3((unsigned)before.blocks()), dim3(256), 0, c->stream, before);
    if (!L.copy) return USL_OK;
    if (copies) USL_TRY(interleave(c, x, b, L.Q, L.row_bytes, &c->xi, &c->xi_cap, along ? before : Before{}));
    *xi = c->xi;
    c->xi_of = c->xi_keep ? x : nullptr;
    c->xi_q = L.Q;
    c->xi_row_bytes = L.row_bytes;
    return USL_OK;
}

// The register-resident kernels need k <= 64, columns that fit 16 bits, and 16-byte aligned idx / W / grad_W.
bool fast_path_ok(const usl_ctx* c, const void* idx, const void* W) {
    return c->d <= 65536 && c->k <= 64 && (uintptr_t)idx % 16 == 0 && (W == nullptr || (uintptr_t)W % 16 == 0);
}

// The bank-aware order belongs to the layout of the largest groups (a small batch with a smaller Q uses it as it is:
// any order is right).  A label subset is new on every call: building an order would cost more than it saves.
usl_status slot_order(usl_ctx* c, const int32_t* idx, const uint8_t** perm) {
    *perm = nullptr;
    if (c->no_order) return USL_OK;
    if (c->slot_order_for != idx) {
        const Layout L = layout_of(c, 4, nullptr);
        USL_TRY(usl_build_slot_order(c, idx, L.K, L.Q * (c->storage == USL_F32 ? 4 : 2)));
    }
    *perm = c->slot_order;
    return USL_OK;
}

// Shape of the streaming kernel: lanes of a label, rounds of a wavefront's turn, wavefronts of a workgroup, workgroups, turns of a wavefront.
struct FewShape {
    int lpl, rounds, nw;
    unsigned grid;
    int64_t turns;
    size_t lds;
};
FewShape few_shape(const usl_ctx* c, const Layout& L, int kk) {
    FewShape f;
    f.lpl = c->k <= 8 ? 2 : c->k <= 16 ? 4 : c->k <= 32 ? 8 : 16;
    // fewer labels per wavefront, then workgroups of 4 or 8 wavefronts, so that a small layer still reaches every compute unit
    f.rounds = f.lpl;
    auto wavefronts = [&]() { const int64_t per = (int64_t)f.rounds * (64 / f.lpl); return (c->m + per - 1) / per; };
    while (f.rounds > 2 && wavefronts() < (int64_t)c->num_cu * 16) f.rounds >>= 1;
    const int64_t waves = wavefronts();
    f.nw = waves >= (int64_t)c->num_cu * 16 ? 16 : waves >= (int64_t)c->num_cu * 8 ? 8 : 4;
    const int64_t blocks = (waves + f.nw - 1) / f.nw;
    f.lds = max_sz((size_t)L.row_bytes + 16, kk > 0 ? (size_t)16 * 32 * 8 + 16 : 0);
    const int by_lds = (int)((size_t)(160 * 1024) / f.lds), resident = by_lds < 32 / f.nw ? (by_lds < 1 ? 1 : by_lds) : 32 / f.nw;
    f.grid = (unsigned)(blocks < (int64_t)c->num_cu * resident ? blocks : (int64_t)c->num_cu * resident);   // usl_forward_few_blocks at most: fewer than 16 wavefronts only where there are fewer than that of them
    f.turns = (waves + (int64_t)f.grid * f.nw - 1) / ((int64_t)f.grid * f.nw);
    return f;
}

// Prediction of one instance: the best labels from the forward kernel, or from kernels over its scores?  The forward kernel's workgroups look for theirs when
// all wavefronts are done, 3 us of chains of maxima for 5 labels, and where two of 16 wavefronts share a compute unit or many labels are asked for their candidates take longer to
// merge; the other way costs a launch and a pass of 6 us over scores in the cache, and 1 us of forward less.  usl_predict, from forward and with the pass, us (captured graphs):
// smaller workgroups: m = 5000, d = 64, k = 8, 5 labels 8.5 and 11.2, 32 labels 31.1 and 41.8; m = 60 867, d = 1344, k = 16, 5 labels 11.7 and 12.0, not so 10 labels 18.9 and 18.0, 32 labels 76.8 and
// 42.9; m = 49k, d = 1762, k = 32, 5 labels 12.9 and 14.5, not so 8 labels 19.2 and 18.1; m = 100k, d = 600, k = 8, 5 labels 9.6 and 11.9, not so 16 labels 27.5 and 24.6; m = 262k, d = 25k, k = 8, 32
// labels (8192 candidates and 4096) 50.7 and 57.8;
// one of 16 wavefronts to a compute unit: m = 500k, d = 32k, k = 32, 5 labels 28.6 and 30.8, 32 labels 70.0 and 74.7; m = 114k, d = 34k, k = 32, 5 labels 12.7 and 14.4 (32 labels 54.7 and 45.8);
// not so two of them: m = 225 711, d = 118, k = 13, 5 labels 22.0 and 18.0; m = 109 071, d = 7213, k = 32 17.8 and 15.9; m = 720 436, d = 2151, k = 13 33.1 and 29.7 (m = 1.02M, d = 2473, k = 8 24.2 and 25.7);
// three turns: m = 1.27M, d = 11k, k = 32, 5 labels 63.7 and 68.4, 32 labels 145 and 156; m = 1.32M, d = 561, k = 56, bfloat16 95.3 and 99.6 (m = 1.34M, d = 11k, k = 3 24.5 and 23.6).
bool best_from_forward(const usl_ctx* c, const FewShape& f, int kk) {
    if (f.nw < 16) {
        const int64_t n = (int64_t)f.grid * kk, by_pass = (c->m + TOPK_SHORT_SEGMENT - 1) / TOPK_SHORT_SEGMENT * kk;   // candidates
        return kk <= 5 || n <= TOPK_SHORT_MERGE || (by_pass > TOPK_SHORT_MERGE && n <= by_pass * 2);
    }
    return f.grid <= (unsigned)c->num_cu || f.turns >= 3;
}

// ... and who merges the workgroups' candidates: the one that comes last, or a launch of its own?  The last one has waited for the others at the count, which
// takes 11.5 ns of each, and saves a launch; a launch of more than TOPK_SHORT_MERGE candidates takes 3 to 6 us longer.  So it is the last one with few workgroups (the more, the
// more labels are asked for), with many candidates, and where the stream of idx and W lasts so long that the workgroups come in spread out.  usl_predict, last workgroup and
// launch, from captured graphs | call by call, us: 47 workgroups, 1 label 5.55 and 5.40 | 6.2 and 8.8; 79, 3 labels 7.5 and 7.3 | 7.6 and 8.4; 79, 10 labels 13.4 and 14.1 | 13.2 and 14.1;
// not so 118, 1 label 6.3 and 5.4 | 7.0 and 8.8; 157, 5 labels 9.9 and 9.3 | 9.9 and 9.9; 254, 2 labels 8.6 and 6.5 | 8.6 and 8.3; 256 of 8 wavefronts (m = 131k, d = 25k, k = 16), 5 labels 12.8 and
// 10.8 | 12.7 and 11.0; 256 of 16 wavefronts with 29 MB (m = 114k, d = 34k, k = 32), 5 labels 14.5 and 13.0 | 14.3 and 13.1, 10 labels 19.7 and 22.5 | 19.5 and 22.4; with 45 MB (m = 175k, d = 33k) 5 labels
// 19.9 and 19.7 | 18.4 and 18.7; with 128 MB (m = 500k, d = 32k) 30.0 and 29.8 | 30.1 and 30.0, 10 labels 33.9 and 37.4 | 35.3 and 39.4.  (Two workgroups to a compute unit: their candidates, twice as many,
// come late; m = 1.34M, d = 11k, k = 3 25.1 us with a launch for the merge, 26.1 without.)
bool last_one_merges(const usl_ctx* c, const FewShape& f, int kk) {
    const int64_t n = (int64_t)f.grid * kk, stream = c->m * c->k * (c->storage == USL_F32 ? 8 : 6);
    if (f.grid > (unsigned)c->num_cu || n > (int64_t)FEW_HELD * f.nw * 64) return false;
    return (int)f.grid <= 32 + 16 * kk || n > TOPK_SHORT_MERGE || stream >= 40000000;
}

// One group of instances: the streaming kernel.  kk > 0, one instance: its best labels; out is scratch then, written only by wavefronts of more than FEW_HELD turns.
usl_status run_forward_few(usl_ctx* c, const Layout& L, const void* x, const int32_t* idx, const void* W, float* out, int b, int kk = 0, int32_t* top_lab = nullptr,
                           float* top_val = nullptr) {
    const void* xi = nullptr;
    USL_TRY(activations(c, L, x, b, &xi));
    const FewShape f = few_shape(c, L, kk);
    const int lpl = f.lpl, rounds = f.rounds, nw = f.nw;
    const unsigned grid = f.grid;
    const size_t lds = f.lds;
    const bool vec = c->k % 4 == 0;
    uint64_t* cand = nullptr;
    bool merge = false;   // by the workgroup that comes last
    if (kk > 0) {
        USL_TRY(usl_reserve_topk(c));
        cand = c->topk_cand;
        merge = c->topk_done_clear && last_one_merges(c, f, kk);
    }
#define USL_FEW_B(LPL, TS, Q, VEC, AHEAD, BEST)                                                                    \
    do {                                                                                                                \
        USL_TRY(allow_lds(c, k_forward_few<LPL, TS, Q, VEC, AHEAD, BEST>, lds));                                    \
        hipLaunchKernelGGL((k_forward_few<LPL, TS, Q, VEC, AHEAD, BEST>), dim3(grid), dim3((unsigned)nw * 64), lds, c->stream,        \
                           (const char*)xi, idx, (const TS*)W, out, c->m, c->k, b, L.row_bytes, rounds, kk, cand,      \
                           c->topk_done, merge ? top_lab : nullptr, top_val);                                                          \
    } while (0)
#define USL_FEW_A(LPL, TS, Q, VEC, AHEAD) do { if (Q == 1 && kk > 0) USL_FEW_B(LPL, TS, Q, VEC, AHEAD, (Q == 1)); else USL_FEW_B(LPL, TS, Q, VEC, AHEAD, false); } while (0)
#define USL_FEW(LPL, TS, Q, VEC)                                                                                    \
    do {                                                                                                                \
        if (Q == 1 && LPL >= 4 && rounds >= 4) USL_FEW_A(LPL, TS, Q, VEC, (Q == 1 && LPL >= 4 ? 4 : 2));            \
        else USL_FEW_A(LPL, TS, Q, VEC, 2);                                                                         \
    } while (0)
#define USL_FEW_V(LPL, TS, Q) do { if (vec) USL_FEW(LPL, TS, Q, true); else USL_FEW(LPL, TS, Q, false); } while (0)
#define USL_FEW_L(TS, Q)                                                                                            \
    do {                                                                                                                \
        if (lpl == 2) USL_FEW_V(2, TS, Q);                                                                          \
        else if (lpl == 4) USL_FEW_V(4, TS, Q);                                                                     \
        else if (lpl == 8) USL_FEW_V(8, TS, Q);                                                                     \
        else USL_FEW_V(16, TS, Q);                                                                                  \
    } while (0)
    if (c->storage == USL_F32) {
        if (L.Q == 4) USL_FEW_L(float, 4);
        else if (L.Q == 2) USL_FEW_L(float, 2);
        else USL_FEW_L(float, 1);
    } else {
        if (L.Q == 4) USL_FEW_L(uint16_t, 4);
        else if (L.Q == 2) USL_FEW_L(uint16_t, 2);
        else USL_FEW_L(uint16_t, 1);
    }
#undef USL_FEW_L
#undef USL_FEW_V
#undef USL_FEW
#undef USL_FEW_A
#undef USL_FEW_B
    USL_TRY(usl_check_launch(c, "forward (one group)"));
    return kk > 0 && !merge ? usl_launch_topk_merge(c, (int)grid, b, kk, top_lab, top_val) : USL_OK;
}

}  // namespace

namespace {

size_t target_words(const usl_ctx* c) { return (size_t)((c->max_b + 31) / 32) * (size_t)c->m; }

// Labels of 24 slots: through the caches the scores take 5 to 15 % longer, but where a row of them does not begin with a line (see put in k_forward), there are many
// of them and rows of x are so short that little else is under way, past the caches up to 50 %: m = 327 357, d = 38, b = 189, bfloat16 132 us and 88;
// m = 413 191, d = 520, b = 219, bfloat16 169 and 138; m = 400 003, d = 300, b = 100 78 and 74.  Past the caches and through them beside the lines: m = 756 271, d = 525,
// b = 136 170 and 195; m = 59 655, b = 387 46 and 50; b = 33 69 and 74; 44 MB of scores 27 and 32.  (Of 32 slots and more they are nowhere faster through the caches.)
bool scores_through_caches(const usl_ctx* c, const Layout& L, const float* out, int32_t b) {
    return L.K == 24 && (c->m % 32 != 0 || (uintptr_t)out % 128 != 0) && (size_t)c->d * (c->storage == USL_F32 ? 4 : 2) <= 1280 && c->m >= 80000 && b >= 36 &&
           c->m * b >= (int64_t)1 << 24;
}

// the forward kernel over the whole batch, with or without the loss (then `before` says what the targets are; their bits are set
// here and taken back by the kernel that ends the step)
usl_status run_forward(usl_ctx* c, const Layout& L, const void* x, const int32_t* idx, const void* W, float* out, int32_t b, LossArgs loss,
                       size_t* blocks, Before before = Before{}) {
    const Launch p = choose(c, L, b, loss.nonzeros ? FORWARD_MARKS : loss.kind >= 0 ? FORWARD_LOSS : scores_through_caches(c, L, out, b) ? FORWARD_CACHED : FORWARD);
    const uint8_t* perm = nullptr;
    const void* xi = nullptr;
    USL_TRY(slot_order(c, idx, &perm));
    if (loss.kind >= 0) {
        const size_t words = target_words(c), had = c->tgt_bits_cap;
        USL_TRY(usl_reserve(c, (void**)&c->tgt_bits, &c->tgt_bits_cap, words * 4));
        if (had != c->tgt_bits_cap || c->tgt_bits_set)   // new, or a call before failed half way
            hipLaunchKernelGGL(k_fill_zero, dim3(c->num_cu * 4), dim3(256), 0, c->stream, reinterpret_cast<float*>(c->tgt_bits), words);
        c->tgt_bits_set = true;
        before.targets.bits = c->tgt_bits;
        loss.targets = c->tgt_bits;
    }
    USL_TRY(activations(c, L, x, b, &xi, before));
    int64_t m = c->m;
    int k = c->k, bb = b;
    Geom tg = p.geom;
    if (loss.kind >= 0) {
        *blocks = (size_t)p.nblk * (size_t)p.G + (size_t)p.extra;
        USL_TRY(usl_reserve_loss_partials(c));
        USL_TRY(usl_reserve(c, (void**)&c->bce_partials, &c->bce_partials_cap, *blocks * sizeof(double)));   // more only with parts asked for by hand
        loss.partials = c->bce_partials;
    }
    Tail tail = p.tail;
    void* args[] = {&xi, &idx, &W, &out, &m, &k, &bb, &tg, &perm, &loss, &tail};
    return launch(c, p, args, "forward");
}

bool streams(const usl_ctx* c, const Layout& L, int b) { return b <= L.Q && !L.halves && !c->part_of_batch; }

}  // namespace

usl_status usl_launch_forward(usl_ctx* c, const void* x, const int32_t* idx, const void* W, float* out, int32_t b) {
    if (!fast_path_ok(c, idx, W))
        return c->storage == USL_F32 ? run_forward_generic<float>(c, x, idx, W, out, b) : run_forward_generic<uint16_t>(c, x, idx, W, out, b);
    const Layout L = layout_of(c, b, x);
    if (streams(c, L, b)) return run_forward_few(c, L, x, idx, W, out, b);
    USL_TRY(run_forward(c, L, x, idx, W, out, b, LossArgs{-1, 0.f, nullptr, nullptr, nullptr, 0, nullptr}, nullptr));
    if (!pads_with_column_0(c, L)) return USL_OK;
    const dim3 grid((unsigned)((c->m + 255) / 256));
    if (c->storage == USL_F32)
        hipLaunchKernelGGL(k_forward_again<float>, grid, dim3(256), 0, c->stream, (const float*)x, idx, (const float*)W, out, c->m, c->d, c->k, b);
    else
        hipLaunchKernelGGL(k_forward_again<uint16_t>, grid, dim3(256), 0, c->stream, (const uint16_t*)x, idx, (const uint16_t*)W, out, c->m, c->d, c->k, b);
    return usl_check_launch(c, "forward (activations that are not finite)");
}

usl_status usl_launch_predict_few(usl_ctx* c, const void* x, const int32_t* idx, const void* W, float* out, int32_t b, int32_t kk,
                                  int32_t* top_lab, float* top_val, bool* done) {
    *done = false;
    if (!fast_path_ok(c, idx, W)) return USL_OK;
    const Layout L = layout_of(c, b, x);
    if (b > 1 || !streams(c, L, b) || !best_from_forward(c, few_shape(c, L, kk), kk)) return USL_OK;
    USL_TRY(run_forward_few(c, L, x, idx, W, out, b, kk, top_lab, top_val));
    *done = true;
    return USL_OK;
}

bool usl_forward_loss_applies(const usl_ctx* c, const void* x, const int32_t* idx, const void* W, int32_t b) {
    const Layout L = layout_of(c, b, x);
    // (at most 1 GiB of target bits, m * max_b of 8.6e9: a context made for far larger batches than it sees pays in time, not memory)
    return fast_path_ok(c, idx, W) && !streams(c, L, b) && !pads_with_column_0(c, L) /* scores are done again, their losses not */ &&
           target_words(c) * 4 <= (size_t)1 << 30;
}

usl_status usl_launch_forward_loss(usl_ctx* c, const void* x, const int32_t* idx, const void* W, float* g, int32_t b, int loss_kind,
                                   const int64_t* tgt_off, const int32_t* tgt_lab, float scale, float* loss, usl_loss_sum* sum, float* marks_clear) {
    size_t blocks = 0;
    const Layout L = layout_of(c, b, x);
    usl_targets targets = {tgt_off, tgt_lab, nullptr, c->m, b};
    const bool check = c->lf[1].built_for == idx;   // lists that the backward product will use
    if (marks_clear) USL_TRY(usl_sparse_marks_ready(c));
    USL_TRY(run_forward(c, L, x, idx, W, g, b, LossArgs{loss_kind, scale, nullptr, nullptr, marks_clear ? c->nz_bits : nullptr, (int64_t)usl_sparse_mark_words(c), marks_clear},
                        &blocks, Before{targets, check ? reinterpret_cast<const uint32_t*>(idx) : nullptr, (size_t)c->m * c->k, c->idx_print, marks_clear ? c->nz_state : nullptr}));
    c->print_done = check;
    targets.bits = c->tgt_bits;
    *sum = usl_loss_sum{c->bce_partials, blocks, scale, loss, targets};
    return USL_OK;
}

usl_status usl_activation_rows(usl_ctx* c, const void* x, int32_t b, int Q, const void** rows, size_t* stride) {
    const int es = c->storage == USL_F32 ? 4 : 2;
    if (Q == 1 && (size_t)c->d * es % 16 == 0 && (uintptr_t)x % 16 == 0) {
        *rows = x;
        *stride = (size_t)c->d;
        return USL_OK;
    }
    if (c->xi_of == x && c->xi_q == Q) {   // usl_train_step: the copy that forward made
        *rows = c->xi;
        *stride = (size_t)c->xi_row_bytes / es;
        return USL_OK;
    }
    const int per = 16 / (Q * es), cols = (c->d + per - 1) / per * per;
    USL_TRY(interleave(c, x, b, Q, cols * Q * es, &c->xr, &c->xr_cap));
    *rows = c->xr;
    *stride = (size_t)cols * Q;
    return USL_OK;
}

// Parts of the batch that the weight gradient's scratch has room for: the most that the largest batch or a half, a quarter
// or an eighth of it would take.  A batch in between makes do with them.
static int weight_gradient_parts(usl_ctx* c, const void* x) {
    if (tune_split() > 0) return 65535;
    if (!c->gw_parts_most) {
        int most = 1;
        for (int b = c->max_b, q = 0; b >= 1 && q < 4; b /= 2, ++q) {
            const int G = choose(c, layout_of(c, b, x), b, WEIGHT_GRADIENT).G;
            if (G > most) most = G;
        }
        c->gw_parts_most = most;
    }
    return c->gw_parts_most;
}

usl_status usl_launch_backward_weight(usl_ctx* c, const float* g, const void* x, const int32_t* idx, float* grad_W, int32_t b, bool dense) {
    if (!fast_path_ok(c, idx, nullptr) || (uintptr_t)grad_W % 16 != 0)
        return c->storage == USL_F32 ? run_backward_weight_generic<float>(c, g, x, idx, grad_W, b)
                                     : run_backward_weight_generic<uint16_t>(c, g, x, idx, grad_W, b);
    const Layout L = layout_of(c, b, x);
    const int most_parts = weight_gradient_parts(c, x);
    const Launch p = choose(c, L, b, WEIGHT_GRADIENT, most_parts);
    const uint8_t* perm = nullptr;
    const void* xi = nullptr;
    USL_TRY(slot_order(c, idx, &perm));
    // a gradient that may be almost all zeros is first tried through the lists of its nonzeros; the device decides which
    // path does the work
    const uint32_t* gate = nullptr;
    if (!dense && usl_sparse_supported(c)) {
        if (c->nz_lists_of == g) gate = c->nz_lists_tried ? c->nz_state : nullptr;
        else USL_TRY(usl_sparse_compact(c, g, b, &gate));
        if (gate) USL_TRY(usl_sparse_backward_weight(c, x, idx, grad_W, b));
    }
    USL_TRY(activations(c, L, x, b, &xi));
    const size_t N = (size_t)c->m * c->k;
    // a batch in several parts: partial gradients in scratch, summed afterwards in a fixed order (no atomics, reproducible)
    size_t stride = (N + 3) / 4 * 4;
    float* dst = grad_W;
    const size_t parts = (size_t)(most_parts < 65535 ? most_parts : p.G);
    if (parts > 1) USL_TRY(usl_reserve(c, (void**)&c->gw_part, &c->gw_part_cap, parts * stride * 4));   // also for a batch in one part: never in a later call
    if (p.G > 1) dst = c->gw_part;
    else stride = 0;
    int64_t m = c->m;
    int k = c->k, bb = b;
    Geom tg = p.geom;
    int labels = p.tail.labels;
    void* args[] = {&g, &xi, &idx, &dst, &m, &k, &bb, &tg, &perm, &stride, &gate, &labels};
    USL_TRY(launch(c, p, args, "backward_weight"));
    if (p.G > 1) {
        const size_t blocks = (N / 4 + 256) / 256;
        hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)(blocks < (size_t)c->num_cu * 8 ? blocks : (size_t)c->num_cu * 8)),
                           dim3(256), 0, c->stream, c->gw_part, p.G, N, stride, grad_W, gate);
    }
    return usl_check_launch(c, "backward_weight");
}
