// Connection redistribution (magnitude prune of the whole layer + random regrow inside each row),
// initial connectivity, the index validator and the raw generator words.
//
// Prune: the n smallest keys (|W| bit pattern, flat slot) are found without sorting: a radix
// select over the magnitude bits (most significant digit first, one histogram pass per digit)
// yields the threshold magnitude T and the number q of slots with magnitude exactly T that still
// have to go; those q are the first in flat order, found with a per-block tie count, a scan of
// the block counts and an in-block rank.  Regrow: a group of lanes owns a row, the lane of slot t
// keeps idx[j][t]; candidates are generated redundantly by the group and tested with a ballot.
#include "usl_internal.h"

namespace {

// ---- Philox-4x32, 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11) --------------------------------
struct U4 { uint32_t x, y, z, w; };
__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c.x), lo0 = 0xD2511F53u * c.x;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z), lo1 = 0xCD9E8D57u * c.z;
        c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}
// candidate number a for slot t of row j: word 0, mapped to [0, d) by multiply-shift
__device__ __forceinline__ int32_t draw_column(uint32_t k0, uint32_t k1, uint32_t epoch_lo,
                                               uint32_t j, uint32_t t, uint32_t a, uint32_t d) {
    const U4 r = philox4x32_10(U4{j, t, a, epoch_lo}, k0, k1);
    return (int32_t)__umulhi(r.x, d);
}

__global__ void k_philox(const uint32_t* __restrict__ ctr, uint32_t k0, uint32_t k1,
                         uint32_t* __restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const U4 r = philox4x32_10(U4{ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]}, k0, k1);
    out[4 * i] = r.x; out[4 * i + 1] = r.y; out[4 * i + 2] = r.z; out[4 * i + 3] = r.w;
}

// ---- radix select ---------------------------------------------------------------------------
constexpr int SEL_BINS = 2048, SEL_NT = 1024;
// device state: [0..SEL_BINS) histogram, then: prefix, remaining count, (unused), keys in the bin picked last
enum { ST_PREFIX = SEL_BINS, ST_REMAIN = SEL_BINS + 1, ST_TIES = SEL_BINS + 3, ST_WORDS = SEL_BINS + 4 };

__device__ __forceinline__ uint32_t mag_of(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }
__device__ __forceinline__ uint32_t mag_of(uint16_t v) { return (uint32_t)v & 0x7FFFu; }
template <typename TS> __device__ __forceinline__ uint32_t mag_key(const TS* W, size_t f) { return mag_of(W[f]); }
// 16 bytes of W, at any element
template <typename TS> struct Piece {
    static constexpr int N = 16 / sizeof(TS);
    typedef TS T __attribute__((ext_vector_type(N), aligned(sizeof(TS))));
};
template <typename TS> __device__ __forceinline__ typename Piece<TS>::T piece_at(const TS* W, size_t f) {
    return *reinterpret_cast<const typename Piece<TS>::T*>(W + f);
}
// Do all keys equal to the threshold go?  (float32: nearly always, there is one.)  Nobody has to count them in order then.
__device__ __forceinline__ bool all_ties_go(const uint32_t* st) { return st[ST_TIES] == st[ST_REMAIN]; }

__global__ void k_sel_init(uint32_t* st, uint32_t n) {
    for (int i = threadIdx.x; i < ST_WORDS; i += blockDim.x) st[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) st[ST_REMAIN] = n;
}

// histogram of digit (key >> shift) & (2^bits - 1) over the keys whose higher bits equal the prefix
template <typename TS>
__global__ void __launch_bounds__(SEL_NT)
k_sel_hist(const TS* __restrict__ W, size_t N, uint32_t* st, int shift, int bits, int first) {
    __shared__ uint32_t h[SEL_BINS];
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_NT) h[i] = 0;
    __syncthreads();
    const uint32_t prefix = st[ST_PREFIX];
    const uint32_t mask = (1u << bits) - 1u;
    constexpr int V = Piece<TS>::N;
    auto one = [&](TS v) {
        const uint32_t key = mag_of(v);
        if (first || (key >> (shift + bits)) == prefix) atomicAdd(&h[(key >> shift) & mask], 1u);
    };
    // 16 bytes a load, four of a lane's in flight (one value a load and 2048 workgroups of 256 lanes, see the launch: 56, 35 and 35 us for the three
    // digits of 16 million float32 weights, now 21, 14 and 14)
    const size_t stride = (size_t)gridDim.x * SEL_NT, pieces = N / V;
    for (size_t q = (size_t)blockIdx.x * SEL_NT + threadIdx.x; q < pieces; q += 4 * stride) {
        typename Piece<TS>::T v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = piece_at(W, min(q + u * stride, pieces - 1) * V);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (q + u * stride >= pieces) continue;
#pragma unroll
            for (int e = 0; e < V; ++e) one(v[u][e]);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < N - pieces * V) one(W[pieces * V + threadIdx.x]);
    __syncthreads();
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_NT)
        if (h[i]) atomicAdd(&st[i], h[i]);
}

// picks the digit in which the running count crosses the remaining count; clears the histogram.
// One block of 256 lanes: each sums a run of consecutive bins, a scan over the lanes finds the run that holds
// the crossing, and that lane walks its few bins.
__global__ void __launch_bounds__(256) k_sel_pick(uint32_t* st, int bits) {
    __shared__ uint32_t run_sum[256];
    const int nb = 1 << bits;
    const int per = (nb + 255) / 256;             // at most SEL_BINS / 256
    const int first = (int)threadIdx.x * per;
    uint32_t mine = 0;
    for (int q = 0; q < per; ++q)
        if (first + q < nb) mine += st[first + q];
    run_sum[threadIdx.x] = mine;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {           // inclusive scan
        const uint32_t v = threadIdx.x >= (unsigned)o ? run_sum[threadIdx.x - o] : 0u;
        __syncthreads();
        run_sum[threadIdx.x] += v;
        __syncthreads();
    }
    const uint32_t remain = st[ST_REMAIN], prefix = st[ST_PREFIX];
    const uint32_t before = run_sum[threadIdx.x] - mine;
    const uint32_t total = run_sum[255];
    __syncthreads();
    if (before < remain && before + mine >= remain) {
        uint32_t cum = before;
        int bin = first;
        uint32_t hcount = 0;
        for (int q = 0; q < per; ++q) {
            hcount = st[first + q];
            if (cum + hcount >= remain) { bin = first + q; break; }
            cum += hcount;
        }
        st[ST_TIES] = hcount;
        st[ST_PREFIX] = (prefix << bits) | (uint32_t)bin;
        st[ST_REMAIN] = remain - cum;  // = how many keys equal to the final prefix must go
    } else if (threadIdx.x == 0 && total < remain) {   // cannot happen for a consistent histogram
        st[ST_PREFIX] = (prefix << bits) | (uint32_t)(nb - 1);
        st[ST_REMAIN] = remain - total;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SEL_BINS; i += blockDim.x) st[i] = 0;
}

// A workgroup of the two kernels below has MARK_CHUNK values: pieces of 16 bytes, lane by lane, MARK_PIECES<TS> of them a lane.
constexpr int MARK_NT = 256;
constexpr int MARK_CHUNK = 4096;
template <typename TS> constexpr int MARK_PIECES = MARK_CHUNK / MARK_NT / Piece<TS>::N;

// the lane's keys; 0xFFFFFFFF behind the last one
template <typename TS>
__device__ __forceinline__ void mark_keys(const TS* __restrict__ W, size_t N, uint32_t (&keys)[MARK_PIECES<TS>][Piece<TS>::N]) {
    constexpr int V = Piece<TS>::N;
    const size_t f0 = (size_t)blockIdx.x * MARK_CHUNK + (size_t)threadIdx.x * V;
    typename Piece<TS>::T v[MARK_PIECES<TS>];
#pragma unroll
    for (int u = 0; u < MARK_PIECES<TS>; ++u) {
        const size_t f = f0 + (size_t)u * MARK_NT * V;
        if (f + V <= N) v[u] = piece_at(W, f);
        else
#pragma unroll
            for (int e = 0; e < V; ++e) v[u][e] = f + e < N ? W[f + e] : (TS)0;
    }
#pragma unroll
    for (int u = 0; u < MARK_PIECES<TS>; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) keys[u][e] = f0 + (size_t)u * MARK_NT * V + e < N ? mag_of((TS)v[u][e]) : 0xFFFFFFFFu;
}

template <typename TS>
__global__ void __launch_bounds__(MARK_NT)
k_tie_count(const TS* __restrict__ W, size_t N, const uint32_t* __restrict__ st,
            uint32_t* __restrict__ tie_counts) {
    __shared__ uint32_t red[MARK_NT / 64];
    if (all_ties_go(st)) return;
    const uint32_t T = st[ST_PREFIX];
    uint32_t keys[MARK_PIECES<TS>][Piece<TS>::N], cnt = 0;
    mark_keys(W, N, keys);
#pragma unroll
    for (int u = 0; u < MARK_PIECES<TS>; ++u)
#pragma unroll
        for (int e = 0; e < Piece<TS>::N; ++e) cnt += keys[u][e] == T;
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_down(cnt, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
        for (int q = 0; q < MARK_NT / 64; ++q) s += red[q];
        tie_counts[blockIdx.x] = s;
    }
}

// exclusive scan of the per-block tie counts, in place (one block)
__global__ void __launch_bounds__(1024) k_tie_scan(uint32_t* tie_counts, size_t nblk, const uint32_t* __restrict__ st) {
    __shared__ uint32_t part[1024];
    if (all_ties_go(st)) return;
    const size_t per = (nblk + 1023) / 1024;
    const size_t a = threadIdx.x * per, e = min(nblk, a + per);
    uint32_t s = 0;
    for (size_t q = a; q < e; ++q) s += tie_counts[q];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int q = 0; q < 1024; ++q) { const uint32_t v = part[q]; part[q] = run; run += v; }
    }
    __syncthreads();
    uint32_t run = part[threadIdx.x];
    for (size_t q = a; q < e; ++q) { const uint32_t v = tie_counts[q]; tie_counts[q] = run; run += v; }
}

// Flags every removed slot and resets its value and moments.  Bound by the lines of the values that it resets.  (Sixteen
// neighbouring values to a lane, a load each, and the ties counted whatever their number took 77 us behind 52 for the counts at
// m = 500k, k = 32, 5 %; now 41 behind 9.)
template <typename TS>
__global__ void __launch_bounds__(MARK_NT)
k_mark(TS* __restrict__ W, float* __restrict__ m1, float* __restrict__ m2, size_t N,
       const uint32_t* __restrict__ st, const uint32_t* __restrict__ tie_off,
       uint8_t* __restrict__ flags) {
    constexpr int V = Piece<TS>::N, P = MARK_PIECES<TS>;
    __shared__ uint32_t ties[P][MARK_NT / 64];
    const uint32_t T = st[ST_PREFIX], q_take = st[ST_REMAIN];
    const bool all = all_ties_go(st);
    const size_t f0 = (size_t)blockIdx.x * MARK_CHUNK + (size_t)threadIdx.x * V;
    uint32_t keys[P][V];
    mark_keys<TS>(W, N, keys);
    uint32_t rank[P] = {};   // of the first tie of the lane's piece, in flat order
    if (!all) {
#pragma unroll
        for (int u = 0; u < P; ++u) {
            uint32_t mine = 0;
#pragma unroll
            for (int e = 0; e < V; ++e) mine += keys[u][e] == T;
            uint32_t upto = mine;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(upto, o);
                if ((int)(threadIdx.x & 63) >= o) upto += t;
            }
            if ((threadIdx.x & 63) == 63) ties[u][threadIdx.x >> 6] = upto;
            rank[u] = upto - mine;
        }
        __syncthreads();
        uint32_t before = tie_off[blockIdx.x];
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int w = 0; w < MARK_NT / 64; ++w) {
                if (w == (int)(threadIdx.x >> 6)) rank[u] += before;
                before += ties[u][w];
            }
    }
#pragma unroll
    for (int u = 0; u < P; ++u) {
        const size_t f = f0 + (size_t)u * MARK_NT * V;
        uint32_t gone[V / 4] = {};   // a byte per value
#pragma unroll
        for (int e = 0; e < V; ++e) {
            bool g = keys[u][e] < T;
            if (keys[u][e] == T) { g = all || rank[u] < q_take; ++rank[u]; }
            gone[e / 4] |= (g ? 1u : 0u) << (8 * (e % 4));
            if (g && f + e < N) {
                W[f + e] = (TS)0;
                m1[f + e] = 0.f;
                m2[f + e] = 0.f;
            }
        }
        if (f + V <= N) {
#pragma unroll
            for (int q = 0; q < V / 4; ++q) *reinterpret_cast<uint32_t*>(flags + f + 4 * q) = gone[q];   // (flags is this library's own, f a multiple of 4)
        } else {
            for (int e = 0; e < V; ++e)
                if (f + e < N) flags[f + e] = (uint8_t)(gone[e / 4] >> (8 * (e % 4)));
        }
    }
}

// Per-row variant of the prune: GS lanes own one row (as in k_regrow); lane t ranks its own magnitude among the
// row's by (key, slot) with GS shuffles and gives up its slot if fewer than per_row rank below it.
template <int GS, typename TS>
__global__ void __launch_bounds__(256)
k_mark_rows(TS* __restrict__ W, float* __restrict__ m1, float* __restrict__ m2, int64_t m, int k, int per_row,
            uint8_t* __restrict__ flags) {
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t row = gid / GS;
    const int t = (int)(gid % GS);
    const int lane = threadIdx.x & 63;
    const int gbase = lane & ~(GS - 1);
    const bool active = row < m && t < k;
    const size_t f = (size_t)row * k + t;
    const uint32_t key = active ? mag_key<TS>(W, f) : 0xFFFFFFFFu;   // idle lanes rank last
    int rank = 0;
#pragma unroll
    for (int u = 0; u < GS; ++u) {
        const uint32_t other = (uint32_t)__shfl((int)key, gbase + u);
        rank += (other < key || (other == key && u < t)) ? 1 : 0;
    }
    if (active) {
        const bool gone = rank < per_row;
        flags[f] = gone ? 1 : 0;
        if (gone) { W[f] = (TS)0; m1[f] = 0.f; m2[f] = 0.f; }
    }
}

// any k: one thread per row; the flags of the whole row are settled before the first value is reset
template <typename TS>
__global__ void __launch_bounds__(256)
k_mark_rows_serial(TS* __restrict__ W, float* __restrict__ m1, float* __restrict__ m2, int64_t m, int k,
                   int per_row, uint8_t* __restrict__ flags) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= m) return;
    const size_t f0 = (size_t)row * k;
    for (int t = 0; t < k; ++t) {
        const uint32_t key = mag_key<TS>(W, f0 + t);
        int rank = 0;
        for (int u = 0; u < k; ++u) {
            const uint32_t other = mag_key<TS>(W, f0 + u);
            rank += (other < key || (other == key && u < t)) ? 1 : 0;
        }
        flags[f0 + t] = rank < per_row ? 1 : 0;
    }
    for (int t = 0; t < k; ++t)
        if (flags[f0 + t]) { W[f0 + t] = (TS)0; m1[f0 + t] = 0.f; m2[f0 + t] = 0.f; }
}

// ---- regrow ---------------------------------------------------------------------------------
// GS lanes own one row (GS = power of two >= k, <= 64); lane t of the group holds slot t.
// flags == nullptr means every slot is empty (initial connectivity).
// What bounds this is the vector unit.  The first candidates of a wavefront's empty slots are drawn together, every lane its own,
// and compared in one short loop; where two columns of a row clash, which is rare but in narrow layers, the wavefront goes slot
// by slot, drawing on.  (Slot by slot from the beginning, each candidate drawn by the whole group, took 109 us at m = 500k, d = 32k, k = 32,
// 5 % empty, between other kernels, now 69.  A list of eight turns' empty slots, drawn by as few lanes as could, took 62 there, but longer
// where slots clash or most are empty: m = 50k, d = 64, k = 64, one slot of ten 1425 us the call, now 1016; all slots of m = 500k, d = 32k,
// k = 32 268 and 201.)
// TURNS of rows to a wavefront: 8 in the largest layers, whose workgroups it saves (calls that redistribute 5 %, with one and eight:
// m = 3M, k = 32 1037 and 989 us; m = 670k, k = 64 483 and 442; m = 500k, k = 32 153 and 155; all slots of m = 100k, k = 32 64 and 96), unless
// the layer is narrow and its slots clash (m = 50k, d = 64, k = 64: 803 and 1004).
template <int GS> struct RowMask { typedef uint32_t T; };   // a bit per slot
template <> struct RowMask<64> { typedef uint64_t T; };
template <int GS, int TURNS>
__global__ void __launch_bounds__(256)
k_regrow(int32_t* __restrict__ idx, const uint8_t* __restrict__ flags, int64_t m, uint32_t d, int k,
         uint32_t k0, uint32_t k1, uint32_t epoch_lo) {
    typedef typename RowMask<GS>::T Mask;
    const Mask gmask = GS >= 32 ? (Mask)~(Mask)0 : (Mask)((1u << (GS & 31)) - 1u);
    const int lane = threadIdx.x & 63, t = lane & (GS - 1), gshift = lane & ~(GS - 1);
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (TURNS * 64 / GS) + lane / GS;
    auto of_row = [&](uint64_t ballot) { return (Mask)(ballot >> gshift) & gmask; };
    auto lowest = [&](Mask v) { return GS == 64 ? __ffsll((unsigned long long)v) - 1 : __ffs((int)v) - 1; };   // -1: none
    bool is[TURNS];   // my slot of the turn is empty
#pragma unroll
    for (int r = 0; r < TURNS; ++r) {
        const int64_t row = row0 + r * (64 / GS);
        is[r] = row < m && t < k && (flags ? flags[(size_t)row * k + t] != 0 : true);
    }
    int32_t columns[TURNS];   // of the full slots, or -1 (nobody asks for the columns of a full row)
#pragma unroll
    for (int r = 0; r < TURNS; ++r) {
        const int64_t row = row0 + r * (64 / GS);
        const Mask empty = of_row(__ballot(is[r]));   // (of all lanes: not behind a condition)
        columns[r] = -1;
        if (row < m && t < k && !is[r] && empty != 0) columns[r] = idx[(size_t)row * k + t];
    }
#pragma unroll
    for (int r = 0; r < TURNS; ++r) {
        const int64_t row = row0 + r * (64 / GS);
        const bool empty = is[r];
        Mask todo = of_row(__ballot(empty));   // empty slots of my row, bit = slot
        if (!__any(empty)) continue;
        int32_t mine = columns[r];
        const int32_t own = draw_column(k0, k1, epoch_lo, (uint32_t)row, (uint32_t)t, 0u, d);   // (full slots' are not asked for; a branch per lane took 5 % longer)
        int32_t* const at = idx + (size_t)row * k + t;
        {
            const int32_t have = empty ? own : mine;
            bool clash = false;
            for (Mask rest = todo; __any(rest != 0); rest &= rest - 1) {
                const int ts = lowest(rest);
                const int32_t c = __shfl(own, gshift + (ts & (GS - 1)));
                clash = clash || (rest != 0 && have == c && t != ts);
            }
            if (!__any(clash)) {
                if (empty) *at = own;
                continue;
            }
        }
        bool occupied = mine >= 0;
        uint32_t attempt = 0;
        while (__any(todo != 0)) {
            const int ts = todo ? lowest(todo) : 0;
            int32_t c = __shfl(own, gshift + ts);
            if (__any(attempt != 0)) {
                const int32_t next = draw_column(k0, k1, epoch_lo, (uint32_t)row, (uint32_t)ts, attempt, d);
                if (attempt != 0) c = next;
            }
            const Mask clash = of_row(__ballot(todo != 0 && occupied && mine == c));
            if (todo) {
                if (clash == 0) {
                    if (t == ts) { mine = c; occupied = true; }
                    todo &= todo - 1;
                    attempt = 0;
                } else {
                    ++attempt;
                }
            }
        }
        if (empty) *at = mine;
    }
}

// any k: one thread per row, row kept in global memory
__global__ void __launch_bounds__(256)
k_regrow_serial(int32_t* __restrict__ idx, uint8_t* __restrict__ flags_rw, int64_t m, uint32_t d, int k,
                uint32_t k0, uint32_t k1, uint32_t epoch_lo) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= m) return;
    int32_t* r = idx + row * k;
    uint8_t* e = flags_rw + row * k;  // 1 = empty; cleared as slots are filled
    for (int t = 0; t < k; ++t) {
        if (!e[t]) continue;
        for (uint32_t a = 0;; ++a) {
            const int32_t c = draw_column(k0, k1, epoch_lo, (uint32_t)row, (uint32_t)t, a, d);
            bool clash = false;
            for (int u = 0; u < k && !clash; ++u) clash = !e[u] && r[u] == c;
            if (!clash) { r[t] = c; e[t] = 0; break; }
        }
    }
}

__global__ void k_fill_u8(uint8_t* p, size_t n, uint8_t v) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t s = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += s) p[i] = v;
}

__global__ void __launch_bounds__(256)
k_validate(const int32_t* __restrict__ idx, int64_t m, int32_t d, int k, unsigned long long* bad) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= m) return;
    const int32_t* r = idx + row * k;
    bool b = false;
    for (int t = 0; t < k && !b; ++t) {
        const int32_t c = r[t];
        if (c < 0 || c >= d) { b = true; break; }
        for (int u = 0; u < t; ++u)
            if (r[u] == c) { b = true; break; }
    }
    if (b) atomicAdd(bad, 1ull);
}

usl_status regrow(usl_ctx* c, int32_t* idx, uint8_t* flags, bool all_empty, uint64_t seed,
                  uint64_t epoch) {
    const uint32_t k0 = (uint32_t)seed;
    const uint32_t k1 = (uint32_t)(seed >> 32) ^ (uint32_t)(epoch >> 32);
    const uint32_t elo = (uint32_t)epoch;
    const int k = c->k;
    if (k > 64) {
        const size_t N = (size_t)c->m * k;
        if (all_empty)
            hipLaunchKernelGGL(k_fill_u8, dim3(c->num_cu * 4), dim3(256), 0, c->stream, flags, N, (uint8_t)1);
        hipLaunchKernelGGL(k_regrow_serial, dim3((unsigned)((c->m + 255) / 256)), dim3(256), 0, c->stream,
                           idx, flags, c->m, (uint32_t)c->d, k, k0, k1, elo);
        return usl_check_launch(c, "regrow (serial)");
    }
    int gs = 1;
    while (gs < k) gs <<= 1;
    const uint8_t* fl = all_empty ? nullptr : flags;
    const int64_t lanes = c->m * gs;
    const bool many = lanes >= (int64_t)8 * 64 * 256 * c->num_cu && c->d >= 16 * k;   // see the kernel
    const int64_t per = many ? 256 * 8 : 256;
    const unsigned grid = (unsigned)((lanes + per - 1) / per);
#define USL_RG_T(GS, TURNS)                                                                    \
    hipLaunchKernelGGL((k_regrow<GS, TURNS>), dim3(grid), dim3(256), 0, c->stream, idx, fl, c->m, \
                       (uint32_t)c->d, k, k0, k1, elo)
#define USL_RG(GS) do { if (many) USL_RG_T(GS, 8); else USL_RG_T(GS, 1); } while (0)
    switch (gs) {
        case 1: USL_RG(1); break;
        case 2: USL_RG(2); break;
        case 4: USL_RG(4); break;
        case 8: USL_RG(8); break;
        case 16: USL_RG(16); break;
        case 32: USL_RG(32); break;
        default: USL_RG(64); break;
    }
#undef USL_RG
#undef USL_RG_T
    return usl_check_launch(c, "regrow");
}

usl_status ensure_flags(usl_ctx* c) {
    if (c->prune_flags) return USL_OK;
    size_t cap = 0;
    return usl_reserve(c, (void**)&c->prune_flags, &cap, (size_t)c->m * c->k);
}

template <typename TS>
usl_status redistribute_t(usl_ctx* c, int32_t* idx, TS* W, float* m1, float* m2, int64_t n,
                          uint64_t seed, uint64_t epoch) {
    const size_t N = (size_t)c->m * c->k;
    if (!c->sel_hist) {
        size_t cap = 0;
        USL_TRY(usl_reserve(c, (void**)&c->sel_hist, &cap, ST_WORDS * sizeof(uint32_t)));
    }
    USL_TRY(ensure_flags(c));
    const size_t nmark = (N + MARK_CHUNK - 1) / MARK_CHUNK;
    size_t cap = c->tie_counts_cap;
    USL_TRY(usl_reserve(c, (void**)&c->tie_counts, &cap, nmark * sizeof(uint32_t)));
    c->tie_counts_cap = cap;
    uint32_t* st = c->sel_hist;
    hipLaunchKernelGGL(k_sel_init, dim3(1), dim3(256), 0, c->stream, st, (uint32_t)n);
    // digits, most significant first: 31 magnitude bits of a float, 15 of a bfloat16
    const int f32_bits[3] = {11, 10, 10}, bf_bits[2] = {8, 7};
    const int npass = sizeof(TS) == 4 ? 3 : 2;
    const int* bits = sizeof(TS) == 4 ? f32_bits : bf_bits;
    int shift = sizeof(TS) == 4 ? 31 : 15;
    // few and large workgroups: each of them adds its bins to the same few words (four times as many of a quarter of the lanes:
    // 49, 31 and 31 us for the three digits of 16 million float32 weights, against 21, 14 and 14)
    size_t hblocks = (N + SEL_NT * 16 - 1) / (SEL_NT * 16);
    if (hblocks > (size_t)c->num_cu * 2) hblocks = (size_t)c->num_cu * 2;
    for (int p = 0; p < npass; ++p) {
        shift -= bits[p];
        hipLaunchKernelGGL(k_sel_hist<TS>, dim3((unsigned)hblocks), dim3(SEL_NT), 0, c->stream, W, N, st,
                           shift, bits[p], p == 0 ? 1 : 0);
        hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(256), 0, c->stream, st, bits[p]);
    }
    hipLaunchKernelGGL(k_tie_count<TS>, dim3((unsigned)nmark), dim3(MARK_NT), 0, c->stream, W, N, st,
                       c->tie_counts);
    hipLaunchKernelGGL(k_tie_scan, dim3(1), dim3(1024), 0, c->stream, c->tie_counts, nmark, st);
    hipLaunchKernelGGL(k_mark<TS>, dim3((unsigned)nmark), dim3(MARK_NT), 0, c->stream, W, m1, m2, N, st,
                       c->tie_counts, c->prune_flags);
    USL_TRY(usl_check_launch(c, "prune"));
    return regrow(c, idx, c->prune_flags, false, seed, epoch);
}

template <typename TS>
usl_status redistribute_rows_t(usl_ctx* c, int32_t* idx, TS* W, float* m1, float* m2, int per_row,
                               uint64_t seed, uint64_t epoch) {
    USL_TRY(ensure_flags(c));
    const int k = c->k;
    if (k > 64) {
        hipLaunchKernelGGL(k_mark_rows_serial<TS>, dim3((unsigned)((c->m + 255) / 256)), dim3(256), 0, c->stream,
                           W, m1, m2, c->m, k, per_row, c->prune_flags);
    } else {
        int gs = 1;
        while (gs < k) gs <<= 1;
        const unsigned grid = (unsigned)((c->m * gs + 255) / 256);
#define USL_MR(GS)                                                                                       \
    hipLaunchKernelGGL((k_mark_rows<GS, TS>), dim3(grid), dim3(256), 0, c->stream, W, m1, m2, c->m, k,   \
                       per_row, c->prune_flags)
        switch (gs) {
            case 1: USL_MR(1); break;
            case 2: USL_MR(2); break;
            case 4: USL_MR(4); break;
            case 8: USL_MR(8); break;
            case 16: USL_MR(16); break;
            case 32: USL_MR(32); break;
            default: USL_MR(64); break;
        }
#undef USL_MR
    }
    USL_TRY(usl_check_launch(c, "prune (per row)"));
    return regrow(c, idx, c->prune_flags, false, seed, epoch);
}

}  // namespace

usl_status usl_launch_redistribute(usl_ctx* c, int32_t* idx, void* W, float* m1, float* m2,
                                   int64_t n, uint64_t seed, uint64_t epoch) {
    return c->storage == USL_F32
               ? redistribute_t<float>(c, idx, (float*)W, m1, m2, n, seed, epoch)
               : redistribute_t<uint16_t>(c, idx, (uint16_t*)W, m1, m2, n, seed, epoch);
}

usl_status usl_launch_redistribute_rows(usl_ctx* c, int32_t* idx, void* W, float* m1, float* m2,
                                        int32_t per_row, uint64_t seed, uint64_t epoch) {
    return c->storage == USL_F32
               ? redistribute_rows_t<float>(c, idx, (float*)W, m1, m2, per_row, seed, epoch)
               : redistribute_rows_t<uint16_t>(c, idx, (uint16_t*)W, m1, m2, per_row, seed, epoch);
}

usl_status usl_launch_init_indices(usl_ctx* c, int32_t* idx, uint64_t seed) {
    if (c->k > 64) USL_TRY(ensure_flags(c));
    return regrow(c, idx, c->prune_flags, true, seed, ~(uint64_t)0);
}

usl_status usl_launch_validate(usl_ctx* c, const int32_t* idx, int64_t* n_bad_host) {
    if (!c->counter64) {
        size_t cap = 0;
        USL_TRY(usl_reserve(c, (void**)&c->counter64, &cap, 64));
    }
    hipLaunchKernelGGL(k_fill_u8, dim3(1), dim3(64), 0, c->stream, (uint8_t*)c->counter64, (size_t)8, (uint8_t)0);
    hipLaunchKernelGGL(k_validate, dim3((unsigned)((c->m + 255) / 256)), dim3(256), 0, c->stream, idx,
                       c->m, c->d, c->k, (unsigned long long*)c->counter64);
    USL_TRY(usl_check_launch(c, "validate"));
    int64_t v = 0;
    USL_HIP(c, hipMemcpyAsync(&v, c->counter64, 8, hipMemcpyDeviceToHost, c->stream));
    USL_HIP(c, hipStreamSynchronize(c->stream));
    *n_bad_host = v;
    return USL_OK;
}

usl_status usl_launch_philox(usl_ctx* c, const uint32_t* ctr, uint32_t key0, uint32_t key1,
                             uint32_t* out, int64_t n) {
    hipLaunchKernelGGL(k_philox, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, ctr, key0,
                       key1, out, n);
    return usl_check_launch(c, "philox");
}
