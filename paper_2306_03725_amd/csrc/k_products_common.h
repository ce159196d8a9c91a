// Device code of the forward and weight-gradient kernels.
//
// Both walk the same gather: for a pair (instance i, label j) the k values x[i][idx[j][t]].  A workgroup owns a block
// of labels and keeps their indices (two 16-bit columns per register) and weights -- or gradient sums -- in registers
// for its whole life; the activations stream through LDS, and every gather is an LDS read.
//
// What bounds it is the number of LDS reads, not their width: a ds_read_b64 of 64 random addresses takes as long as a
// ds_read_b32 (8.7 lanes per clock and compute unit both; 25 both when no two lanes of a pass meet in a bank), a
// ds_read_b128 little longer (5.1 and 14.7; all measured by csrc/ceilings.hip).  So the activations are interleaved: Q instances form a group,
// and the group's row holds x[i0][c], x[i0+1][c], ... side by side, one unit of 4, 8 or 16 bytes per column, which one
// read brings to a lane.  A row of units has to fit LDS (160 KB):
//     float32   Q = 4 up to d = 10 200,  Q = 2 up to 20 400,  Q = 1 up to 40 800,  beyond that the row in two halves
//     bfloat16  Q = 4 up to d = 20 400,  Q = 2 up to 40 800,  Q = 1 up to 65 536
// The interleaved copy of x (k_interleave, [groups][row], rows padded to 16 bytes and, where the fan-in is padded, by a
// column of zeros) costs one pass over b * d values; it also takes the alignment of d out of the row copies.  Q = 1
// needs no copy when rows of x are 16-byte aligned already.
//
// Fan-ins are padded to K, the next multiple of 8 up to 32, 48 or 64; padding slots have weight 0 and read the column of
// zeros (a real column times weight 0 would make NaN of an infinity that the label has no connection to).
#pragma once
#include <type_traits>

#include "usl_internal.h"

namespace usl_products {

struct Geom {
    int row_bytes;         // bytes from one group's row to the next in the interleaved activations (a multiple of 16)
    int tile_rows;         // rows staged together (small rows)
    int nbuf;              // 2: the next tile is copied in while this one is gathered
    int buf_bytes;         // LDS bytes from one buffer to the next
    int groups;            // instance groups of the batch
    int groups_per_block;  // ... that one workgroup walks
    int share;             // workgroups resident together on one XCD that walk the same rows: they split the warm-up of the next row
    int zero_col;          // column that padding slots read (a unit of zeros)
    int parts_first;       // blockIdx.x is the part of the batch and blockIdx.y the block of labels, not the other way round
    int dummy;             // 256 bytes of LDS that the warm-up loads are thrown into
};
// The blocks of labels from `first` on (INT_MAX: none), `blocks` of them, take the batch in parts of `groups` groups: blockIdx.x
// runs over them part by part, behind the others.  (Forward's alone: as part of Geom it made the compiler's weight gradient
// 3 % slower at m = 500k, d = 32k.)
struct Tail {
    int first, blocks, groups, share;
    int labels;            // of any block: at most its lanes times the labels of a lane, a multiple of 32
};

static constexpr int ROW_LDS_MAX = 160 * 1024 - 512;    // largest tile
static constexpr int HALF_COLS = 32768;                 // columns per half of a row in two halves

// --------------------------------------------------------------------------------------------- row copies
// nbytes (a multiple of 16) from global memory to LDS, both 16-byte aligned, by global_load_lds_dwordx4: each wavefront
// moves 1 KiB per instruction, no registers are used, all of it is in flight together.  In the last instruction the
// lanes past the end are masked off.  The caller waits (vmcnt) before its barrier.  Inline assembly: behind the builtin
// the compiler waits for the copy before the next LDS read of any address, so nothing would overlap it.
// M0 is written here without being listed as clobbered: the compiler holds it in reserve and takes no clobber of it, and
// sets it itself only where it emits an instruction that reads it.  No kernel of these files does (no LDS-DMA builtin, no
// register index known at run time only); tests/test_listing_m0.py looks at what the compiler made.
__device__ __forceinline__ void stage_async(const char* __restrict__ src, uint32_t lds, int nbytes, int tid, int nt) {
    for (int v = (tid >> 6) * 1024; v < nbytes; v += (nt / 64) * 1024) {
        const uint32_t off = (uint32_t)(v + (tid & 63) * 16);
        const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds + (uint32_t)v));
        if ((int)off < nbytes)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(src) : "memory");
    }
}

// Touches one word of every 128-byte line of [row + first line * 128, + n lines): the words go to `dummy` (256 bytes of
// LDS that nobody reads), so no register waits for them.
template <int NT>
__device__ __forceinline__ void touch_lines(const char* __restrict__ row, int first, int n, uint32_t dummy, int tid) {
    const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)dummy);
    for (int l = tid; l < n; l += NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"((uint32_t)(first + l) * 128u), "s"(row) : "memory");
}

// Warms the L2 of this workgroup's XCD with a share of the next tile.  All workgroups walk the batch in step, so without
// this every row is first touched by all of them at once and the whole chip waits out an HBM round trip per row.
// Workgroups are dealt to the 8 XCDs round robin; those of one XCD that walk the same rows and are resident together
// split the row between them, one load per 128-byte line.
struct WarmShare {
    int slice, slices;
    __device__ __forceinline__ WarmShare(uint32_t at, int share) : slice((int)at % share), slices(share) {}
    __device__ __forceinline__ explicit WarmShare(const Geom& tg)   // no tail
        : WarmShare(tg.parts_first ? blockIdx.y : blockIdx.x >> 3, tg.share) {}
    // first and number of this workgroup's lines of a tile of nbytes
    __device__ __forceinline__ int per(int nbytes) const { return ((nbytes + 127) / 128 + slices - 1) / slices; }
};
// A workgroup of forward: its block of labels, and its groups g0 .. g1 - 1 of the batch.  (The weight gradient has no tail: its
// parts would have to be added up.)
struct Turn {
    uint32_t block;
    int g0, g1;
    uint32_t warm_at;   // number among the workgroups that share the warm-up
    int warm_share;
    __device__ __forceinline__ Turn(const Geom& tg, const Tail& tail) {
        block = tg.parts_first ? blockIdx.y : blockIdx.x;
        uint32_t part = tg.parts_first ? blockIdx.x : blockIdx.y, at = block;
        int groups = tg.groups_per_block;
        warm_share = tg.share;
        if (__builtin_expect(block >= (uint32_t)tail.first, 0)) {
            at -= (uint32_t)tail.first;
            part = at / (uint32_t)tail.blocks;   // (with a loop of subtractions the step at m = 500k, b = 256 took 1 % longer)
            at %= (uint32_t)tail.blocks;
            block = (uint32_t)tail.first + at;
            groups = tail.groups;
            warm_share = tail.share;
        }
        warm_at = tg.parts_first ? at : at >> 3;
        g0 = (int)part * groups;
        g1 = min(tg.groups, g0 + groups);
    }
};
template <int NT>
__device__ __forceinline__ void warm_slice(const char* __restrict__ row, int nbytes, int per, int slice, uint32_t dummy, int tid) {
    touch_lines<NT>(row, slice * per, min(per, (nbytes + 127) / 128 - slice * per), dummy, tid);
}

// --------------------------------------------------------------------------------------------- labels into registers
// Private slot order of one label: K bytes (slot visited at step s).  A null table means stored order.
template <int K>
struct SlotOrder {
    uint32_t w[K / 4];
    bool on;
    __device__ __forceinline__ void load(const uint8_t* __restrict__ perm, int64_t j, bool valid) {
        on = perm != nullptr;
        if (on) {
            const uint2* p = reinterpret_cast<const uint2*>(perm + j * K);
#pragma unroll
            for (int q = 0; q < K / 8; ++q) {
                const uint2 u = valid ? p[q] : make_uint2(0x03020100u + 0x08080808u * q, 0x07060504u + 0x08080808u * q);
                w[2 * q] = u.x;
                w[2 * q + 1] = u.y;
            }
        }
    }
    __device__ __forceinline__ int at(int s) const { return on ? (int)((w[s >> 2] >> (8 * (s & 3))) & 0xFFu) : s; }
};

// The rows of 64 consecutive labels go through a piece of LDS that belongs to the wavefront alone: coalesced loads in,
// every lane reads its own row out (odd row strides, no bank conflicts), no barrier of the workgroup in between.
// Rows of 32-bit words take more LDS than rows of 16-bit ones, so for K > 32 the wavefronts take two turns.
template <int K> constexpr int turns_of() { return K > 32 ? 2 : 1; }
template <int K> constexpr int words_stride() { return K + 1; }        // words per row of 32-bit values
template <int K> constexpr int halves_stride() { return K / 2 + 1; }   // words per row of 16-bit values
// LDS one wavefront's rows take (32-bit rows, shared between the turns)
template <int K, int NT> constexpr int transpose_bytes() {
    constexpr int waves = NT / 64;
    constexpr int w32 = (waves + turns_of<K>() - 1) / turns_of<K>() * 64 * words_stride<K>() * 4;
    constexpr int w16 = waves * 64 * halves_stride<K>() * 4;
    return w32 > w16 ? w32 : w16;
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The prologue brings the rows of a wavefront's 64 labels in: order, indices and weights are requested together
// (coalesced; one trip to memory instead of three in a row), then indices and weights go through LDS.
template <typename TS, int K, int NT> constexpr bool raw_rows() {
    return (K & (K - 1)) == 0 && (sizeof(TS) == 2 ? K <= 32 || NT < 1024 : K <= 32 && NT < 1024);
}
template <typename TS, int K>
struct RawRows {
    SlotOrder<K> so;
    uint32_t idx[K];
    uint32_t w[sizeof(TS) == 4 ? K : K / 2];

    // 16-byte (bfloat16: 8-byte) pieces where k is a multiple of 4, single values elsewhere
    __device__ __forceinline__ void load_idx(const uint8_t* __restrict__ perm, const int32_t* __restrict__ ip, int64_t row0, int64_t m,
                                             int k, uint32_t zero_col) {
        const int lane = threadIdx.x & 63;
        const int64_t wrow0 = row0 + (threadIdx.x & ~63);
        so.load(perm, row0 + threadIdx.x, row0 + threadIdx.x < m);
        if ((k & 3) == 0) {
            constexpr int U = K / 4;   // 4-slot pieces per (padded) row
#pragma unroll
            for (int it = 0; it < U; ++it) {
                const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
                uint4 q = make_uint4(zero_col, zero_col, zero_col, zero_col);
                if (wrow0 + r < m && t < k) q = *reinterpret_cast<const uint4*>(ip + (wrow0 + r) * k + t);
                idx[4 * it] = q.x; idx[4 * it + 1] = q.y; idx[4 * it + 2] = q.z; idx[4 * it + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int it = 0; it < K; ++it) {
                const int u = it * 64 + lane, r = u / K, t = u % K;
                idx[it] = wrow0 + r < m && t < k ? (uint32_t)ip[(wrow0 + r) * k + t] : zero_col;
            }
        }
    }
    __device__ __forceinline__ void load_w(const TS* __restrict__ W, int64_t row0, int64_t m, int k) {
        const int lane = threadIdx.x & 63;
        const int64_t wrow0 = row0 + (threadIdx.x & ~63);
        if ((k & 3) == 0) {
            constexpr int U = K / 4;
#pragma unroll
            for (int it = 0; it < U; ++it) {
                const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
                const bool in = wrow0 + r < m && t < k;
                if constexpr (sizeof(TS) == 4) {
                    uint4 v = make_uint4(0, 0, 0, 0);
                    if (in) v = *reinterpret_cast<const uint4*>(W + (wrow0 + r) * k + t);
                    w[4 * it] = v.x; w[4 * it + 1] = v.y; w[4 * it + 2] = v.z; w[4 * it + 3] = v.w;
                } else {
                    uint2 v = make_uint2(0, 0);
                    if (in) v = *reinterpret_cast<const uint2*>(W + (wrow0 + r) * k + t);
                    w[2 * it] = v.x; w[2 * it + 1] = v.y;
                }
            }
        } else {
#pragma unroll
            for (int it = 0; it < K; ++it) {
                const int u = it * 64 + lane, r = u / K, t = u % K;
                const bool in = wrow0 + r < m && t < k;
                if constexpr (sizeof(TS) == 4) w[it] = in ? __float_as_uint(W[(wrow0 + r) * k + t]) : 0u;
                else if (it & 1) w[it / 2] |= in ? (uint32_t)W[(wrow0 + r) * k + t] << 16 : 0u;
                else w[it / 2] = in ? (uint32_t)W[(wrow0 + r) * k + t] : 0u;
            }
        }
    }
};

// pk[q] = columns of steps 2q, 2q+1 of label row0 + threadIdx.x (16 bits each), in the label's slot order.
template <int K, typename TS>
__device__ __forceinline__ void unpack_idx(const RawRows<TS, K>& raw, int k, uint32_t* lds, uint32_t (&pk)[K / 2]) {
    constexpr int S = halves_stride<K>();
    const int lane = threadIdx.x & 63;
    uint16_t* mine = reinterpret_cast<uint16_t*>(lds + (threadIdx.x >> 6) * 64 * S);
    if ((k & 3) == 0) {
        constexpr int U = K / 4;
#pragma unroll
        for (int it = 0; it < U; ++it) {
            const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
            uint32_t* p = reinterpret_cast<uint32_t*>(mine) + r * S + t / 2;
            p[0] = (raw.idx[4 * it] & 0xFFFFu) | (raw.idx[4 * it + 1] << 16);
            p[1] = (raw.idx[4 * it + 2] & 0xFFFFu) | (raw.idx[4 * it + 3] << 16);
        }
    } else {
#pragma unroll
        for (int it = 0; it < K; ++it) {
            const int u = it * 64 + lane, r = u / K, t = u % K;
            mine[r * 2 * S + t] = (uint16_t)raw.idx[it];
        }
    }
    wave_sync();
    const uint16_t* p = mine + lane * 2 * S;
#pragma unroll
    for (int q = 0; q < K / 2; ++q) {
        pk[q] = (uint32_t)p[raw.so.at(2 * q)] | ((uint32_t)p[raw.so.at(2 * q + 1)] << 16);
        if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // a few addresses at a time: all of them would not fit
    }
    wave_sync();
}

// w[s] = weight of step s, float32 (0 for padding slots and labels past m).  All threads of the workgroup call it.
template <int K, int NT>
__device__ __forceinline__ void unpack_w(const RawRows<float, K>& raw, int k, uint32_t* lds, float (&w)[K]) {
    constexpr int S = words_stride<K>(), T = turns_of<K>(), WAVES = NT / 64, PER = (WAVES + T - 1) / T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t* mine = lds + (wave % PER) * 64 * S;
#pragma unroll 1
    for (int turn = 0; turn < T; ++turn) {
        __syncthreads();
        if (wave / PER != turn) continue;
        if ((k & 3) == 0) {
            constexpr int U = K / 4;
#pragma unroll
            for (int it = 0; it < U; ++it) {
                const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
                uint32_t* p = mine + r * S + t;
                p[0] = raw.w[4 * it]; p[1] = raw.w[4 * it + 1]; p[2] = raw.w[4 * it + 2]; p[3] = raw.w[4 * it + 3];
            }
        } else {
#pragma unroll
            for (int it = 0; it < K; ++it) {
                const int u = it * 64 + lane, r = u / K, t = u % K;
                mine[r * S + t] = raw.w[it];
            }
        }
        wave_sync();
        const uint32_t* p = mine + lane * S;
#pragma unroll
        for (int s = 0; s < K; ++s) {
            w[s] = __uint_as_float(p[raw.so.at(s)]);
            if ((s & 7) == 7) __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
    }
    __syncthreads();
}
// The same two where the raw rows would not fit beside what is resident (K > 32, or 128 registers a lane), a few pieces at
// a time, and for a K that is no power of two: there the unrolled address arithmetic made the raw form slower (75 -> 97 us
// for the forward product at m = 70k, d = 10k, k = 48, b = 100).
template <int K>
__device__ __forceinline__ void fetch_idx(const int32_t* __restrict__ idx, int64_t row0, int64_t m, int k, uint32_t zero_col,
                                          uint32_t* lds, const SlotOrder<K>& so, uint32_t (&pk)[K / 2]) {
    constexpr int S = halves_stride<K>();
    const int lane = threadIdx.x & 63;
    uint16_t* mine = reinterpret_cast<uint16_t*>(lds + (threadIdx.x >> 6) * 64 * S);
    const int64_t wrow0 = row0 + (threadIdx.x & ~63);
    if ((k & 3) == 0) {
        constexpr int U = K / 4;
#pragma unroll 4
        for (int it = 0; it < U; ++it) {
            const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
            uint4 q = make_uint4(zero_col, zero_col, zero_col, zero_col);
            if (wrow0 + r < m && t < k) q = *reinterpret_cast<const uint4*>(idx + (wrow0 + r) * k + t);
            uint32_t* p = reinterpret_cast<uint32_t*>(mine) + r * S + t / 2;
            p[0] = (q.x & 0xFFFFu) | (q.y << 16);
            p[1] = (q.z & 0xFFFFu) | (q.w << 16);
        }
    } else {
#pragma unroll 4
        for (int it = 0; it < K; ++it) {
            const int u = it * 64 + lane, r = u / K, t = u % K;
            mine[r * 2 * S + t] = (uint16_t)(wrow0 + r < m && t < k ? (uint32_t)idx[(wrow0 + r) * k + t] : zero_col);
        }
    }
    wave_sync();
    const uint16_t* p = mine + lane * 2 * S;
#pragma unroll
    for (int q = 0; q < K / 2; ++q) {
        pk[q] = (uint32_t)p[so.at(2 * q)] | ((uint32_t)p[so.at(2 * q + 1)] << 16);
        if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_sync();
}
template <int K, int NT>
__device__ __forceinline__ void fetch_w(const float* __restrict__ W, int64_t row0, int64_t m, int k, uint32_t* lds,
                                        const SlotOrder<K>& so, float (&w)[K]) {
    constexpr int S = words_stride<K>(), T = turns_of<K>(), WAVES = NT / 64, PER = (WAVES + T - 1) / T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t wrow0 = row0 + (threadIdx.x & ~63);
    uint32_t* mine = lds + (wave % PER) * 64 * S;
#pragma unroll 1
    for (int turn = 0; turn < T; ++turn) {
        __syncthreads();
        if (wave / PER != turn) continue;
        if ((k & 3) == 0) {
            constexpr int U = K / 4;
#pragma unroll 4
            for (int it = 0; it < U; ++it) {
                const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
                uint4 q = make_uint4(0, 0, 0, 0);
                if (wrow0 + r < m && t < k) q = *reinterpret_cast<const uint4*>(W + (wrow0 + r) * k + t);
                uint32_t* p = mine + r * S + t;
                p[0] = q.x; p[1] = q.y; p[2] = q.z; p[3] = q.w;
            }
        } else {
#pragma unroll 4
            for (int it = 0; it < K; ++it) {
                const int u = it * 64 + lane, r = u / K, t = u % K;
                mine[r * S + t] = wrow0 + r < m && t < k ? __float_as_uint(W[(wrow0 + r) * k + t]) : 0u;
            }
        }
        wave_sync();
        const uint32_t* p = mine + lane * S;
#pragma unroll
        for (int s = 0; s < K; ++s) {
            w[s] = __uint_as_float(p[so.at(s)]);
            if ((s & 7) == 7) __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
    }
    __syncthreads();
}
template <int K, int NT>
__device__ __forceinline__ void fetch_w(const uint16_t* __restrict__ W, int64_t row0, int64_t m, int k, uint32_t* lds,
                                        const SlotOrder<K>& so, uint32_t (&wp)[K / 2]) {
    constexpr int S = halves_stride<K>();
    const int lane = threadIdx.x & 63;
    uint16_t* mine = reinterpret_cast<uint16_t*>(lds + (threadIdx.x >> 6) * 64 * S);
    const int64_t wrow0 = row0 + (threadIdx.x & ~63);
    if ((k & 3) == 0) {
        constexpr int U = K / 4;
#pragma unroll 4
        for (int it = 0; it < U; ++it) {
            const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
            uint2 q = make_uint2(0, 0);
            if (wrow0 + r < m && t < k) q = *reinterpret_cast<const uint2*>(W + (wrow0 + r) * k + t);
            uint32_t* p = reinterpret_cast<uint32_t*>(mine) + r * S + t / 2;
            p[0] = q.x; p[1] = q.y;
        }
    } else {
#pragma unroll 4
        for (int it = 0; it < K; ++it) {
            const int u = it * 64 + lane, r = u / K, t = u % K;
            mine[r * 2 * S + t] = wrow0 + r < m && t < k ? W[(wrow0 + r) * k + t] : (uint16_t)0;
        }
    }
    wave_sync();
    const uint16_t* p = mine + lane * 2 * S;
#pragma unroll
    for (int q = 0; q < K / 2; ++q) {
        wp[q] = (uint32_t)p[so.at(2 * q)] | ((uint32_t)p[so.at(2 * q + 1)] << 16);
        if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_sync();
}
// bfloat16 weights stay in pairs: wp[q] = weights of steps 2q (low half) and 2q+1.
template <int K, int NT>
__device__ __forceinline__ void unpack_w(const RawRows<uint16_t, K>& raw, int k, uint32_t* lds, uint32_t (&wp)[K / 2]) {
    constexpr int S = halves_stride<K>();
    const int lane = threadIdx.x & 63;
    uint16_t* mine = reinterpret_cast<uint16_t*>(lds + (threadIdx.x >> 6) * 64 * S);
    if ((k & 3) == 0) {
        constexpr int U = K / 4;
#pragma unroll
        for (int it = 0; it < U; ++it) {
            const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
            uint32_t* p = reinterpret_cast<uint32_t*>(mine) + r * S + t / 2;
            p[0] = raw.w[2 * it]; p[1] = raw.w[2 * it + 1];
        }
    } else {
#pragma unroll
        for (int it = 0; it < K; ++it) {
            const int u = it * 64 + lane, r = u / K, t = u % K;
            mine[r * 2 * S + t] = (uint16_t)(raw.w[it / 2] >> (16 * (it & 1)));
        }
    }
    wave_sync();
    const uint16_t* p = mine + lane * 2 * S;
#pragma unroll
    for (int q = 0; q < K / 2; ++q) {
        wp[q] = (uint32_t)p[raw.so.at(2 * q)] | ((uint32_t)p[raw.so.at(2 * q + 1)] << 16);
        if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    wave_sync();
}
// The reverse: acc[s] of every lane becomes row row0 + threadIdx.x of dst[m][k].  All threads of the workgroup call it.
template <int K, int NT>
__device__ __forceinline__ void store_rows(const float (&acc)[K], float* __restrict__ dst, int64_t row0, int64_t m, int k,
                                           uint32_t* lds, const SlotOrder<K>& so) {
    constexpr int S = words_stride<K>(), T = turns_of<K>(), WAVES = NT / 64, PER = (WAVES + T - 1) / T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t wrow0 = row0 + (threadIdx.x & ~63);
    uint32_t* mine = lds + (wave % PER) * 64 * S;
    for (int turn = 0; turn < T; ++turn) {
        __syncthreads();
        if (wave / PER != turn) continue;
        uint32_t* p = mine + lane * S;
#pragma unroll
        for (int s = 0; s < K; ++s) {
            p[so.at(s)] = __float_as_uint(acc[s]);
            if ((s & 7) == 7) __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
        if ((k & 3) == 0) {
            constexpr int U = K / 4;
#pragma unroll 4
            for (int it = 0; it < U; ++it) {
                const int u = it * 64 + lane, r = u / U, t = (u % U) * 4;
                const uint32_t* q = mine + r * S + t;
                if (wrow0 + r < m && t < k)
                    *reinterpret_cast<float4*>(dst + (wrow0 + r) * k + t) =
                        make_float4(__uint_as_float(q[0]), __uint_as_float(q[1]), __uint_as_float(q[2]), __uint_as_float(q[3]));
            }
        } else {
#pragma unroll 4
            for (int it = 0; it < K; ++it) {
                const int u = it * 64 + lane, r = u / K, t = u % K;
                if (wrow0 + r < m && t < k) dst[(wrow0 + r) * k + t] = __uint_as_float(mine[r * S + t]);
            }
        }
        wave_sync();
    }
    __syncthreads();
}

// --------------------------------------------------------------------------------------------- gathers
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <typename TS, int Q> struct Unit;                      // what one LDS read brings: Q instances of one column
template <> struct Unit<float, 1> { typedef float T; };
template <> struct Unit<float, 2> { typedef f32x2 T; };
template <> struct Unit<float, 4> { typedef f32x4 T; };
template <> struct Unit<uint16_t, 1> { typedef uint16_t T; };
template <> struct Unit<uint16_t, 2> { typedef uint32_t T; };
template <> struct Unit<uint16_t, 4> { typedef u32x2 T; };

template <typename T>
__device__ __forceinline__ T lds_read(uint32_t byte_addr) {
    typedef const __attribute__((address_space(3))) T lds_t;
    return *reinterpret_cast<lds_t*>(static_cast<uintptr_t>(byte_addr));
}

// LDS address of step t: base + column * BYTES, one instruction (16-bit multiply-add that picks either half of the word).
template <int BYTES, int N>
__device__ __forceinline__ uint32_t unit_addr(const uint32_t (&pk)[N], int t, uint32_t base) {
    uint32_t a;
    if (t & 1) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(a) : "v"(pk[t >> 1]), "n"(BYTES), "s"(base));
    else       asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(a) : "v"(pk[t >> 1]), "n"(BYTES), "s"(base));
    return a;
}

// Stops the compiler from hoisting the unpacked addresses out of the loop over the batch: rebuilding one is a single
// instruction, holding all of them would double the register need.
template <int N>
__device__ __forceinline__ void keep_packed(uint32_t (&pk)[N]) {
#pragma unroll
    for (int q = 0; q < N; ++q) asm volatile("" : "+v"(pk[q]));
}
// Reads in flight per wavefront: their results would otherwise crowd out the resident indices and weights.
template <typename TS, int Q> constexpr int batch_of() { return sizeof(typename Unit<TS, Q>::T) == 16 ? 4 : 8; }

// HALVES: a float32 row of more than ROW_LDS_MAX in two halves of HALF_COLS columns; a step of the half that is not
// staged reads one word of zeros behind the buffer (the same word for every lane: one broadcast).  While the upper
// half is staged the base is HALF_COLS words lower, so a column of the lower half wraps round to a huge address, and "in
// this half" is one unsigned minimum both times.
template <typename TS, int Q, bool HALVES, int N>
__device__ __forceinline__ typename Unit<TS, Q>::T gather(const uint32_t (&pk)[N], int t, uint32_t base, uint32_t zbyte) {
    typedef typename Unit<TS, Q>::T U;
    uint32_t a = unit_addr<(int)sizeof(U)>(pk, t, base);
    if (HALVES) a = a < zbyte ? a : zbyte;
    return lds_read<U>(a);
}

template <bool HALVES, int B, int ARITH>
__device__ __forceinline__ void schedule_batch() {   // the addresses of a batch, its reads, then the arithmetic
    __builtin_amdgcn_sched_group_barrier(0x002, HALVES ? 2 * B : B, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, B, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, ARITH, 0);
    __builtin_amdgcn_sched_barrier(0);
}

// acc[q] += sum over the label's steps of w * x[instance q]
template <int K, int Q, bool HALVES>
__device__ __forceinline__ void label_dot(const uint32_t (&pk)[K / 2], const float (&w)[K], uint32_t base, uint32_t zbyte, float (&acc)[Q]) {
    constexpr int B = batch_of<float, Q>();
    typedef typename Unit<float, Q>::T U;
#pragma unroll
    for (int t0 = 0; t0 < K; t0 += B) {
        U v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = gather<float, Q, HALVES>(pk, t0 + u, base, zbyte);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if constexpr (Q == 1) acc[0] = fmaf(w[t0 + u], v[u], acc[0]);
            else {
#pragma unroll
                for (int q = 0; q < Q; ++q) acc[q] = fmaf(w[t0 + u], v[u][q], acc[q]);
            }
        }
        schedule_batch<HALVES, B, B * Q>();
    }
}
// bfloat16: the activations of two steps are joined per instance and one dot-product instruction does both
// multiply-adds in float32.
__device__ __forceinline__ float dot2(uint32_t x2, uint32_t w2, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x2), __builtin_bit_cast(bf16x2, w2), acc, false);
}
__device__ __forceinline__ uint32_t join_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t join_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
template <int K, int Q, bool HALVES>
__device__ __forceinline__ void label_dot(const uint32_t (&pk)[K / 2], const uint32_t (&wp)[K / 2], uint32_t base, uint32_t zbyte, float (&acc)[Q]) {
    constexpr int B = 8;
    typedef typename Unit<uint16_t, Q>::T U;
#pragma unroll
    for (int t0 = 0; t0 < K; t0 += B) {
        U v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = gather<uint16_t, Q, HALVES>(pk, t0 + u, base, zbyte);
#pragma unroll
        for (int u = 0; u < B; u += 2) {
            const uint32_t w2 = wp[(t0 + u) / 2];
            if constexpr (Q == 1) acc[0] = dot2((uint32_t)v[u] | ((uint32_t)v[u + 1] << 16), w2, acc[0]);
            else if constexpr (Q == 2) {
                acc[0] = dot2(join_lo(v[u], v[u + 1]), w2, acc[0]);
                acc[1] = dot2(join_hi(v[u], v[u + 1]), w2, acc[1]);
            } else {
                acc[0] = dot2(join_lo(v[u].x, v[u + 1].x), w2, acc[0]);
                acc[1] = dot2(join_hi(v[u].x, v[u + 1].x), w2, acc[1]);
                acc[2] = dot2(join_lo(v[u].y, v[u + 1].y), w2, acc[2]);
                acc[3] = dot2(join_hi(v[u].y, v[u + 1].y), w2, acc[3]);
            }
        }
        schedule_batch<HALVES, B, B * Q>();
    }
}

// acc[s] += sum over the group's instances of g[q] * x[instance q]
template <int K, typename TS, int Q, bool HALVES>
__device__ __forceinline__ void label_outer(const uint32_t (&pk)[K / 2], const float (&gv)[Q], uint32_t base, uint32_t zbyte, float (&acc)[K]) {
    constexpr int B = batch_of<TS, Q>();
    typedef typename Unit<TS, Q>::T U;
#pragma unroll
    for (int t0 = 0; t0 < K; t0 += B) {
        U v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = gather<TS, Q, HALVES>(pk, t0 + u, base, zbyte);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            float& a = acc[t0 + u];
            if constexpr (sizeof(TS) == 4 && Q == 1) a = fmaf(gv[0], v[u], a);
            else if constexpr (sizeof(TS) == 4) {
#pragma unroll
                for (int q = 0; q < Q; ++q) a = fmaf(gv[q], v[u][q], a);
            } else if constexpr (Q == 1) a = fmaf(gv[0], usl_bf16_to_f32(v[u]), a);
            else if constexpr (Q == 2) {
                a = fmaf(gv[0], __uint_as_float(v[u] << 16), a);
                a = fmaf(gv[1], __uint_as_float(v[u] & 0xFFFF0000u), a);
            } else {
                a = fmaf(gv[0], __uint_as_float(v[u].x << 16), a);
                a = fmaf(gv[1], __uint_as_float(v[u].x & 0xFFFF0000u), a);
                a = fmaf(gv[2], __uint_as_float(v[u].y << 16), a);
                a = fmaf(gv[3], __uint_as_float(v[u].y & 0xFFFF0000u), a);
            }
        }
        schedule_batch<HALVES, B, B * Q>();
    }
}

// --------------------------------------------------------------------------------------------- the walk over the batch
// Calls body(group, first LDS byte of its row, part) for every instance group of this part of the batch, with the rows staged
// tile by tile; late(first group of the tile, groups in it, lane) right after a tile has arrived, early(first group,
// groups) right before the wait for it: what is loaded there can be waited for at no cost.
// MULTI = false: one row fills the buffer (tiles of one row, one buffer); HALVES: part 0 / 1 of every row.
template <int NT, bool MULTI, bool HALVES, typename BODY, typename LATE, typename EARLY>
__device__ __forceinline__ void walk(const char* __restrict__ xi, uint32_t lds0, const Geom& tg, const WarmShare& ws, int g0, int g1, BODY body, LATE late, EARLY early) {
    const uint32_t dummy = lds0 + (uint32_t)tg.dummy;
    if (!MULTI) {
        const int per = ws.per(tg.row_bytes);
        constexpr int HB = HALF_COLS * 4;
        const char* row = xi + (size_t)g0 * tg.row_bytes;
#pragma unroll 1
        for (int g = g0; g < g1; ++g, row += tg.row_bytes) {
#pragma unroll 1
            for (int part = 0; part < (HALVES ? 2 : 1); ++part) {
                // the lane number is taken afresh every time: addresses derived from it are then rebuilt with a few
                // instructions instead of living in a dozen registers across the gathers, which need them more
                int tid = (int)threadIdx.x;
                asm volatile("" : "+v"(tid));
                __syncthreads();
                if (HALVES) stage_async(row + (part ? HB : 0), lds0, part ? tg.row_bytes - HB : HB, tid, NT);
                else stage_async(row, lds0, tg.row_bytes, tid, NT);
                if (part == 0) early(g, 1);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if ((!HALVES || part == 1) && g + 1 < g1) warm_slice<NT>(row + tg.row_bytes, tg.row_bytes, per, ws.slice, dummy, tid);
                if (part == 0) late(g, 1, tid);
                body(g, part ? lds0 - (uint32_t)HB : lds0, part);
            }
        }
        return;
    }
    // one or two buffers: with two, the next tile is copied in while this one is gathered
    const bool two = tg.nbuf == 2;
    const int per = ws.per(tg.tile_rows * tg.row_bytes);
    uint32_t base = lds0, other = lds0 + (uint32_t)tg.buf_bytes;
    __syncthreads();
    if (two && g0 < g1) stage_async(xi + (size_t)g0 * tg.row_bytes, base, min(tg.tile_rows, g1 - g0) * tg.row_bytes, (int)threadIdx.x, NT);
#pragma unroll 1
    for (int t = g0; t < g1; t += tg.tile_rows) {
        int tid = (int)threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int rows = min(tg.tile_rows, g1 - t), next = t + tg.tile_rows, after = two ? next + tg.tile_rows : next;
        if (!two) {
            __syncthreads();   // the buffer is no longer read
            stage_async(xi + (size_t)t * tg.row_bytes, base, rows * tg.row_bytes, tid, NT);
        }
        early(t, rows);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this tile has landed
        __syncthreads();                                   // (two buffers: and the other one is no longer read)
        if (two && next < g1)
            stage_async(xi + (size_t)next * tg.row_bytes, other, min(tg.tile_rows, g1 - next) * tg.row_bytes, tid, NT);
        if (after < g1)
            warm_slice<NT>(xi + (size_t)after * tg.row_bytes, min(tg.tile_rows, g1 - after) * tg.row_bytes, per, ws.slice, dummy, tid);
        late(t, rows, tid);
#pragma unroll 1
        for (int r = 0; r < rows; ++r) body(t + r, base + (uint32_t)r * (uint32_t)tg.row_bytes, 0);
        if (two) { const uint32_t s = base; base = other; other = s; }
    }
}

template <typename TS, int K> struct WReg;                      // weights of one label in registers
template <int K> struct WReg<float, K> { float v[K]; };
template <int K> struct WReg<uint16_t, K> { uint32_t v[K / 2]; };

__device__ __forceinline__ uint32_t lds_base(const void* p) {
    return (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) void*)p);
}

// ------------------------------------------------------------------------------------------------ forward
// out[i][j] = sum_t W[j][t] x[i][idx[j][t]].  grid (label blocks, parts of the batch), or the other way round.
// With a loss (training): out receives the gradient of the loss by the score, and the workgroup's part of the loss goes to
// partials[block].  The scores then never go to memory: the separate pass over them took 24 us at m = 200k, b = 64 and 170 us at
// m = 500k, b = 256.  Which labels are targets comes as one bit per score; a lane reads a word for 32 instances at a time.
struct LossArgs {
    int kind;           // usl_loss_one's
    float scale;
    double* partials;
    const uint32_t* targets;   // [b / 32][m], see usl_ctx::tgt_bits
    uint32_t* nonzeros;        // LOSS = 2: usl_ctx::nz_bits
    int64_t words;             // ... of an instance
    float* clear;              // ... [m][k], which the kernels over the lists of the nonzeros add into (16-byte aligned)
};
// EVEN: blocks of tail.labels labels, not of as many as the lanes take.  (An instance of its own: with the number known only at run time the others'
// prologues came out otherwise and they were up to 4 % slower.)
// LOSS: 0 the scores, 1 either loss, 2 the squared hinge with its nonzeros marked, one bit per score, where few of them are expected: the
// pass over g that listed them took 105 us at m = 500k, b = 256, and clearing the weight gradient, which goes out here while the chip waits
// for LDS anyway, 11.  (Instances of their own: with a test at run time the step of the binary cross-entropy there took 1 % longer.)
template <int K, int LPT, int NT, typename TS, int Q, bool HALVES, int LOSS, bool EVEN, bool CACHED>
__global__ void __launch_bounds__(NT)
k_forward(const char* __restrict__ xi, const int32_t* __restrict__ idx, const TS* __restrict__ W, float* __restrict__ out,
          int64_t m, int k, int b, Geom tg, const uint8_t* __restrict__ perm, LossArgs loss, Tail tail) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const uint32_t lds0 = lds_base(lds_raw);
    const Turn turn(tg, tail);
    const int64_t j0 = (int64_t)turn.block * (EVEN ? tail.labels : NT * LPT), end = EVEN ? min(m, j0 + tail.labels) : m;
    if (LOSS)   // the first words of target bits come to the L2 while the labels' rows are brought in (1 % of the step at m = 500k, b = 256)
        touch_lines<NT>(reinterpret_cast<const char*>(loss.targets + (size_t)(turn.g0 * Q >> 5) * m + j0), 0,
                        ((int)min((int64_t)NT * LPT, end - j0) * 4 + 127) / 128, lds0 + (uint32_t)tg.dummy, (int)threadIdx.x);
    if (LOSS == 2 && turn.g0 == 0) {
        const size_t n = (size_t)min((int64_t)NT * LPT, end - j0) * k;
        float* to = loss.clear + (size_t)j0 * k;   // j0 is a multiple of 32
        const f32x4 zeros = {0.f, 0.f, 0.f, 0.f};
        for (size_t v = threadIdx.x; v < n / 4; v += NT) __builtin_nontemporal_store(zeros, reinterpret_cast<f32x4*>(to) + v);
        if (threadIdx.x < (n & 3)) to[(n & ~(size_t)3) + threadIdx.x] = 0.f;
    }
    uint32_t pk[LPT][K / 2];
    WReg<TS, K> w[LPT];
#pragma unroll
    for (int l = 0; l < LPT; ++l) {
        const int64_t row0 = j0 + (int64_t)l * NT;
        if constexpr (raw_rows<TS, K, NT>()) {
            RawRows<TS, K> raw;
            raw.load_idx(perm, idx, row0, end, k, (uint32_t)tg.zero_col);
            raw.load_w(W, row0, end, k);
            unpack_idx<K, TS>(raw, k, reinterpret_cast<uint32_t*>(lds_raw), pk[l]);
            unpack_w<K, NT>(raw, k, reinterpret_cast<uint32_t*>(lds_raw), w[l].v);
        } else {
            SlotOrder<K> so;
            so.load(perm, row0 + threadIdx.x, row0 + threadIdx.x < end);
            if (l) __syncthreads();
            fetch_idx<K>(idx, row0, end, k, (uint32_t)tg.zero_col, reinterpret_cast<uint32_t*>(lds_raw), so, pk[l]);
            fetch_w<K, NT>(W, row0, end, k, reinterpret_cast<uint32_t*>(lds_raw), so, w[l].v);
        }
    }
    const uint32_t zbyte = lds0 + HALF_COLS * 4u;
    if (HALVES) {
        __syncthreads();
        if (threadIdx.x < 4) reinterpret_cast<uint32_t*>(lds_raw)[HALF_COLS + threadIdx.x] = 0u;
    }
    const int g0 = turn.g0, g1 = turn.g1;
    const int nlab = (int)min((int64_t)NT * LPT, end - j0);
    const int wave0 = EVEN ? __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~63) : 0;   // a wavefront without labels gathers nothing
    // Q <= 2: the scores of a group are written while the next group is gathered, before the last label's gathers (a store
    // right before the next copy would make that copy's wait include it; four stores in a row would hold the wavefront
    // at the memory pipeline).  Q = 4 has no registers left for that, and a quarter of the waits.  All labels' losses
    // in one place, and the gathers before everything else (setprio): 805 us at m = 500k, d = 32k, k = 32, b = 256, where
    // a label's loss in front of its own gathers took 866, and 852 with the priority.
    constexpr bool DELAY = Q <= 2;
    float prev[DELAY ? LPT : 1][Q] = {};
    double lost = 0.0;
    // Bit i % 32 of marks[l]: the label is a target of instance i.  Good for 32 instances, before `until`; loaded
    // with the tile that leaves them and waited for together with that tile: a load still under way when the losses are
    // added up would be waited for there, with the stores and the warm-up loads behind it (50 of 825 us at m = 500k, b = 256).
    uint32_t marks[LPT];
    int until = -1;
    auto load_targets = [&](int first, int last) {   // for the instances first .. last, at most 32 of them
        if (!LOSS || last < until) return;
        until = first + 32;
        uint32_t behind[LPT];
#pragma unroll
        for (int l = 0; l < LPT; ++l) {
            int jl = (int)threadIdx.x + l * NT;
            asm volatile("" : "+v"(jl));
            const uint32_t* p = loss.targets + (size_t)(first >> 5) * m + j0;
            marks[l] = jl < nlab ? p[(uint32_t)jl] : 0u;
            behind[l] = jl < nlab && (first & 31) != 0 && (first | 31) + 1 < b ? p[m + jl] : 0u;
        }
        const uint32_t later = (1u << (first & 31)) - 1u;   // the bits of the second word
#pragma unroll
        for (int l = 0; l < LPT; ++l) {
            marks[l] = (behind[l] & later) | (marks[l] & ~later);
            asm volatile("" : "+v"(marks[l]));
        }
    };
    // Scores leave past the caches: as ordinary stores they push rows of x out of the L2 (forward of m = 600k, d = 20k, k = 32, b = 128: 331
    // and 320 us; m = 500k, d = 32k, b = 256: 761 and 751).  But two wavefronts share a line where a row of scores does not begin with
    // one, and past the caches its halves reach the memory one by one: labels of few slots, whose stores weigh as much as their
    // gathers, wait for that (m = 173 019, d = 64, k = 4, b = 438: 124 and, through the caches, 74; k = 12 133 and 89; m = 400 003, d = 300, k = 16,
    // b = 100 76 and 62), and lose 4 to 8 % through the caches where it does (m = 1M, d = 2000, k = 8, b = 32: 39.0 and 40.6).  A test at run time
    // cost both (80 and 40.5 us).  So labels of up to 16 slots go through the caches, of 24 where scores_through_caches says so.  Not where the loss
    // is part of it: there is more between the stores (steps at these sizes 2 to 4 % slower through the caches).
    constexpr bool past = LOSS || !CACHED;
    // Addresses of the scores: a base in scalar registers and a lane's 32-bit offset or, where scores leave alone and a read brings 4 bytes, one address a
    // lane (16 to 48 slots; of bfloat16 32 and 48): the compiler's registers and spills come out otherwise.  Forward with the base and with one address a
    // lane, us: m = 500k, d = 32k, k = 32, b = 256 756.3 and 749.8; m = 210 007, d = 40k, b = 60, k = 32 114.9 and 111.1, k = 16 78.7 and 77.0, k = 48 183.4 and 182.1;
    // m = 500k, d = 36k, k = 32, b = 100, bfloat16 206.0 and 201.9.  The others, the same way round: m = 400k, d = 18k, k = 16, b = 48 82.4 and 89.1; d = 6k, k = 32, bfloat16
    // 77.1 and 81.0; two halves of rows, m = 250k, d = 65 536, k = 48, b = 64 337 and 346; the step with the loss inside at m = 500k, d = 32k, b = 256 1950.5 and 1955.4.
    constexpr bool LANE_ADDRESSES = LOSS == 0 && !HALVES && Q * sizeof(TS) == 4 && K >= (sizeof(TS) == 4 ? 16 : 32) && K < 64;
    auto put = [&](int g, int l, const float (&z)[Q]) {
        int jl = (int)threadIdx.x + l * NT;   // rebuilt here: kept, every label's offset would be a register across the gathers
        asm volatile("" : "+v"(jl));
        if (jl < nlab) {
            float sum = 0.f, logs = 0.f;
            // Targets are few: a wavefront without one among these scores takes the short form of the loss (a step at m = 670k, d = 16k, b = 32:
            // 584 us with the general form for all, 571 with both).  A kernel of its own for the targets, which took their scores once more, cost
            // 8 us a step at m = 31k, d = 1k, b = 128 and at m = 200k, d = 8k, b = 64, 13 at m = 500k, b = 256.
            const uint32_t hits = LOSS ? __builtin_amdgcn_ubfe(marks[l], (uint32_t)(g * Q) & 31u, (uint32_t)Q) : 0u;
            auto finish = [&](auto any_target) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (g * Q + q < b) {
                        float o = z[q];
                        if (LOSS) {
                            const usl_loss_parts r = usl_loss_in_parts(LOSS == 2 ? 1 : loss.kind, o, any_target.value && (hits >> q & 1u) ? 1.f : 0.f, loss.scale);
                            o = r.g;
                            sum += r.lin;
                            logs += r.log2;
                        }
                        float* row = out + ((size_t)(g * Q + q) * m + j0);
                        float* to = LANE_ADDRESSES ? row + (uint32_t)jl : reinterpret_cast<float*>(reinterpret_cast<char*>(row) + (uint32_t)jl * 4u);
                        if constexpr (past) __builtin_nontemporal_store(o, to); else *to = o;
                        if constexpr (LOSS == 2) {   // lane 0's word and, where the wavefront has more than 32 labels, lane 1's
                            const uint64_t set = __ballot(o != 0.f);
                            const int first = __builtin_amdgcn_readfirstlane(jl), lane = jl & 63;   // (blocks of labels begin at a multiple of 32)
                            uint32_t* words = loss.nonzeros + ((int64_t)(g * Q + q) * loss.words + ((j0 + first) >> 5));
                            if (lane < 2 && first + lane * 32 < nlab) words[lane] = lane ? (uint32_t)(set >> 32) : (uint32_t)set;
                        }
                    }
            };
            if (LOSS == 2 || (LOSS && __builtin_expect(__any(hits != 0u), 0))) finish(std::true_type());
            else finish(std::false_type());
            lost += (double)fmaf(logs, 0.6931471805599453f, sum);
        }
    };
    walk<NT, (Q > 1), HALVES>(xi, lds0, tg, WarmShare(turn.warm_at, turn.warm_share), g0, g1,
        [&](int g, uint32_t base, int part) {
            float before[DELAY ? LPT : 1][Q];
#pragma unroll
            for (int l = 0; l < (DELAY ? LPT : 0); ++l) {
#pragma unroll
                for (int q = 0; q < Q; ++q) before[l][q] = prev[l][q];
            }
#pragma unroll
            for (int l = 0; l < LPT; ++l) {
                if (DELAY && l == LPT - 1 && part == 0 && g > g0) {
#pragma unroll
                    for (int l2 = 0; l2 < LPT; ++l2) put(g - 1, l2, before[DELAY ? l2 : 0]);
                }
                float acc[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) acc[q] = HALVES && part ? prev[DELAY ? l : 0][q] : 0.f;   // the first half's sums
                keep_packed(pk[l]);
                __builtin_amdgcn_s_setprio(1);
                if (!EVEN || wave0 + l * NT < nlab) label_dot<K, Q, HALVES>(pk[l], w[l].v, base, zbyte, acc);
                __builtin_amdgcn_s_setprio(0);
                // finish the sums here; left alone the compiler sinks the multiply-adds into the guarded store
                // and keeps every gathered value alive until then
#pragma unroll
                for (int q = 0; q < Q; ++q) asm volatile("" : "+v"(acc[q]));
                if (DELAY) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) prev[DELAY ? l : 0][q] = acc[q];
                } else {
                    put(g, l, acc);
                }
            }
        },
        [&](int, int, int) {},
        [&](int t, int rows) {   // (the groups that are put while this tile is gathered)
            const int first = (DELAY && t > g0 ? t - 1 : t) * Q;
            load_targets(first, first + rows * Q - 1);
        });
    if (DELAY && g1 > g0) {
        load_targets((g1 - 1) * Q, g1 * Q - 1);
#pragma unroll
        for (int l = 0; l < LPT; ++l) put(g1 - 1, l, prev[DELAY ? l : 0]);
    }
    if (LOSS) {   // the workgroup's share, added up in a fixed order
        for (int o = 32; o > 0; o >>= 1) lost += __shfl_down(lost, o);
        double* red = reinterpret_cast<double*>(lds_raw);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lost;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int q = 0; q < NT / 64; ++q) t += red[q];
            loss.partials[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
        }
    }
}

// ------------------------------------------------------------------------------------------------ weight gradient
// grad_W[j][t] = sum_i g[i][j] x[i][idx[j][t]].  With the batch split every part of it leaves a partial
// gradient (part_stride elements apart) that a later kernel adds up in a fixed order.  A label whose gradients of a
// group are zero in all 64 lanes skips its gathers (Algorithm 3 skips zero entries).
template <int K, int LPT, int NT, typename TS, int Q, bool HALVES, bool EVEN>
__global__ void __launch_bounds__(NT)
k_backward_weight(const float* __restrict__ g, const char* __restrict__ xi, const int32_t* __restrict__ idx, float* __restrict__ grad_W,
                  int64_t m, int k, int b, Geom tg, const uint8_t* __restrict__ perm, size_t part_stride, const uint32_t* __restrict__ gate, int labels) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    if (gate && *gate == 0) return;   // the gradient is almost all zeros: the kernels over its nonzeros do the work
    const uint32_t lds0 = lds_base(lds_raw);
    const uint32_t part = tg.parts_first ? blockIdx.x : blockIdx.y;
    const int64_t j0 = (int64_t)(tg.parts_first ? blockIdx.y : blockIdx.x) * (EVEN ? labels : NT * LPT), end = EVEN ? min(m, j0 + labels) : m;
    uint32_t pk[LPT][K / 2];
    float acc[LPT][K];
#pragma unroll
    for (int l = 0; l < LPT; ++l) {
        const int64_t row0 = j0 + (int64_t)l * NT;
        if constexpr (raw_rows<float, K, NT>()) {
            RawRows<TS, K> raw;
            raw.load_idx(perm, idx, row0, end, k, (uint32_t)tg.zero_col);
            unpack_idx<K, TS>(raw, k, reinterpret_cast<uint32_t*>(lds_raw), pk[l]);
        } else {
            SlotOrder<K> so;
            so.load(perm, row0 + threadIdx.x, row0 + threadIdx.x < end);
            fetch_idx<K>(idx, row0, end, k, (uint32_t)tg.zero_col, reinterpret_cast<uint32_t*>(lds_raw), so, pk[l]);
        }
#pragma unroll
        for (int t = 0; t < K; ++t) acc[l][t] = 0.f;
    }
    const uint32_t zbyte = lds0 + HALF_COLS * 4u;
    if (HALVES) {
        __syncthreads();
        if (threadIdx.x < 4) reinterpret_cast<uint32_t*>(lds_raw)[HALF_COLS + threadIdx.x] = 0u;
    }
    const int g0 = (int)part * tg.groups_per_block, g1 = min(tg.groups, g0 + tg.groups_per_block);
    const int nlab = (int)min((int64_t)NT * LPT, end - j0);
    // The gradients of the next group come from HBM and are requested one group ahead, right after this group's row
    // copy: before it, the copy's wait would wait for them too.  (Q = 4 on wide blocks has no registers for that: their
    // lines are brought to the L2 one group ahead instead and read behind the copy.)
    constexpr bool AHEAD = LPT * Q <= 4;
    float gnext[AHEAD ? LPT : 1][Q], gv[LPT][Q];
    auto load_g = [&](int grp, int l, float (&v)[Q]) {
        int jl = (int)threadIdx.x + l * NT;
        asm volatile("" : "+v"(jl));
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = jl < nlab && grp < g1 && grp * Q + q < b ? (g + ((size_t)(grp * Q + q) * m + j0))[(uint32_t)jl] : 0.f;
    };
    if (AHEAD) {
#pragma unroll
        for (int l = 0; l < LPT; ++l) load_g(g0, l, gnext[AHEAD ? l : 0]);
    }
    walk<NT, (Q > 1), HALVES>(xi, lds0, tg, WarmShare(tg), g0, g1,
        [&](int grp, uint32_t base, int part) {
            if (part == 0) {
                if (AHEAD) {
#pragma unroll
                    for (int l = 0; l < LPT; ++l) {
#pragma unroll
                        for (int q = 0; q < Q; ++q) gv[l][q] = gnext[AHEAD ? l : 0][q];
                        load_g(grp + 1, l, gnext[AHEAD ? l : 0]);
                    }
                } else {
#pragma unroll
                    for (int l = 0; l < LPT; ++l) load_g(grp, l, gv[l]);
                }
            }
#pragma unroll
            for (int l = 0; l < LPT; ++l) {
                bool any = false;
#pragma unroll
                for (int q = 0; q < Q; ++q) any = any || gv[l][q] != 0.f;
                if (!__any(any)) continue;
                keep_packed(pk[l]);
                label_outer<K, TS, Q, HALVES>(pk[l], gv[l], base, zbyte, acc[l]);
            }
        },
        [&](int t, int rows, int tid) {
            if (!AHEAD) {   // one load per 128-byte line of the next tile's gradients
                for (int q = 0; q < Q * rows; ++q) {
                    const int64_t i = (int64_t)(t + rows) * Q + q;
                    if (i < b && i < (int64_t)g1 * Q)
                        touch_lines<NT>(reinterpret_cast<const char*>(g + i * m + j0), 0, nlab * 4 / 128, lds0 + (uint32_t)tg.dummy, tid);
                }
            }
        },
        [](int, int) {});
#pragma unroll
    for (int l = 0; l < LPT; ++l) {
        const int64_t row0 = j0 + (int64_t)l * NT;
        SlotOrder<K> so;
        so.load(perm, row0 + threadIdx.x, row0 + threadIdx.x < end);
        store_rows<K, NT>(acc[l], grad_W + (size_t)part * part_stride, row0, end, k, reinterpret_cast<uint32_t*>(lds_raw), so);
    }
}

}  // namespace usl_products
