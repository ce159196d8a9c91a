// Input gradient (Algorithm 2) in its feature-stationary LDS form: the mirror image of the forward kernel.
//
//   grad_x[i][c] = sum over connections (j,t) with idx[j][t]==c of W[j][t] * g[i][j]
//
// A workgroup owns a window of wl labels and a block of NF features.  Every lane keeps the list of one pair of
// features -- (label-in-window, 16 bit) and weight of every connection that leads from the window into the feature
// -- in registers for the workgroup's whole life, walks the batch staging g[i][window] (wl floats) through LDS with
// LDS-DMA, and gathers: the same ds_read_b32 stream as the forward kernel, reading g row-major (no transposed copy
// of the gradient, no zero flags).  The sums of a window go to partial[window][i][c]; a second kernel adds the
// windows up.
//
// Lists of one (window, feature) have Poisson-distributed lengths (mean wl*k/d, at most 32: the windows are sized
// for that), registers are allocated for a fixed number of slots.  Per (window, feature block) the features are
// therefore ranked by list length and paired longest with shortest: lane l holds list A = rank l from slot 0 upwards
// and list B = rank NF-1-l from slot KTOT-1 downwards; a wavefront (64 neighbouring ranks: nearly equal lengths)
// visits slots [0, acap) for its A lists and [KTOT-bcap, KTOT) for its B lists, acap + bcap <= KTOT chosen per
// wavefront so that as little as possible is left over.  Entries that do not fit (a few dozen per workgroup for
// uniform connectivity: the very longest lists; anything for a caller's skewed idx) go to an overflow list of the
// workgroup, kept list by list: its first 1024 entries sit in LDS with their weights and the list's own lane adds
// them after its registers; what is beyond that is added with LDS atomics from memory: slow, rare, and what keeps
// the form valid for any connectivity.  Within a lane's allowance the entries are put in a bank-aware order
// (k_lf_schedule), the empty places of shorter lists included.
//
// Registers: 34 for the packed labels and 68 for the weights of the 68 slots leave 26 of a lane's 128 (1024 lanes
// per compute unit) for everything else; the gathers are therefore written out in assembly, four in flight.
#include <stdlib.h>

#include <type_traits>

#include "usl_internal.h"

#include "k_lists_cut.h"
#include "k_sums.h"
#include "k_matching.h"

using namespace usl_lists;

namespace {

constexpr int KT_BWI = 68;     // list slots per lane, shared by its two lists (with the rest of the kernel: the 128 registers a lane has)
constexpr int KT_BOTH = 36, KT_BOTH4 = 32;    // ... in the kernel that also keeps a weight-gradient sum per slot (windows of half the length)
constexpr uint32_t PAD_SLOT = 0xFFFFFFFFu;
// LDS of the gather kernel: the row slice, NF floats through which the sums are un-permuted, NT words (the features of
// every lane), NT entries of 8 bytes (the nearest part of the overflow list), 2 * NT words (each lane's share of it) and
// 32 words of zeros, one per bank: what the empty places of a list read (weight 0 times a real gradient would turn an
// infinity in g into NaNs in features that have nothing to do with it).  ZERO_LABEL + b is the "label" whose address is
// zero word b; it fits the 16 bits of a packed label.
constexpr size_t LDS_BYTES = (size_t)32768 * 4 + (size_t)2048 * 4 + (size_t)1024 * 4 + (size_t)1024 * 8 + (size_t)1024 * 8 + 128;
constexpr uint32_t ZERO_LABEL = (uint32_t)((LDS_BYTES - 128) / 4);
static_assert(ZERO_LABEL % 32 == 0 && ZERO_LABEL + 31 < 65536 && LDS_BYTES <= 160 * 1024, "zero words: bank b, 16-bit label, inside LDS");
// LDS of the kernel for both backward products.  It stages the slices of Q instances interleaved: label l's Q values are the
// 4 Q bytes at 4 Q l (one ds_read_b64 or ds_read_b128 brings them), behind them 32 units of zeros (zero_label is their
// "label": a window has at most that many labels).  Then Q * NF floats for the sums of the instances, for Q = 4 the
// activations of the block's features where there is room for them (OWN; else they lie in the place of the sums until those are
// ready), NT words (features; with OWN another NT: their places among the activations), NEAR2 overflow entries of 8 bytes, NT
// words (each lane's share of them), NEAR2 floats (their weight-gradient sums), and a word for what an empty place of a list
// brings or leaves.
constexpr int NEAR2 = 510;   // even, and counted in pairs by 8 bits
template <int Q, bool OWN> struct BothLayout {
    static constexpr uint32_t zero_label = Q == 2 ? BOTH2_LABELS : OWN ? BOTH4_OWN_LABELS : BOTH4_LABELS;
    static constexpr uint32_t row_bytes = (zero_label + 32) * 4 * Q, x_bytes = OWN ? 4 * 2048 * 4 : 0, feat_words = OWN ? 2048 : 1024;
};
template <int Q, bool OWN> constexpr size_t both_lds_bytes() {
    typedef BothLayout<Q, OWN> L;
    return (size_t)L::row_bytes + (size_t)Q * 2048 * 4 + L::x_bytes + (size_t)L::feat_words * 4 + (size_t)NEAR2 * 8 + (size_t)1024 * 4 + (size_t)NEAR2 * 4 + 16;
}
// places that LDS holds at a time below the sums of the overflow entries; a workgroup with no more has 16-bit places
template <int Q, bool OWN> constexpr uint32_t both_places() { return (uint32_t)((both_lds_bytes<Q, OWN>() - 16 - (size_t)NEAR2 * 4) / 4); }
template <int Q, bool OWN> constexpr uint32_t no_place() { return (uint32_t)((both_lds_bytes<Q, OWN>() - 16) / 4); }
template <int Q, bool OWN> constexpr bool both_layout_ok() {
    return both_places<Q, OWN>() >= (Q == 4 ? KT_BOTH4 : KT_BOTH) * NT          // a lane's slots have places of their own
           && both_lds_bytes<Q, OWN>() >= (both_places<Q, OWN>() + 63) * 4 && no_place<Q, OWN>() < 65535   // 16 bits, and one value for no place
           && BothLayout<Q, OWN>::zero_label % 32 == 0                          // zero units on the banks of their number
           && both_lds_bytes<Q, OWN>() <= 160 * 1024;
}
static_assert(both_layout_ok<2, false>() && both_layout_ok<4, true>() && both_layout_ok<4, false>(), "LDS of k_both_lds");
// The labels (and, in the kernel for both products, the places) of a lane's slots lie in 16-bit halves of words, four words to a
// 16-byte piece, a piece of all lanes behind the other: what bounds bringing them in is the number of loads.  Index in 16-bit units of slot t of lane l.
template <int KT> constexpr int pieces_of() { return (KT / 2 + 3) / 4; }
template <int KT> __device__ __forceinline__ size_t half_at(size_t wg, int t, int l) { return ((wg * pieces_of<KT>() + t / 8) * NT + l) * 8 + t % 8; }
// all of a lane's words
template <int KT>
__device__ __forceinline__ void load_words(const void* base, uint32_t lane, uint32_t (&w)[KT / 2]) {
#pragma unroll
    for (int q = 0; q < pieces_of<KT>(); ++q) {
        const uint4 v = (reinterpret_cast<const uint4*>(base) + (size_t)q * NT)[lane];
        w[4 * q] = v.x;
        if (4 * q + 1 < KT / 2) w[4 * q + 1 < KT / 2 ? 4 * q + 1 : 0] = v.y;
        if (4 * q + 2 < KT / 2) w[4 * q + 2 < KT / 2 ? 4 * q + 2 : 0] = v.z;
        if (4 * q + 3 < KT / 2) w[4 * q + 3 < KT / 2 ? 4 * q + 3 : 0] = v.w;
    }
}
// Where label l of a window of wl lies in the rows of k_both_lds, in units of Q values.  A lane brings four neighbouring labels
// of every instance: four writes of 16 bytes with four instances, and with the labels in order a wavefront's would be 64
// bytes apart, four to a bank.  So each of the four goes into a quarter of the row of its own, next to those of the other
// lanes; the lists hold these numbers instead of the labels', which costs nothing.  (Two instances, two writes 32 bytes apart:
// in order; by halves it measured the same.)
template <int Q> __host__ __device__ __forceinline__ uint32_t unit_of_label(uint32_t l, uint32_t wl) {
    return Q == 4 ? (l & 3u) * (wl / 4u) + (l >> 2) : l;
}
template <int KT> struct ListLayout;   // what depends on which kernel the lists are for
template <> struct ListLayout<68> { static constexpr uint32_t near = 1024; };
template <> struct ListLayout<36> { static constexpr uint32_t near = NEAR2; };
template <> struct ListLayout<32> { static constexpr uint32_t near = NEAR2; };
// label of flat slot e within its window (w0: the window's first label), as the lists hold it.  inv_k: inverse_of(k)
__device__ __forceinline__ uint32_t inverse_of(int k) { return k > 1 ? (uint32_t)(0x100000000ull / (uint32_t)k) : 0xFFFFFFFFu; }
template <int KTOT>
__device__ __forceinline__ uint32_t label_of_slot(uint32_t e, int k, uint32_t inv_k, uint32_t w0, const Cut& cut) {
    uint32_t q = __umulhi(e, inv_k);   // e / k, at most one too low
    if (e - q * (uint32_t)k >= (uint32_t)k) ++q;
    q -= w0;
    return KTOT == KT_BOTH4 ? unit_of_label<4>(q, (uint32_t)cut.wl) : q;
}
// Sum of v over the lanes up to this one; *total = over all.  sh: NT / 64 words that no other use of them is still reading.
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o);
        if ((int)(threadIdx.x & 63) >= o) v += t;
    }
    if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t below = 0, all = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
        const uint32_t t = sh[q];
        below += q < (int)(threadIdx.x >> 6) ? t : 0u;
        all += t;
    }
    *total = all;
    return below + v;
}

// The connections of a workgroup of the gather kernel, by place (k_lf_seg_place): their flat slots and features.  Where a
// window has one block of features only, the places are the flat slots, and idx has the features.
constexpr size_t LF_STAGED = 36864 + 512;
struct LfPlaces {
    const int32_t* idx;
    const uint32_t* slot_at;   // [m*k] by place
    const uint16_t* feat_at;   // [m*k] by place: feature within the block
    uint32_t* pos;             // one block only: place of every flat slot, written here (or NULL)
    uint32_t small_wg;         // workgroups with no more connections have entries of label and place in one word (0: none)
    int staged;                // entries that LDS holds
};
// One workgroup per (window, feature block): counts the connections of the block's NF features, ranks these by list length, pairs
// them, fixes the slot ranges of every wavefront, counts what will not fit, and groups the connections by feature:
// ent[ent_base[wg] + where[w][c] + p] = the p-th connection from window w into feature c (p by a cursor: the order inside a list
// is not fixed): its flat slot j*k+t, or, for the kernel of both products unless the connectivity is skewed, its label within
// the window and its place, 16 bits each.  The groups are put together in LDS and leave it in whole lines (beyond what LDS holds
// each entry goes where it belongs by itself).
// Reading every connection once from its place, a workgroup counts and groups without a global atomic; with shares of a window's
// slots that counted all features and reserved their places in every list by atomics, counting, ranking and grouping took
// 414 us at m = 500k, d = 32k, k = 32, with the places 462, now 189.
//   count[w][c]       = length of a list
//   feat[wg][z][lane] = feature (within the block) whose list lane holds in zone z
//   caps[wg][wave]    = acap | bcap << 8
//   where[w][c]       = where the list of feature c starts among the workgroup's entries
//   ov_off[w][c]      = where what does not fit of that list starts in the workgroup's overflow list
//   n_ov[wg]          = entries beyond the allowances
//   ovr[wg][z][lane]  = start | n << 16: the part of that list's overflow among the first NT (NEAR2) entries (those the
//                       gather kernel keeps in LDS and the list's own lane adds up)
template <int KTOT>
__global__ void __launch_bounds__(NT)
k_lf_plan(LfPlaces in, int64_t m, int k, int d, Cut cut, uint32_t* __restrict__ ent_base, uint32_t* __restrict__ count,
          uint32_t* __restrict__ where, uint32_t* __restrict__ ov_off, uint16_t* __restrict__ feat, uint32_t* __restrict__ caps,
          uint32_t* __restrict__ n_ov, uint32_t* __restrict__ ovr, uint32_t* __restrict__ ent) {
    extern __shared__ uint32_t staged[];
    __shared__ uint32_t start[256];
    __shared__ uint32_t cur[NF];            // lengths of the lists, then where their next entries go
    __shared__ uint32_t sh[2][NT / 64];
    __shared__ uint16_t len_of[2][NT];
    __shared__ uint32_t cap_of[NT / 64];
    const int nfb = cut.nfb, fpb = cut.fpb, vd = cut.vd;
    const int wg = blockIdx.x, w = wg / nfb, fb = wg % nfb;
    const uint32_t w0 = (uint32_t)((size_t)w * cut.wl * k);
    if (nfb == 1 && threadIdx.x == 0) {   // (the launch order makes it known to the kernels that follow)
        ent_base[wg] = w0;
        if (wg == cut.nwin - 1) ent_base[wg + 1] = (uint32_t)(m * k);
    }
    const uint32_t e0 = nfb == 1 ? w0 : ent_base[wg];
    const uint32_t n_ent = nfb == 1 ? (uint32_t)(min((int64_t)(w + 1) * cut.wl, m) * k) - w0 : ent_base[wg + 1] - e0;
    // use(place, feature within the block) for the workgroup's connections, eight of a lane's loads in flight together
    auto connections = [&](auto use) {
        for (uint32_t p = threadIdx.x; p < n_ent; p += 8 * NT) {
            uint32_t f[8];
            if (nfb == 1) {
#pragma unroll
                for (int u = 0; u < 8; ++u) f[u] = (uint32_t)in.idx[e0 + min(p + u * NT, n_ent - 1)];
                if (cut.S > 1) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) f[u] = f[u] < (uint32_t)d ? cut.vfeat(f[u], (p + u * NT) / (uint32_t)k, d) : (uint32_t)NF;
                }
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) f[u] = in.feat_at[e0 + min(p + u * NT, n_ent - 1)];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p + u * NT >= n_ent) f[u] = NF;   // none
            use(p, f);
        }
    };
    const int nf = min(fpb, vd - fb * fpb);   // features of the block that exist; the others have empty lists
    if (threadIdx.x < 256) start[threadIdx.x] = 0;
    cur[threadIdx.x] = cur[threadIdx.x + NT] = 0;
    __syncthreads();
    connections([&](uint32_t, const uint32_t (&f)[8]) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (f[u] < (uint32_t)nf) atomicAdd(&cur[f[u]], 1u);
    });
    __syncthreads();
    const size_t bin = (size_t)w * vd + (size_t)fb * fpb + threadIdx.x;
    uint32_t n[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        n[q] = cur[threadIdx.x + q * NT];
        if ((int)threadIdx.x + q * NT < nf) count[bin + q * NT] = n[q];
        atomicAdd(&start[min(n[q], 255u)], 1u);
    }
    __syncthreads();
    {   // ranks of the buckets, longest lists first: how many lists the buckets above hold, four buckets a lane
        // (one lane going through all of them took 9 of this kernel's 16 us on a small layer)
        uint32_t mine[4], above = 0;
        if (threadIdx.x < 64) {
            uint32_t sum = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) sum += mine[u] = start[255 - 4 * threadIdx.x - u];
            above = sum;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(above, o);
                if ((int)threadIdx.x >= o) above += t;
            }
            above -= sum;
#pragma unroll
            for (int u = 0; u < 4; ++u) { start[255 - 4 * threadIdx.x - u] = above; above += mine[u]; }
        }
    }
    __syncthreads();
    uint32_t lane_of[2], zone_of[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t r = atomicAdd(&start[min(n[q], 255u)], 1u);   // rank (order among equal lengths is arbitrary)
        zone_of[q] = r < (uint32_t)NT ? 0u : 1u;
        lane_of[q] = r < (uint32_t)NT ? r : (uint32_t)(NF - 1) - r;
        len_of[zone_of[q]][lane_of[q]] = (uint16_t)min(n[q], 65535u);
        feat[((size_t)wg * 2 + zone_of[q]) * NT + lane_of[q]] = (uint16_t)(threadIdx.x + q * NT);
    }
    __syncthreads();
    {   // the wavefront's two slot allowances (multiples of 4, KTOT together): those that leave the least outside
        // the registers, counting the longest leftover of a single lane (its lane walks that alone) 16-fold
        const uint32_t la = len_of[0][threadIdx.x], lb = len_of[1][threadIdx.x];
        uint32_t best = 0xFFFFFFFFu;
        for (uint32_t ca = 0; ca <= (uint32_t)KTOT; ca += 4) {
            const uint32_t cb = (uint32_t)KTOT - ca;
            uint32_t tot = (la > ca ? la - ca : 0u) + (lb > cb ? lb - cb : 0u);
            uint32_t mx = max(la > ca ? la - ca : 0u, lb > cb ? lb - cb : 0u);
            for (int o = 32; o > 0; o >>= 1) {
                tot += __shfl_xor(tot, o);
                mx = max(mx, (uint32_t)__shfl_xor(mx, o));
            }
            const uint32_t cost = min(tot + 16u * mx, 0xFFFFFFu);
            best = min(best, cost << 8 | ca);
        }
        // no more than the longest list needs (slots a wavefront visits are time)
        uint32_t amax = la, bmax = lb;
        for (int o = 32; o > 0; o >>= 1) {
            amax = max(amax, (uint32_t)__shfl_xor(amax, o));
            bmax = max(bmax, (uint32_t)__shfl_xor(bmax, o));
        }
        const uint32_t acap = min(best & 0xFFu, (amax + 3u) & ~3u);
        const uint32_t bcap = min((uint32_t)KTOT - (best & 0xFFu), (bmax + 3u) & ~3u);
        if ((threadIdx.x & 63) == 0) {
            cap_of[threadIdx.x >> 6] = acap | (bcap << 8);
            caps[(size_t)wg * (NT / 64) + (threadIdx.x >> 6)] = acap | (bcap << 8);
        }
    }
    __syncthreads();
    uint32_t ov[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t cw = cap_of[lane_of[q] >> 6];
        const uint32_t cap = zone_of[q] == 0 ? (cw & 0xFFu) : (cw >> 8);
        ov[q] = n[q] > cap ? n[q] - cap : 0u;
        ov[q] = (ov[q] + 1u) & ~1u;   // an even number of places: the list's lane walks them two at a time
    }
    {
        uint32_t all, at = block_inclusive_scan(n[0] + n[1], sh[0], &all) - n[0] - n[1];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if ((int)threadIdx.x + q * NT < nf) where[bin + q * NT] = at;
            cur[threadIdx.x + q * NT] = at;   // (read as a length by this lane alone)
            at += n[q];
        }
    }
    {
        uint32_t all, at = block_inclusive_scan(ov[0] + ov[1], sh[1], &all) - ov[0] - ov[1];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if ((int)threadIdx.x + q * NT < nf) ov_off[bin + q * NT] = at;
            const uint32_t first = min(at, ListLayout<KTOT>::near);
            ovr[((size_t)wg * 2 + zone_of[q]) * NT + lane_of[q]] = first | (min(ov[q], ListLayout<KTOT>::near - first) << 16);
            at += ov[q];
        }
        if (threadIdx.x == 0) n_ov[wg] = all;
    }
    // (the second scan's barrier stands between the cursors and their use)
    const bool small = n_ent <= in.small_wg, stage = n_ent <= (uint32_t)in.staged;
    const uint32_t inv_k = inverse_of(k), first_label = (uint32_t)w * (uint32_t)cut.wl;
    uint32_t* to = stage ? staged : ent + e0;
    connections([&](uint32_t p, const uint32_t (&f)[8]) {
        uint32_t e[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t place = min(p + u * NT, n_ent - 1);
            e[u] = nfb == 1 ? e0 + place : in.slot_at[e0 + place];
            if (nfb == 1 && in.pos) in.pos[e[u]] = e[u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (f[u] < (uint32_t)nf)
                to[atomicAdd(&cur[f[u]], 1u)] = small ? label_of_slot<KTOT>(e[u], k, inv_k, first_label, cut) | (p + u * NT) << 16 : e[u];
    });
    if (!stage) return;
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < n_ent; q += NT) ent[e0 + q] = staged[q];
}

// base[wg] = sum of count over the workgroups before wg, base[nwg] = all of them.  Block 1, if there is one, records the
// fingerprint of idx.
__global__ void __launch_bounds__(1024)
k_lf_scan(const uint32_t* __restrict__ count, uint32_t* __restrict__ base, int nwg, const uint32_t* __restrict__ idx, size_t n_words,
          uint64_t* __restrict__ print, int which) {
    __shared__ uint32_t part[1024];
    if (blockIdx.x == 1) {
        usl_idx_fingerprint_block(idx, n_words, print, which, 1);
        return;
    }
    const int per = (nwg + 1023) / 1024;
    const int a = min(nwg, (int)threadIdx.x * per), e = min(nwg, a + per);
    uint32_t s = 0;
    for (int q = a; q < e; ++q) s += count[q];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const uint32_t t = threadIdx.x >= (unsigned)o ? part[threadIdx.x - o] : 0u;
        __syncthreads();
        part[threadIdx.x] += t;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - s;
    for (int q = a; q < e; ++q) { base[q] = run; run += count[q]; }
    if (threadIdx.x == 1023) base[nwg] = part[1023];
}

struct OvEntry { uint16_t feature; uint16_t label; uint32_t slot; };
// The place of every connection, out of m * k: those of a (window, feature block) workgroup together (from ent_base[wg], as in
// ent), and within it in the order of their flat slots, up to the order inside a run of SEG slots.  k_lf_plan goes through a
// workgroup's connections by place, and the kernel for both products leaves the weight gradients there (pos[flat slot]): the
// Adam kernel, which goes through the slots in order, then reads 16 or so neighbouring places from each of the window's nfb
// workgroups per wavefront -- whole lines; in the order of the lists it would fetch a line per value.
// slot_at[place] is the way back: the kernel reads the weights in the order of the places, for the same reason.
// Three kernels (and the sums of the workgroups in between): the counts of every run per feature block, their running sums, the
// places.  Where a window has one block only, the places are the flat slots themselves, and none of this is needed.
constexpr int SEG = 256;   // slots of a run: one wavefront, four per lane
struct LfRun {
    int w, seg;
    bool on;
    size_t e;       // the lane's first slot
    int n;          // how many it has, up to four
    uint32_t col[4], block[4];   // feature, block of features (nfb: a feature that the layer does not have)
    // An XCD (blockIdx.x % 8) takes an eighth of the runs in order: neighbours write into the same lines, through one L2.
    __device__ __forceinline__ LfRun(const int32_t* __restrict__ idx, int64_t m, int k, const Cut& cut, int nseg, int64_t total) {
        typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
        const int64_t gs = ((int64_t)(blockIdx.x & 7) * (gridDim.x / 8) + (blockIdx.x >> 3)) * 4 + (threadIdx.x >> 6);
        on = gs < total;
        w = seg = n = 0;
        e = 0;
        if (!on) return;
        w = (int)(gs / nseg);
        seg = (int)(gs % nseg);
        const size_t w0 = (size_t)w * cut.wl * k, w1 = (size_t)min((int64_t)(w + 1) * cut.wl, m) * k;
        const size_t s0 = min(w0 + (size_t)seg * SEG, w1), s1 = min(s0 + SEG, w1);
        e = s0 + (threadIdx.x & 63) * 4;
        n = e < s1 ? (int)min(s1 - e, (size_t)4) : 0;
        if (n == 4) {
            const i32x4_any v = *reinterpret_cast<const i32x4_any*>(idx + e);
#pragma unroll
            for (int u = 0; u < 4; ++u) col[u] = (uint32_t)v[u];
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) col[u] = u < n ? (uint32_t)idx[e + u] : 0u;
        }
        const uint32_t inv = inverse_of(cut.fpb);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            block[u] = __umulhi(col[u], inv);   // at most one too low
            if (col[u] - block[u] * (uint32_t)cut.fpb >= (uint32_t)cut.fpb) ++block[u];
            block[u] = min(block[u], (uint32_t)cut.nfb);
        }
    }
};
__global__ void __launch_bounds__(256)
k_lf_seg_count(const int32_t* __restrict__ idx, int64_t m, int k, Cut cut, int nseg, int64_t total, uint32_t* __restrict__ segcnt) {
    __shared__ uint32_t h[4][33];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < 33) h[wave][lane] = 0;
    __syncthreads();
    const LfRun run(idx, m, k, cut, nseg, total);
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u < run.n) atomicAdd(&h[wave][run.block[u]], 1u);
    __syncthreads();
    if (run.on && lane < cut.nfb) segcnt[((size_t)run.w * cut.nfb + lane) * nseg + run.seg] = h[wave][lane];
}
// segcnt[wg][seg] -> the counts of the runs before seg (in place); n_ent[wg] = all of them.  One block per workgroup wg.
__global__ void __launch_bounds__(256)
k_lf_seg_scan(uint32_t* __restrict__ segcnt, int nseg, uint32_t* __restrict__ n_ent) {
    __shared__ uint32_t part[256];
    uint32_t* c = segcnt + (size_t)blockIdx.x * nseg;
    uint32_t carry = 0;
    for (int q0 = 0; q0 < nseg; q0 += 256) {
        const int q = q0 + (int)threadIdx.x;
        const uint32_t mine = q < nseg ? c[q] : 0u;
        part[threadIdx.x] = mine;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const uint32_t t = threadIdx.x >= (unsigned)o ? part[threadIdx.x - o] : 0u;
            __syncthreads();
            part[threadIdx.x] += t;
            __syncthreads();
        }
        if (q < nseg) c[q] = carry + part[threadIdx.x] - mine;
        carry += part[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) n_ent[blockIdx.x] = carry;
}
__global__ void __launch_bounds__(256)
k_lf_seg_place(const int32_t* __restrict__ idx, int64_t m, int k, Cut cut, int nseg, int64_t total, const uint32_t* __restrict__ segbase,
               const uint32_t* __restrict__ ent_base, uint32_t* __restrict__ pos /* or NULL */, uint32_t* __restrict__ slot_at,
               uint16_t* __restrict__ feat_at) {
    // A run's connections are put into the order of their places in LDS, so that a store writes a few stretches of consecutive
    // places; each lane storing its own four, what bounded this was the number of lines per store (80 us at m = 500k, d = 32k,
    // k = 32, now 69).
    __shared__ uint32_t h[4][33], base[4][33];   // per block: connections; first place, less what lies before it in the run
    __shared__ uint32_t sorted[4][SEG];          // slot within the run | feature within the block << 8 | block << 19
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < 33) h[wave][lane] = 0;
    __syncthreads();
    const LfRun run(idx, m, k, cut, nseg, total);
    uint32_t r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = u < run.n ? atomicAdd(&h[wave][run.block[u]], 1u) : 0u;
    __syncthreads();
    {
        const uint32_t n = lane < cut.nfb ? h[wave][lane] : 0u;   // (features that the layer does not have get no place)
        uint32_t before = n;
        for (int o = 1; o < 32; o <<= 1) {
            const uint32_t t = __shfl_up(before, o);
            if (lane >= o) before += t;
        }
        before -= n;
        if (run.on && lane < cut.nfb) {
            h[wave][lane] = before;
            base[wave][lane] = ent_base[run.w * cut.nfb + lane] + segbase[((size_t)run.w * cut.nfb + lane) * nseg + run.seg] - before;
        }
        if (lane == cut.nfb - 1) h[wave][32] = before + n;   // all that have a place
    }
    __syncthreads();
    const int have = run.on ? (int)h[wave][32] : 0;
    uint32_t place[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t b = run.block[u];
        place[u] = PAD_SLOT;
        if (u < run.n && b < (uint32_t)cut.nfb) {
            const uint32_t at = h[wave][b] + r[u];
            place[u] = base[wave][b] + at;
            sorted[wave][at] = (uint32_t)(lane * 4 + u) | (run.col[u] - b * (uint32_t)cut.fpb) << 8 | b << 19;
        }
    }
    if (pos) {
        typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
        if (run.n == 4) *reinterpret_cast<u32x4_any*>(pos + run.e) = (u32x4_any){place[0], place[1], place[2], place[3]};
        else
            for (int u = 0; u < run.n; ++u) pos[run.e + u] = place[u];
    }
    __syncthreads();
    const uint32_t first = (uint32_t)(run.e - (size_t)lane * 4);
#pragma unroll
    for (int u = 0; u < SEG / 64; ++u) {
        const int i = u * 64 + lane;
        if (i >= have) break;
        const uint32_t v = sorted[wave][i], p = base[wave][v >> 19] + (uint32_t)i;
        slot_at[p] = first + (v & 255u);
        feat_at[p] = (uint16_t)(v >> 8 & 2047u);
    }
}

// Bank-aware order of the entries in every lane's lists.  At step t of the gathers the 32 lanes of a half-wavefront
// read slot t of their own lists; the sum does not depend on the order of a list, so each list is permuted so that
// the 32 addresses of a step fall into different LDS banks as far as possible (a step costs as many LDS cycles as its
// fullest bank has lanes).  The order is built step by step as a sequence of matchings between the 32 lanes and the
// 32 banks over the entries not placed yet (k_matching.h), the same construction as for the slots of a label in the
// forward product, with one addition: a list shorter than the wavefront's allowance has
// empty places, which may go to any step and read any bank.  A lane that finds no bank among its entries spends an
// empty place (it then reads the zero word of a free bank, see ZERO_LABEL) while it has one.
// One half-wavefront per (workgroup of the gather kernel, zone, 32 lanes); lane i is list i and also bank i.
// Reads the lists as k_lf_plan grouped them (ent), writes them ordered into the places the gather kernel loads its
// registers from (lab: [workgroup][slot / 8][lane][slot % 8], see half_at; slot: [workgroup][slot][lane]) and what exceeds the
// allowance into the overflow list.  Any outcome is a valid order: it changes speed, never results.  rounds = 0: the lists stay in the order of ent.
// pos (if given, see k_lf_seg_place): every entry's place among its workgroup's weight gradients goes along, into rk
// (laid out like slot) or ovrk (beside ov); an empty place gets PAD_SLOT.  A workgroup of at most small_wg entries, as all are
// unless the connectivity is skewed, has labels and places in ent, and places of 16 bits in rk, laid out like lab, at the
// beginning of its part; slot_at (NULL: one block of features) has its flat slots by place.
// GS = lanes and banks of a group: 32, or 16 where the gathers are 16 bytes wide (the lanes of a half-wavefront that such a
// read serves together: 0-3, 12-15, 20-27 and the other 16).
constexpr int SG_NT = 256;   // lanes per workgroup
template <int KTOT, int GS>
__global__ void __launch_bounds__(SG_NT)
k_lf_schedule(const uint32_t* __restrict__ ent, const uint32_t* __restrict__ ent_base, const uint32_t* __restrict__ where,
              const uint32_t* __restrict__ count, const uint16_t* __restrict__ feat, const uint32_t* __restrict__ caps,
              const uint32_t* __restrict__ ov_base, const uint32_t* __restrict__ ov_off, int k, Cut cut,
              uint32_t zero_label, int rounds, uint16_t* __restrict__ lab, uint32_t* __restrict__ slot, OvEntry* __restrict__ ov,
              const uint32_t* __restrict__ pos, const uint32_t* __restrict__ slot_at, uint32_t small_wg, uint32_t* __restrict__ rk,
              uint32_t* __restrict__ ovrk) {
    constexpr int SG = SG_NT / GS;
    typedef usl_bank_lists<GS, KTOT> Lists;
    __shared__ typename Lists::Lane lists[SG][GS];
    __shared__ uint8_t ord[SG][GS][KTOT + 4];     // first the bank of every entry of mine, then the entry at step s (128 + b: none, bank b)
    __shared__ int deg0[SG][GS];                  // entries of the group that read a bank and are not placed yet
    __shared__ uint32_t win[SG][GS];
    const int gl = threadIdx.x / GS, lane = threadIdx.x & (GS - 1);
    // half-wavefront of the gather kernel; an XCD (blockIdx.x % 8) takes an eighth of them in this order: the places that the
    // lists of a window look up (pos) are then read through one L2
    const size_t gid = ((size_t)(blockIdx.x & 7) * (gridDim.x / 8) + (blockIdx.x >> 3)) * (SG_NT / 32) + (threadIdx.x >> 5);
    const size_t wg = gid >> 6;
    const int zone = (int)(gid >> 5) & 1, half = (int)gid & 31;   // the two halves of a wavefront are neighbours: same allowance
    const int mypos = half * 32 + usl_lane_of_position<GS>(threadIdx.x & 31);
    const uint32_t cw = caps[wg * (NT / 64) + (half >> 1)];
    const int cap = zone ? (int)(cw >> 8) : (int)(cw & 0xFFu);
    const int w = (int)(wg / cut.nfb), fb = (int)(wg % cut.nfb);
    auto at = [&](int p) -> size_t { return (wg * KTOT + (zone ? KTOT - 1 - p : p)) * NT + mypos; };
    const bool small = pos && ent_base[wg + 1] - ent_base[wg] <= small_wg;
    const uint32_t inv_k = inverse_of(k);   // the same for all lanes
    auto label_of = [&](uint32_t e) { return small ? e & 0xFFFFu : label_of_slot<KTOT>(e, k, inv_k, (uint32_t)w * (uint32_t)cut.wl, cut); };
    auto place_of = [&](uint32_t e) { return small ? e >> 16 : pos[e] - ent_base[wg]; };
    // four steps' labels, entries (PAD_SLOT: none; no entry is that: a place is below 65535) and places at once: neighbours in the lane's record (caps are multiples of 4)
    auto leave = [&](int s, const uint32_t (&l)[4], const uint32_t (&e)[4]) {
        const int t = zone ? KTOT - 4 - s : s;
        auto two = [&](uint32_t lo, uint32_t hi) { return zone ? hi & 0xFFFFu | lo << 16 : lo & 0xFFFFu | hi << 16; };
        auto four = [&](const uint32_t (&v)[4]) { return zone ? make_uint2(two(v[2], v[3]), two(v[0], v[1])) : make_uint2(two(v[0], v[1]), two(v[2], v[3])); };
        *reinterpret_cast<uint2*>(lab + half_at<KTOT>(wg, t, mypos)) = four(l);
        if (slot) {
#pragma unroll
            for (int u = 0; u < 4; ++u) slot[at(s + u)] = e[u];
        }
        if (pos) {
            uint32_t place[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) place[u] = e[u] != PAD_SLOT ? place_of(e[u]) : PAD_SLOT;
            if (small) {
                *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(rk + wg * KTOT * NT) + half_at<KTOT>(0, t, mypos)) = four(place);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) rk[at(s + u)] = place[u];
            }
        }
    };
    // my list: feature, length, where its entries are
    const uint32_t f = feat[(wg * 2 + zone) * NT + mypos];
    const bool exists = (int)f < min(cut.fpb, cut.vd - fb * cut.fpb);
    const size_t bin = exists ? (size_t)w * cut.vd + (size_t)fb * cut.fpb + f : 0;
    const uint32_t len = exists ? count[bin] : 0u;
    const uint32_t* my = ent + ent_base[wg] + (exists ? where[bin] : 0u);
    const int n = (int)min(len, (uint32_t)cap);     // entries that get a register slot
    for (uint32_t p = (uint32_t)cap; p < len; ++p) {   // the others: to the list's part of the overflow list
        OvEntry o;
        const uint32_t e = my[p];
        o.feature = (uint16_t)f; o.label = (uint16_t)label_of(e);
        o.slot = !small ? e : slot_at ? slot_at[ent_base[wg] + place_of(e)] : ent_base[wg] + place_of(e);
        ov[(size_t)ov_base[wg] + ov_off[bin] + (p - (uint32_t)cap)] = o;
        if (pos) ovrk[(size_t)ov_base[wg] + ov_off[bin] + (p - (uint32_t)cap)] = place_of(e);
    }
    if (len > (uint32_t)cap && ((len - (uint32_t)cap) & 1u)) {   // an odd number: one empty place behind them
        OvEntry o;
        o.feature = (uint16_t)f; o.label = (uint16_t)zero_label; o.slot = PAD_SLOT;
        ov[(size_t)ov_base[wg] + ov_off[bin] + (len - (uint32_t)cap)] = o;
        if (pos) ovrk[(size_t)ov_base[wg] + ov_off[bin] + (len - (uint32_t)cap)] = PAD_SLOT;
    }
    if (rounds <= 0) {
        for (int s = 0; s < cap; s += 4) {
            uint32_t l[4], e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                e[u] = s + u < n ? my[s + u] : PAD_SLOT;
                l[u] = s + u < n ? label_of(e[u]) : zero_label;
            }
            leave(s, l, e);
        }
        return;   // the whole wavefront: rounds is the same for all
    }
    deg0[gl][lane] = 0;
    __syncthreads();
    uint32_t avail = Lists::build(lists[gl][lane], ord[gl][lane], n, deg0[gl], [&](int p) { return (int)(label_of(my[p]) & (GS - 1u)); });
    int wild = cap - n;            // empty places left
    __syncthreads();
    usl_matching<GS> match(win[gl], lane);
    for (int s = 0; s < cap; ++s) {
        match.run(avail, rounds);
        // lists without a bank: an empty place if one is left, on a bank nobody reads (there are as many free banks as
        // lists without one)
        const bool spend = match.mb < 0 && wild > 0;
        int wb = 0;
        if (__any(spend)) {
            const uint32_t spenders = match.ballot(spend);
            uint32_t fb = match.ballot(match.ml < 0);
            if (spend) {
                for (int q = __popc(spenders & ((1u << lane) - 1u)); q > 0; --q) fb &= fb - 1;
                wb = __ffs((int)fb) - 1;
                --wild;
            }
        }
        const int mb = match.double_up(avail, match.mb < 0 && !spend, deg0[gl], cap - s);
        if (spend) {               // the zero word of the free bank
            ord[gl][lane][s] = (uint8_t)(128 + wb);
        } else {                   // my next unplaced entry in that bank
            ord[gl][lane][s] = (uint8_t)Lists::take(lists[gl][lane], mb, avail);
            atomicSub(&deg0[gl][mb], 1);
        }
    }
    // out, several places' loads in flight together
#pragma unroll 2
    for (int s = 0; s < cap; s += 4) {
        uint32_t l[4], e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int pick = ord[gl][lane][s + u];
            e[u] = pick < 128 ? my[pick] : PAD_SLOT;
            l[u] = pick < 128 ? label_of(e[u]) : zero_label + (uint32_t)(pick - 128);
        }
        leave(s, l, e);
    }
}

typedef const __attribute__((address_space(3))) float lds_f32_t;
// acc += sum of w[u] * row[label u] over the four labels packed in p0, p1 (16 bits each).  One instruction per
// address (the 16-bit half is selected and scaled to a byte offset in one go; the row starts at LDS address 0: the
// kernel has no static LDS, and the launcher checks that), the four reads in flight together, each multiply-add as
// soon as its value is there.  Written out because the compiler, short of registers in this kernel, issues one read
// at a time and waits for it.
__device__ __forceinline__ void gather4(float& acc, uint32_t p0, uint32_t p1, float w0, float w1, float w2, float w3) {
    uint32_t a0, a1, a2, a3;
    const uint32_t two = 2;
    asm volatile(
        "v_lshlrev_b32_sdwa %1, %5, %6 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "v_lshlrev_b32_sdwa %2, %5, %6 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "v_lshlrev_b32_sdwa %3, %5, %7 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "v_lshlrev_b32_sdwa %4, %5, %7 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "ds_read_b32 %1, %1\n\t"
        "ds_read_b32 %2, %2\n\t"
        "ds_read_b32 %3, %3\n\t"
        "ds_read_b32 %4, %4\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %8, %1\n\t"
        "s_waitcnt lgkmcnt(2)\n\t"
        "v_fmac_f32 %0, %9, %2\n\t"
        "s_waitcnt lgkmcnt(1)\n\t"
        "v_fmac_f32 %0, %10, %3\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_fmac_f32 %0, %11, %4"
        : "+&v"(acc), "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3)
        : "s"(two), "v"(p0), "v"(p1), "v"(w0), "v"(w1), "v"(w2), "v"(w3)
        : "memory");
}

// The gathers.  grid: ceil(nwin / 8) * 8 * nfb workgroups; all feature blocks of a window run on one XCD (workgroups
// are dealt to the 8 XCDs round robin), so its slice of g is fetched from HBM once and served from that XCD's L2.
// LDS: see LDS_BYTES.
template <typename TS>
__global__ void __launch_bounds__(NT)
k_bwi_lds(const float* __restrict__ g, const TS* __restrict__ W, int64_t m, int k, int rows, int d, int wl, int nfb, int nwin,
          const uint16_t* __restrict__ lab, const uint32_t* __restrict__ slot, const uint16_t* __restrict__ feat,
          const uint32_t* __restrict__ caps, const uint32_t* __restrict__ ov_base, const OvEntry* __restrict__ ov,
          const uint32_t* __restrict__ ovr, float* __restrict__ partial, const uint32_t* __restrict__ gate) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    if (gate && *gate == 0) return;   // the kernels over the nonzero gradients do this call's work
    const int w = (blockIdx.x & 7) + 8 * (blockIdx.x / (8 * nfb)), fb = (blockIdx.x >> 3) % nfb;
    if (w >= nwin) return;
    const size_t wg = (size_t)w * nfb + fb;
    const uint32_t cw = caps[wg * (NT / 64) + (threadIdx.x >> 6)];
    const int acap = __builtin_amdgcn_readfirstlane((int)(cw & 0xFFu)), bcap = __builtin_amdgcn_readfirstlane((int)(cw >> 8));
    uint32_t pk[KT_BWI / 2];
    float wt[KT_BWI];
    const uint32_t last_slot = (uint32_t)(m * k - 1);
    load_words<KT_BWI>(reinterpret_cast<const uint4*>(lab) + wg * pieces_of<KT_BWI>() * NT, threadIdx.x, pk);
#pragma unroll
    for (int q = 0; q < KT_BWI / 4; ++q) {
        const bool used = q * 4 < acap || q * 4 >= KT_BWI - bcap;   // the same for the whole wavefront
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = q * 4 + u;
            float wv = 0.f;
            if (used) {
                const uint32_t s = slot[(wg * KT_BWI + t) * NT + threadIdx.x];
                wv = usl_load_f32<TS>(W, (size_t)min(s, last_slot));   // an empty place reads some weight and drops it
                wv = s != PAD_SLOT ? wv : 0.f;
            }
            wt[t] = wv;
        }
    }
    const uint32_t ov0 = ov_base[wg], ov_n = ov_base[wg + 1] - ov0;
    float* row = reinterpret_cast<float*>(lds_raw);
    float* outbuf = row + WL;
    // which features the lane's two sums belong to: kept in LDS, not in registers (the lists need those)
    uint32_t* feat_of = reinterpret_cast<uint32_t*>(outbuf + NF);
    feat_of[threadIdx.x] = (uint32_t)feat[(wg * 2 + 0) * NT + threadIdx.x] | (uint32_t)feat[(wg * 2 + 1) * NT + threadIdx.x] << 16;
    // the first NT entries that did not fit the registers, with their weights: {feature | label << 16, weight}
    uint2* ov_near = reinterpret_cast<uint2*>(feat_of + NT);
    if (threadIdx.x < ov_n) {
        const OvEntry o = ov[(size_t)ov0 + threadIdx.x];
        ov_near[threadIdx.x] = make_uint2((uint32_t)o.label * 4u,   // an empty place: the zero word, no weight
                                          o.slot == PAD_SLOT ? 0u : __float_as_uint(usl_load_f32<TS>(W, (size_t)o.slot)));
    } else {
        ov_near[threadIdx.x] = make_uint2(ZERO_LABEL * 4u, 0u);
    }
    // ... and which of them belong to the lane's two lists (start | n << 16)
    uint32_t* ovr_a = reinterpret_cast<uint32_t*>(ov_near + NT);
    uint32_t* ovr_b = ovr_a + NT;
    ovr_a[threadIdx.x] = ovr[(wg * 2 + 0) * NT + threadIdx.x];
    ovr_b[threadIdx.x] = ovr[(wg * 2 + 1) * NT + threadIdx.x];
    if (threadIdx.x < 32) reinterpret_cast<uint32_t*>(lds_raw)[ZERO_LABEL + threadIdx.x] = 0u;
    const int nl = (int)max((int64_t)0, min((int64_t)wl, m - (int64_t)w * wl));   // labels of this window (the last one may be short)
    const int nv = nl / 4, full = nv & ~63;                      // 16-byte pieces of a row slice; those in whole 1 KiB runs
    const int lines = (nl * 4 + 127) / 128, per = (lines + nfb - 1) / nfb;   // 128-byte lines; this workgroup's share of the warm-up
    const bool warms = (int)threadIdx.x < per && fb * per + (int)threadIdx.x < lines;
    // the rest of a list (r = start | n << 16 in ov_near, n even), two entries in flight at a time
    auto more = [&](float& acc, uint32_t r) {
        for (uint32_t q = r & 0xFFFFu, e = q + (r >> 16); q < e; q += 2) {
            const uint2 o0 = ov_near[q], o1 = ov_near[q + 1];
            const float v0 = *reinterpret_cast<lds_f32_t*>(static_cast<uintptr_t>(o0.x));
            const float v1 = *reinterpret_cast<lds_f32_t*>(static_cast<uintptr_t>(o1.x));
            acc = fmaf(__uint_as_float(o0.y), v0, acc);
            acc = fmaf(__uint_as_float(o1.y), v1, acc);
        }
    };
    // Receives the L2 warm-up loads, which are issued from inline assembly: the compiler then puts no wait behind them
    // (behind a load it knows of whose value is never used, or a volatile one, it waits on the spot: a trip to memory
    // at the start of this wavefront's gathers, 0.14 ms per call at m = 500k).  The register must not be touched until
    // the vmcnt(0) wait at the top of the next pass; the build checks that in the compiler's listing (build.py).
    uint32_t token = 0;
    for (int i = 0; i < rows; ++i) {
        const char* grow = reinterpret_cast<const char*>(g + (size_t)w * wl + (size_t)i * m);   // uniform
        {   // the row slice: whole 1 KiB pieces by LDS-DMA, the ragged end through registers
            for (int v = (threadIdx.x >> 6) * 64; v < full; v += NT)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(grow + ((uint32_t)v * 16u + (threadIdx.x & 63u) * 16u)),
                                                 (__attribute__((address_space(3))) void*)(lds_raw + (size_t)v * 16), 16, 0, 0);
            for (int v = full + threadIdx.x; v < nv; v += NT)
                reinterpret_cast<uint4*>(lds_raw)[v] = reinterpret_cast<const uint4*>(grow)[v];
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            asm volatile("" : "+v"(token));
        }
        __syncthreads();
        if (i + 1 < rows && warms)   // the window's workgroups share the warm-up of the next row slice, one load per 128-byte line
            asm volatile("global_load_dword %0, %1, %2" : "=v"(token) : "v"((uint32_t)(fb * per + (int)threadIdx.x) * 128u), "s"(grow + (size_t)m * 4));
        float acc_a = 0.f, acc_b = 0.f;
        // compared afresh in every pass (one scalar compare per group): kept across the loop, the 34 outcomes would
        // each take a pair of scalar registers, more than there are
        int ac = acap, bc = bcap;
        asm volatile("" : "+s"(ac), "+s"(bc));
#pragma unroll
        for (int q = 0; q < KT_BWI / 4; ++q) {
            if (q * 4 < ac) {
                gather4(acc_a, pk[q * 2], pk[q * 2 + 1], wt[q * 4], wt[q * 4 + 1], wt[q * 4 + 2], wt[q * 4 + 3]);
            }
        }
#pragma unroll
        for (int q = 0; q < KT_BWI / 4; ++q) {
            if (q * 4 >= KT_BWI - bc) {
                gather4(acc_b, pk[q * 2], pk[q * 2 + 1], wt[q * 4], wt[q * 4 + 1], wt[q * 4 + 2], wt[q * 4 + 3]);
            }
        }
        if (ov_n) {   // the same for the whole workgroup: the few lanes whose lists did not fit go on through LDS
            more(acc_a, ovr_a[threadIdx.x]);
            more(acc_b, ovr_b[threadIdx.x]);
        }
        {
            const uint32_t f = feat_of[threadIdx.x];
            outbuf[f & 0xFFFFu] = acc_a;
            outbuf[f >> 16] = acc_b;
        }
        if (ov_n > (uint32_t)NT) {   // only a skewed connectivity gets here: what LDS does not hold, by atomics
            __syncthreads();
            for (uint32_t q = NT + threadIdx.x; q < ov_n; q += NT) {
                const OvEntry o = ov[(size_t)ov0 + q];
                if (o.slot != PAD_SLOT) unsafeAtomicAdd(&outbuf[o.feature], usl_load_f32<TS>(W, (size_t)o.slot) * row[o.label]);
            }
        }
        __syncthreads();
        {   // the block's NF sums leave as one contiguous run
            float* dst = partial + ((size_t)w * rows + i) * d + (size_t)fb * NF;
            for (int v = threadIdx.x; v < NF / 4; v += NT)
                reinterpret_cast<float4*>(dst)[v] = reinterpret_cast<const float4*>(outbuf)[v];
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("" : "+v"(token));
}

// ---------------------------------------------------------------------------------------------------------------
// Both backward products from one pass of gathers (usl_train_step, usl_backward).  Every gathered g[i][j] serves twice:
// times the connection's weight it goes into the feature's sum (Algorithm 2), times the feature's activation x[i][c] into a
// sum that the lane keeps per slot over the whole batch (Algorithm 3) and stores at the end -- every slot of the layer
// belongs to exactly one list of one workgroup, so every weight gradient is written once, without atomics.  The third
// register per slot halves the slots (KT_BOTH = 36) and with them the windows; the row buffer then has room for the
// slices of two instances, and a pass of the loop does two instances.  They lie interleaved, so a slot costs one address,
// one ds_read_b64 and four multiply-adds: 64 random 8-byte reads take LDS no longer than 64 random 4-byte ones (before,
// with the slices one behind the other and two ds_read_b32, usl_backward took 1408 us at m = 500k, d = 32k, k = 32,
// b = 256 and 6662 us at m = 670k, k = 64, b = 512; now 1310 and 5350 to 5590).  What bounds it at the first of these
// (1052 us, two windows of 128 passes per workgroup, the lists of a window 20 us): LDS is busy for half of the time, nearly
// half of that with bank conflicts (profiles/products_large_f32_lds_bank_conflicts.txt), the row copies take a third of a
// pass at the L2 -> LDS rate, and copy, gathers and sums of a pass follow one another, with barriers between them.
// The sums of overflow entries live in LDS (ov_sum) or, beyond the NEAR2 that LDS holds, in memory (ovgw).
// acc and x are arrays on purpose: handed over one by one, the second list's activations are asked for in a branch of their own, and every group of the
// first list begins with a wait for all LDS reads (m = 500k, d = 32k, k = 32, b = 256: the step 1965 us, so 1956).
__device__ __forceinline__ void gather4_two(float (&acc)[2], float& s0, float& s1, float& s2, float& s3,
                                            uint32_t p0, uint32_t p1, float w0, float w1, float w2, float w3, const float (&x)[2]) {
    const uint32_t three = 3;
    asm volatile(
        "v_lshlrev_b32_sdwa v112, %6, %7 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "v_lshlrev_b32_sdwa v114, %6, %7 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "v_lshlrev_b32_sdwa v116, %6, %8 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "v_lshlrev_b32_sdwa v118, %6, %8 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "ds_read_b64 v[112:113], v112\n\t"
        "ds_read_b64 v[114:115], v114\n\t"
        "ds_read_b64 v[116:117], v116\n\t"
        "ds_read_b64 v[118:119], v118\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %9, v112\n\t"
        "v_fmac_f32 %1, %9, v113\n\t"
        "v_fmac_f32 %2, %13, v112\n\t"
        "v_fmac_f32 %2, %14, v113\n\t"
        "s_waitcnt lgkmcnt(2)\n\t"
        "v_fmac_f32 %0, %10, v114\n\t"
        "v_fmac_f32 %1, %10, v115\n\t"
        "v_fmac_f32 %3, %13, v114\n\t"
        "v_fmac_f32 %3, %14, v115\n\t"
        "s_waitcnt lgkmcnt(1)\n\t"
        "v_fmac_f32 %0, %11, v116\n\t"
        "v_fmac_f32 %1, %11, v117\n\t"
        "v_fmac_f32 %4, %13, v116\n\t"
        "v_fmac_f32 %4, %14, v117\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_fmac_f32 %0, %12, v118\n\t"
        "v_fmac_f32 %1, %12, v119\n\t"
        "v_fmac_f32 %5, %13, v118\n\t"
        "v_fmac_f32 %5, %14, v119"
        : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(s0), "+&v"(s1), "+&v"(s2), "+&v"(s3)
        : "s"(three), "v"(p0), "v"(p1), "v"(w0), "v"(w1), "v"(w2), "v"(w3), "v"(x[0]), "v"(x[1])
        : "memory", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119");
}

// The same for four instances, 16-byte reads and eight multiply-adds per slot: a group of four and, where n > most, the next one of its list, with four reads in flight throughout, in the same registers: each of the second group's
// is asked for where the one four before it has been used.  (The branch is in here: two statements that change the same registers on either side
// of one cost copies and reloads.)  Steps with groups of four by themselves and so: m = 200k, d = 8k, k = 32, b = 64, bfloat16 213.0 and 211.1 us, b = 128 352.7 and 349.0; m = 70k,
// d = 10k, k = 48, b = 100 193.5 and 193.2; m = 670k, d = 16k, k = 32, b = 32 549.9 and 548.1; m = 31k, d = 1k, b = 128 81.6 both (two runs of one side differ by up to 0.2 %).  Not
// with two instances: 500k x 32k, b = 256 1940 both, and its code, which every launch has to bring in, costs small batches up to 1 us (58k x 6k, k = 8, b = 8 47.4 and
// 48.4; 150k x 30k, b = 64 298.8 and 299.9).
__device__ __forceinline__ void gather8(float (&acc)[4], float* s, const uint32_t* p, const float* w, float* s_far, const uint32_t* p_far, const float* w_far,
                                        const float (&x)[4], int n, int most) {
    const uint32_t shift = 4;
    asm volatile(
        "v_lshlrev_b32_sdwa v112, %12, %13 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "ds_read_b128 v[112:115], v112\n\t"
        "v_lshlrev_b32_sdwa v116, %12, %13 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "ds_read_b128 v[116:119], v116\n\t"
        "v_lshlrev_b32_sdwa v120, %12, %14 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "ds_read_b128 v[120:123], v120\n\t"
        "v_lshlrev_b32_sdwa v124, %12, %14 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "ds_read_b128 v[124:127], v124\n\t"
        "s_cmp_le_i32 %29, %30\n\t"
        "s_cbranch_scc1 .Lnear%=\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %17, v112\n\t"
        "v_fmac_f32 %1, %17, v113\n\t"
        "v_fmac_f32 %2, %17, v114\n\t"
        "v_fmac_f32 %3, %17, v115\n\t"
        "v_fmac_f32 %4, %25, v112\n\t"
        "v_fmac_f32 %4, %26, v113\n\t"
        "v_fmac_f32 %4, %27, v114\n\t"
        "v_fmac_f32 %4, %28, v115\n\t"
        "v_lshlrev_b32_sdwa v112, %12, %15 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "ds_read_b128 v[112:115], v112\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %18, v116\n\t"
        "v_fmac_f32 %1, %18, v117\n\t"
        "v_fmac_f32 %2, %18, v118\n\t"
        "v_fmac_f32 %3, %18, v119\n\t"
        "v_fmac_f32 %5, %25, v116\n\t"
        "v_fmac_f32 %5, %26, v117\n\t"
        "v_fmac_f32 %5, %27, v118\n\t"
        "v_fmac_f32 %5, %28, v119\n\t"
        "v_lshlrev_b32_sdwa v116, %12, %15 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "ds_read_b128 v[116:119], v116\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %19, v120\n\t"
        "v_fmac_f32 %1, %19, v121\n\t"
        "v_fmac_f32 %2, %19, v122\n\t"
        "v_fmac_f32 %3, %19, v123\n\t"
        "v_fmac_f32 %6, %25, v120\n\t"
        "v_fmac_f32 %6, %26, v121\n\t"
        "v_fmac_f32 %6, %27, v122\n\t"
        "v_fmac_f32 %6, %28, v123\n\t"
        "v_lshlrev_b32_sdwa v120, %12, %16 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t"
        "ds_read_b128 v[120:123], v120\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %20, v124\n\t"
        "v_fmac_f32 %1, %20, v125\n\t"
        "v_fmac_f32 %2, %20, v126\n\t"
        "v_fmac_f32 %3, %20, v127\n\t"
        "v_fmac_f32 %7, %25, v124\n\t"
        "v_fmac_f32 %7, %26, v125\n\t"
        "v_fmac_f32 %7, %27, v126\n\t"
        "v_fmac_f32 %7, %28, v127\n\t"
        "v_lshlrev_b32_sdwa v124, %12, %16 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t"
        "ds_read_b128 v[124:127], v124\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %21, v112\n\t"
        "v_fmac_f32 %1, %21, v113\n\t"
        "v_fmac_f32 %2, %21, v114\n\t"
        "v_fmac_f32 %3, %21, v115\n\t"
        "v_fmac_f32 %8, %25, v112\n\t"
        "v_fmac_f32 %8, %26, v113\n\t"
        "v_fmac_f32 %8, %27, v114\n\t"
        "v_fmac_f32 %8, %28, v115\n\t"
        "s_waitcnt lgkmcnt(2)\n\t"
        "v_fmac_f32 %0, %22, v116\n\t"
        "v_fmac_f32 %1, %22, v117\n\t"
        "v_fmac_f32 %2, %22, v118\n\t"
        "v_fmac_f32 %3, %22, v119\n\t"
        "v_fmac_f32 %9, %25, v116\n\t"
        "v_fmac_f32 %9, %26, v117\n\t"
        "v_fmac_f32 %9, %27, v118\n\t"
        "v_fmac_f32 %9, %28, v119\n\t"
        "s_waitcnt lgkmcnt(1)\n\t"
        "v_fmac_f32 %0, %23, v120\n\t"
        "v_fmac_f32 %1, %23, v121\n\t"
        "v_fmac_f32 %2, %23, v122\n\t"
        "v_fmac_f32 %3, %23, v123\n\t"
        "v_fmac_f32 %10, %25, v120\n\t"
        "v_fmac_f32 %10, %26, v121\n\t"
        "v_fmac_f32 %10, %27, v122\n\t"
        "v_fmac_f32 %10, %28, v123\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_fmac_f32 %0, %24, v124\n\t"
        "v_fmac_f32 %1, %24, v125\n\t"
        "v_fmac_f32 %2, %24, v126\n\t"
        "v_fmac_f32 %3, %24, v127\n\t"
        "v_fmac_f32 %11, %25, v124\n\t"
        "v_fmac_f32 %11, %26, v125\n\t"
        "v_fmac_f32 %11, %27, v126\n\t"
        "v_fmac_f32 %11, %28, v127\n\t"
        "s_branch .Lend%=\n"
        ".Lnear%=:\n\t"
        "s_waitcnt lgkmcnt(3)\n\t"
        "v_fmac_f32 %0, %17, v112\n\t"
        "v_fmac_f32 %1, %17, v113\n\t"
        "v_fmac_f32 %2, %17, v114\n\t"
        "v_fmac_f32 %3, %17, v115\n\t"
        "v_fmac_f32 %4, %25, v112\n\t"
        "v_fmac_f32 %4, %26, v113\n\t"
        "v_fmac_f32 %4, %27, v114\n\t"
        "v_fmac_f32 %4, %28, v115\n\t"
        "s_waitcnt lgkmcnt(2)\n\t"
        "v_fmac_f32 %0, %18, v116\n\t"
        "v_fmac_f32 %1, %18, v117\n\t"
        "v_fmac_f32 %2, %18, v118\n\t"
        "v_fmac_f32 %3, %18, v119\n\t"
        "v_fmac_f32 %5, %25, v116\n\t"
        "v_fmac_f32 %5, %26, v117\n\t"
        "v_fmac_f32 %5, %27, v118\n\t"
        "v_fmac_f32 %5, %28, v119\n\t"
        "s_waitcnt lgkmcnt(1)\n\t"
        "v_fmac_f32 %0, %19, v120\n\t"
        "v_fmac_f32 %1, %19, v121\n\t"
        "v_fmac_f32 %2, %19, v122\n\t"
        "v_fmac_f32 %3, %19, v123\n\t"
        "v_fmac_f32 %6, %25, v120\n\t"
        "v_fmac_f32 %6, %26, v121\n\t"
        "v_fmac_f32 %6, %27, v122\n\t"
        "v_fmac_f32 %6, %28, v123\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "v_fmac_f32 %0, %20, v124\n\t"
        "v_fmac_f32 %1, %20, v125\n\t"
        "v_fmac_f32 %2, %20, v126\n\t"
        "v_fmac_f32 %3, %20, v127\n\t"
        "v_fmac_f32 %7, %25, v124\n\t"
        "v_fmac_f32 %7, %26, v125\n\t"
        "v_fmac_f32 %7, %27, v126\n\t"
        "v_fmac_f32 %7, %28, v127\n"
        ".Lend%=:"
        : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(s[0]), "+&v"(s[1]), "+&v"(s[2]), "+&v"(s[3]), "+&v"(s_far[0]), "+&v"(s_far[1]), "+&v"(s_far[2]), "+&v"(s_far[3])
        : "s"(shift), "v"(p[0]), "v"(p[1]), "v"(p_far[0]), "v"(p_far[1]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w_far[0]), "v"(w_far[1]), "v"(w_far[2]), "v"(w_far[3]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "s"(n), "s"(most)
        : "memory", "scc", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127");
}
// The values of Q instances at one place of LDS.
__device__ __forceinline__ void unit_of(const float* p, float (&v)[2]) { const float2 t = *reinterpret_cast<const float2*>(p); v[0] = t.x; v[1] = t.y; }
__device__ __forceinline__ void unit_of(const float* p, float (&v)[4]) { const float4 t = *reinterpret_cast<const float4*>(p); v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w; }
__device__ __forceinline__ void unit_of(const uint16_t* p, float (&v)[4]) {
    const uint2 t = *reinterpret_cast<const uint2*>(p);
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xFFFF0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xFFFF0000u);
}
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes of a row that starts anywhere

// base is the same for all lanes, byte the lane's offset: one 32-bit register, no 64-bit address per load
template <typename T>
__device__ __forceinline__ T at_byte(const T* base, uint32_t byte) { return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + byte); }

// Q = 2: windows of up to 15 968 labels (wide layers), x as rows of x_stride elements, 16-byte aligned.
// Q = 4: windows of up to 7 232 labels (4 672 where OWN), x interleaved by fours (x_stride = elements from group to group, k_interleave).
// grid: at least windows * parts of the batch * feature blocks, a multiple of 8.  A part of the batch (rows_per_part
// instances, a multiple of Q) leaves its weight gradient at stage + part * part_stride.
template <typename TS, int Q, bool OWN>
__global__ void __launch_bounds__(NT)
k_both_lds(const float* __restrict__ g, const TS* __restrict__ W, const TS* __restrict__ x, size_t x_stride, int64_t m, int k, int rows, int d,
           int dp, Cut cut, const uint16_t* __restrict__ lab, const uint32_t* __restrict__ slot_at,
           const uint16_t* __restrict__ feat, const uint32_t* __restrict__ caps, const uint32_t* __restrict__ ov_base,
           const OvEntry* __restrict__ ov, const uint32_t* __restrict__ ovr, float* __restrict__ partial,
           const uint32_t* __restrict__ rk, const uint32_t* __restrict__ ovrk, const uint32_t* __restrict__ ent_base,
           float* __restrict__ stage, float* __restrict__ ovgw, int chains, int parts, int rows_per_part, size_t part_stride, size_t ov_stride,
           const uint32_t* __restrict__ gate, int accumulate, const uint32_t* __restrict__ stale) {
    constexpr int KT = Q == 4 ? KT_BOTH4 : KT_BOTH;   // (with four instances 36 slots spill)
    static_assert(KT_BOTH4 % 8 == 0, "groups by twos");
    constexpr uint32_t ZL = BothLayout<Q, OWN>::zero_label, U = 4 * Q;   // U: bytes of a unit
    extern __shared__ __align__(16) unsigned char lds_raw[];
    if (gate && *gate == 0) return;   // the kernels over the nonzero gradients do this call's work
    const int nfb = cut.nfb;
    // workgroup b runs on XCD b % 8: an XCD takes an eighth of the tiles (window, part, feature block) in this order, so that
    // the blocks of a window, which read the same slices of g, and its parts, which read the same lists, share an L2
    const int per_xcd = (int)gridDim.x / 8, tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    const int chain = tile / (parts * nfb), part = tile / nfb % parts, fb = tile % nfb;
    if (chain >= chains) return;
    const int i_begin = part * rows_per_part, i_end = min(rows, i_begin + rows_per_part);
    stage += (size_t)part * part_stride;
    ovgw += (size_t)part * ov_stride;
    if (stale && *stale != 0) {   // one window: partial is grad_x itself, and this kernel does k_lf_reduce's check
        for (size_t v = threadIdx.x; v < (size_t)max(i_end - i_begin, 0) * dp; v += NT) partial[(size_t)i_begin * dp + v] = __uint_as_float(0x7FC00000u);
        return;
    }
    // One window after the other: windows chain, chain + chains, ...  The sums of the later ones are added to the first one's
    // (every value by the lane that wrote it), so that there is one set of partial sums for each chain, not for each window.
#pragma unroll 1
    for (int w = chain; w < cut.nwin; w += chains) {
    uint32_t lane = threadIdx.x;   // taken afresh for each window: nothing computed from it lives through the passes
    asm volatile("" : "+v"(lane));
    const size_t wg = (size_t)__builtin_amdgcn_readfirstlane(w * nfb + fb);
    uint32_t pk[KT / 2];
    float wt[KT], gw[KT];
    // The weights come in the order of the places (slot_at; rk: see the end of the kernel) and are picked up from LDS: in the
    // order of the lists every value was a 128-byte line of its own (96 of 1320 us at m = 500k, d = 32k, k = 32, 25 of 210 at
    // m = 200k, d = 8k, b = 64).  What bounds a window's beginning is the number of loads and the waits for them: the lane's
    // labels and places come 16 bytes at a time, the places of all weights in one go, the weights by LDS-DMA without a register.
    // With loads of 4 bytes and a wait for every eight places a window began in 44 us at m = 500k and ended in 10 (clock
    // counters), now 23 and 8; the step 33.3 -> 31.6 us at m = 1024, d = 64, k = 8, b = 16, 258 -> 251 at m = 200k, d = 8k,
    // k = 32, b = 64 (bfloat16), 2034 -> 1999 at m = 500k, d = 32k, k = 32, b = 256.
    constexpr uint32_t CH = both_places<Q, OWN>();   // places LDS holds at a time
    float* perm = reinterpret_cast<float*>(lds_raw);
    const uint32_t e0 = ent_base[wg], n_ent = ent_base[wg + 1] - e0;
    const uint32_t ov0 = ov_base[wg], ov_n = ov_base[wg + 1] - ov0;
    uint32_t tid4 = threadIdx.x * 4u;
    asm volatile("" : "+v"(tid4));
    const uint32_t first_slot = (uint32_t)w * (uint32_t)cut.wl * (uint32_t)k;   // of the window: 32-bit offsets from there
    const TS* W_window = W + first_slot;
    const bool one_go = n_ent <= CH;   // (unless the connectivity is skewed)
    const uint32_t cw = caps[wg * (NT / 64) + (lane >> 6)];
    uint32_t r[KT / 2];
    load_words<KT>(rk + wg * KT * NT, lane, r);
    load_words<KT>(reinterpret_cast<const uint4*>(lab) + wg * pieces_of<KT>() * NT, lane, pk);
    const uint32_t fa = feat[(wg * 2 + 0) * NT + lane], fbb = feat[(wg * 2 + 1) * NT + lane];
    const uint32_t ovra = ovr[(wg * 2 + 0) * NT + lane], ovrb = ovr[(wg * 2 + 1) * NT + lane];
    OvEntry o = {0, 0, PAD_SLOT};
    if (lane < min((uint32_t)NEAR2, ov_n)) o = ov[(size_t)ov0 + lane];
    __builtin_amdgcn_sched_barrier(0);
    // The weights of the first N * NT places: float32 ones by LDS-DMA, a lane's own address each and no registers.  The weight of
    // the lane's overflow entry goes out with them: behind them it was another trip to memory.
    TS ov_raw = (TS)0;
    auto bring = [&](auto N_) {
        constexpr int N = decltype(N_)::value;
        const uint32_t n_bytes = min(n_ent, CH) * 4;
        uint32_t at = threadIdx.x * 4u, sl[N];   // (a lane past the end reads the last place again)
        asm volatile("" : "+v"(at));
        const uint32_t wave_at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        // Does the wavefront fetch a weight for its lanes' u-th places?  bfloat16 ones always: sl[u] has to hold a slot then.  Float32 ones
        // up to the last place, and a window of few places asks for no more slots than that (a step at m = 31k, d = 1k, k = 32, b = 128:
        // 100.4 and 95.7 us; usl_backward at m = 130k, d = 15k, k = 32, b = 64: 172 and 168; m = 10k, d = 39k, b = 54: 51.0 and 49.4).
        auto fetches = [&](int u) { return sizeof(TS) != 4 || wave_at + (uint32_t)(u * NT * 4) < n_bytes; };
        if (nfb > 1) {
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (u < 8 || fetches(u)) sl[u] = at_byte(slot_at + e0, min(at + (uint32_t)(u * NT * 4), n_bytes - 4));
        } else {
#pragma unroll
            for (int u = 0; u < N; ++u) sl[u] = e0 + min(at + (uint32_t)(u * NT * 4), n_bytes - 4) / 4;
        }
        __builtin_amdgcn_sched_barrier(0);
        if (ov_n) ov_raw = W_window[o.slot != PAD_SLOT ? o.slot - first_slot : 0u];
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (sizeof(TS) == 4) {
            // All slots are waited for here, in one go.  Left to the compiler, each is waited for where its weight is asked for, and where the spills
            // of this kernel came out so that it does not know the order in which those loads return, every wait is for the weights asked for before
            // as well: a chain of trips to memory, 5 us of every launch at m = 31k, d = 1k, k = 32, b = 128.  (With two instances the weights of the first slots are
            // better on their way before the last slots have come: m = 20k, d = 30k, k = 16, b = 64 71.8 and, waited for in one go, 72.6; m = 150k, d = 30k, k = 32, b = 32
            // 197.5 and 199.2, though m = 500k, d = 32k, b = 256 1951 and 1944.)
            if constexpr (Q == 4) {
#pragma unroll
                for (int u = 0; u < N; ++u) asm volatile("" : "+v"(sl[u]));
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (fetches(u))   // (whole wavefronts: at most 63 places behind the last one are written too)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(W_window + (sl[u] - first_slot)),
                                                     (__attribute__((address_space(3))) void*)(lds_raw + wave_at + (size_t)(u * NT * 4)), 4, 0, 0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
            constexpr int B = N < 10 ? N : (N + 3) / 4;
#pragma unroll
            for (int u0 = 0; u0 < N; u0 += B) {
                TS v[B];
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if (u0 + u < N) v[u] = at_byte(W_window, (sl[u0 + u] - first_slot) * (uint32_t)sizeof(TS));
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if (u0 + u < N && wave_at + (uint32_t)((u0 + u) * NT * 4) < n_bytes)
                        *reinterpret_cast<float*>(lds_raw + at + (uint32_t)((u0 + u) * NT * 4)) = usl_to_f32(v[u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    __syncthreads();   // LDS is free
    if (one_go && n_ent > 8 * NT) bring(std::integral_constant<int, ((int)CH + NT - 1) / NT>{});
    else if (one_go && n_ent > 0) bring(std::integral_constant<int, 8>{});
    else if (ov_n) ov_raw = W_window[o.slot != PAD_SLOT ? o.slot - first_slot : 0u];
    const float ov_weight = o.slot != PAD_SLOT ? usl_to_f32(ov_raw) : 0.f;
    const int acap = __builtin_amdgcn_readfirstlane((int)(cw & 0xFFu)), bcap = __builtin_amdgcn_readfirstlane((int)(cw >> 8));
    // (a skewed connectivity: one by one, and the places are just the lane's slots)
    auto own_places = [&](uint32_t (&places)[KT / 2]) {
#pragma unroll
        for (int t = 0; t < KT / 2; ++t) places[t] = (uint32_t)(2 * t * NT) + tid4 / 4 | ((uint32_t)((2 * t + 1) * NT) + tid4 / 4) << 16;
    };
    auto used = [&](int t) { return t / 4 * 4 < acap || t / 4 * 4 >= KT - bcap; };   // the same for the whole wavefront
    constexpr uint32_t NOWHERE = no_place<Q, OWN>();
    auto place_of = [&](const uint32_t (&places)[KT / 2], int t) { return min(t & 1 ? places[t / 2] >> 16 : places[t / 2] & 0xFFFFu, NOWHERE); };
    if (threadIdx.x == 0) perm[NOWHERE] = 0.f;
    if (!one_go) {
#pragma unroll 1
        for (int t = 0; t < KT; ++t) {
            const uint32_t place = used(t) ? (rk + (wg * KT + t) * NT)[threadIdx.x] : PAD_SLOT;
            perm[t * NT + threadIdx.x] = place != PAD_SLOT ? usl_load_f32<TS>(W, (size_t)(nfb > 1 ? (slot_at + e0)[place] : e0 + place)) : 0.f;
        }
        own_places(r);
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < KT; ++t) wt[t] = perm[place_of(r, t)];   // (of slots that nobody visits: anything)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < KT; ++t) {   // (written here, not by the compiler at the top: there the registers are needed)
        float zero = 0.f;
        asm volatile("" : "+v"(zero));
        gw[t] = zero;
    }
    __syncthreads();   // LDS is free
    const float* row = reinterpret_cast<const float*>(lds_raw);           // row[Q * unit + q]: instance q of a pass
    float* outbuf = reinterpret_cast<float*>(lds_raw + BothLayout<Q, OWN>::row_bytes);   // [Q][NF]
    TS* xbuf = reinterpret_cast<TS*>(outbuf + (OWN ? Q * NF : 0));   // Q = 4: [NF][4]; Q = 2: [2][NF]
    uint32_t* feat_of = reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(outbuf + Q * NF) + BothLayout<Q, OWN>::x_bytes);   // [NT]
    uint2* ov_near = reinterpret_cast<uint2*>(feat_of + BothLayout<Q, OWN>::feat_words);   // [NEAR2] {address of the label in the row, weight}
    uint32_t* ov_share = reinterpret_cast<uint32_t*>(ov_near + NEAR2);    // [NT] of the lane's two lists, in pairs of entries: start | n << 8, << 16
    float* ov_sum = reinterpret_cast<float*>(ov_share + NT);              // [NEAR2]
    lane = threadIdx.x;
    asm volatile("" : "+v"(lane));
    const uint32_t feat2 = fa | fbb << 16;
    feat_of[lane] = feat2;
    // OWN: where the features' activations are (a list of a feature that does not exist reads some place, and is empty)
    if (OWN) feat_of[NT + lane] = cut.S == 1 ? feat2 : (feat2 & 0xFFFFu) % (uint32_t)d | (feat2 >> 16) % (uint32_t)d << 16;
    if (lane < NEAR2) {
        ov_near[lane] = make_uint2(o.slot != PAD_SLOT ? (uint32_t)o.label * U : ZL * U, __float_as_uint(ov_weight));   // an empty place: the unit of zeros, no weight
        ov_sum[lane] = 0.f;
    }
    ov_share[lane] = (ovra & 0xFFFFu) / 2 | ovra >> 17 << 8 | (ovrb & 0xFFFFu) / 2 << 16 | ovrb >> 17 << 24;
    if (lane < 32 * Q) reinterpret_cast<uint32_t*>(lds_raw)[ZL * Q + lane] = 0u;   // what empty places read
    for (uint32_t q = NEAR2 + lane; q < ov_n; q += NT) ovgw[(size_t)ov0 + q] = 0.f;   // in the passes entry q is lane (q - NEAR2) % NT's
    const int nl = (int)max((int64_t)0, min((int64_t)cut.wl, m - (int64_t)w * cut.wl));   // labels of this window (the last one may be short)
    const int nv = nl / 4, quarter = cut.wl / 4;                         // whole 16-byte pieces of a row slice; see unit_of_label
    const int nf = min(cut.fpb, cut.vd - fb * cut.fpb);                            // features of this block that exist
    const int nx = cut.S > 1 ? d : nf;                                   // ... and activations
    const int lines = (nl * 4 + 127) / 128, per = (lines + nfb - 1) / nfb;   // 128-byte lines; this workgroup's share of the warm-up
    const int plines = w >= chains && cut.S == 1 ? (nf * 4 + 127) / 128 : 0;   // ... and of its earlier sums (per instance)
    const int xlines = ((Q == 4 ? Q : 1) * nx * (int)sizeof(TS) + 127) / 128;    // 128-byte lines of the block's activations (per row of x)
    // the rest of a list (r = start | n << 8 in pairs of entries of ov_near), two entries in flight at a time
    auto more = [&](float (&acc)[Q], uint32_t r, const float (&xv)[Q]) {
        constexpr int AT_ONCE = Q == 2 ? 2 : 1;   // (four instances leave no registers for two)
#pragma unroll 1
        for (uint32_t q = (r & 0xFFu) * 2, e = q + (r >> 8 & 0xFFu) * 2; q < e; q += AT_ONCE) {
            uint2 o[AT_ONCE];
            float u[AT_ONCE][Q], t[AT_ONCE];
#pragma unroll
            for (int a = 0; a < AT_ONCE; ++a) o[a] = ov_near[q + a];
#pragma unroll
            for (int a = 0; a < AT_ONCE; ++a) { unit_of(row + o[a].x / 4, u[a]); t[a] = ov_sum[q + a]; }   // the entries of a list are its lane's alone
#pragma unroll
            for (int a = 0; a < AT_ONCE; ++a) {
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    acc[i] = fmaf(__uint_as_float(o[a].y), u[a][i], acc[i]);
                    t[a] = fmaf(xv[i], u[a][i], t[a]);
                }
                ov_sum[q + a] = t[a];
            }
        }
    };
    uint32_t token = 0;   // receives the L2 warm-up loads
    for (int i = i_begin; i < i_end; i += Q) {
        const int have = min(Q, i_end - i);                              // instances of this pass; the others read as zeros
        const char* grow = reinterpret_cast<const char*>(g + (size_t)w * cut.wl + (size_t)i * m);   // uniform
        const TS* xrow = Q == 4 ? x + (size_t)(i / Q) * x_stride + (size_t)fb * cut.fpb * Q : x + (size_t)i * x_stride + (size_t)fb * cut.fpb;
        float* dst = partial + ((size_t)chain * rows + i) * dp + (size_t)fb * cut.fpb;   // (one block where S > 1)
        // The lane's number, taken afresh in each part of a pass: whatever is computed from it (addresses in LDS, offsets
        // of copies) is then computed there, in a few instructions, and not kept in a register of its own across the
        // gathers -- there are none to spare, and a value that is spilled comes back through a load whose wait also
        // waits for the warm-up loads.
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        if (Q == 2) {   // the block's activations of the two instances: 1 KiB pieces by LDS-DMA into the place of the sums (free
            // until the gathers are done); read from memory by feature they cost as much as the slices of g.
            // Wavefront v overwrites bytes [1024 v, 1024 v + 1024) of that place: the piece that it alone read when the
            // sums of the pass before left (no barrier since then), so nobody else's sums are lost.
            static_assert(2 * NF / 4 == NT, "a lane copies out one float4 of the sums: wavefront v the v-th KiB");
            constexpr int PR = NF * (int)sizeof(TS) / 1024;
            const int wv = (int)(tid >> 6), piece = (wv % PR) * 1024 + (int)(tid & 63u) * 16;
            if (wv < have * PR && piece < nx * (int)sizeof(TS))
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(xrow + (size_t)(wv / PR) * x_stride) + piece),
                                                 (__attribute__((address_space(3))) void*)(reinterpret_cast<unsigned char*>(outbuf) + (size_t)(wv / PR) * NF * sizeof(TS) + (size_t)(wv % PR) * 1024), 16, 0, 0);
        } else {   // ... of the four in one run, into a place of their own or that of the sums (there, too, a wavefront overwrites
            // only what it alone read: kibibytes v and v + 16)
            const int bytes = nx * Q * (int)sizeof(TS);
            for (int v = (int)(tid >> 6) * 1024; v < bytes; v += NT * 16)
                if (v + (int)(tid & 63u) * 16 < bytes)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(xrow) + v + (tid & 63u) * 16),
                                                     (__attribute__((address_space(3))) void*)(reinterpret_cast<unsigned char*>(xbuf) + v), 16, 0, 0);
        }
        {   // The slices of the instances side by side, through registers: 16 bytes of each, interleaved, Q writes of 16
            // bytes.  (LDS-DMA cannot interleave them but by single words, 13.8 bytes per clock.  Loads of 4 bytes, a label
            // per lane, held the memory pipe for as long as loads of 16.)  For rows of any alignment.
            const size_t rb = (size_t)m * 4;
            const char* r[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) r[q] = grow + (q < have ? q * rb : 0);
#pragma unroll 1
            for (uint32_t o = tid * 16u; o < (uint32_t)nv * 16u; o += NT * 16u) {
                f32x4_any v[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) v[q] = *reinterpret_cast<const f32x4_any*>(r[q] + o);
#pragma unroll
                for (int q = 1; q < Q; ++q)
                    if (have <= q) v[q] = (f32x4_any){0.f, 0.f, 0.f, 0.f};
                if constexpr (Q == 2) {
                    float4* to = reinterpret_cast<float4*>(lds_raw + 2u * o);
                    to[0] = make_float4(v[0].x, v[1].x, v[0].y, v[1].y);
                    to[1] = make_float4(v[0].z, v[1].z, v[0].w, v[1].w);
                } else {
                    float4* to = reinterpret_cast<float4*>(lds_raw + o);
                    to[0] = make_float4(v[0].x, v[1].x, v[2].x, v[3].x);
                    to[quarter] = make_float4(v[0].y, v[1].y, v[2].y, v[3].y);
                    to[2 * quarter] = make_float4(v[0].z, v[1].z, v[2].z, v[3].z);
                    to[3 * quarter] = make_float4(v[0].w, v[1].w, v[2].w, v[3].w);
                }
            }
            if ((int)tid < (nl & 3) * Q) {   // the last labels of a slice that is no multiple of four
                const uint32_t l = (uint32_t)nv * 4 + tid / Q, q = tid % Q;
                reinterpret_cast<float*>(lds_raw)[unit_of_label<Q>(l, (uint32_t)cut.wl) * Q + q] = (int)q < have ? *reinterpret_cast<const float*>(grow + (size_t)q * rb + (size_t)l * 4) : 0.f;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            asm volatile("" : "+v"(token));
        }
        __syncthreads();
        tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        // the activations of the lane's features (Q = 2: of both, before their place is needed for the sums)
        float xa[Q], xb[Q];
        if constexpr (Q == 2) {
            const uint32_t f = feat_of[tid];
            xa[0] = usl_load_f32<TS>(xbuf, (size_t)(f & 0xFFFFu));
            xb[0] = usl_load_f32<TS>(xbuf, (size_t)(f >> 16));
            xa[1] = have > 1 ? usl_load_f32<TS>(xbuf, (size_t)NF + (f & 0xFFFFu)) : 0.f;
            xb[1] = have > 1 ? usl_load_f32<TS>(xbuf, (size_t)NF + (f >> 16)) : 0.f;
        }
        // the earlier windows' sums, on their way during the gathers
        float4 prior[Q / 2];
#pragma unroll
        for (int u = 0; u < Q / 2; ++u) prior[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        // One load per 128-byte line of what the next pass reads: the window's workgroups share the lines of its slices of g, then
        // come the block's own lines of x and those of its earlier sums.  Exactly one in every wavefront (of any line, where
        // there is none to warm up), so that the compiler's wait for `prior`, which is older, can leave it in flight: it comes
        // from memory and takes longer than the gathers (waited for, it cost 130 of 1140 us at m = 500k, d = 32k, k = 32, b = 256).
        {
            constexpr int XR = Q == 4 ? 1 : Q;
            const char* line = grow;
            auto item = [&](int j) {   // (no divisions: every lane comes through here)
                const bool of_g = j < Q * per, of_p = j >= Q * per + XR * xlines;
                const int jj = of_g ? j : of_p ? j - Q * per - XR * xlines : j - Q * per, half = of_g ? per : of_p ? plines : xlines;
                int r = 0;
#pragma unroll
                for (int q = 1; q < Q; ++q) r += jj >= q * half ? 1 : 0;
                const int c = (of_g ? fb * per : 0) + jj - r * half;
                const char* at = (of_g   ? grow + (size_t)m * 4 * (Q + r)
                                  : of_p ? reinterpret_cast<const char*>(dst + (size_t)(Q + r) * dp)
                                         : reinterpret_cast<const char*>(xrow + (Q == 4 ? x_stride : (size_t)(Q + r) * x_stride))) + (size_t)c * 128;
                return i + Q + r < i_end && (!of_g || c < lines) ? at : grow;
            };
            const int items = i + Q < i_end ? Q * per + XR * xlines + Q * plines : 0;
            if (__builtin_amdgcn_readfirstlane((int)tid) < items && (int)tid < items) line = item((int)tid);
            // (the last lines of more than NT, possible where one block is the whole layer, stay cold)
            if (w >= chains) {
                if (Q == 2 || cut.S == 1) {
#pragma unroll
                    for (int u = 0; u < Q / 2; ++u) {
                        const int v = (int)tid + u * NT;
                        if (v < have * (NF / 4) && v % (NF / 4) * 4 < nf)
                            prior[u] = reinterpret_cast<const float4*>(dst + (size_t)(v / (NF / 4)) * dp)[v % (NF / 4)];
                    }
                } else if ((int)tid < d) {
                    float* p = &prior[0].x;
#pragma unroll
                    for (int j = 0; j < Q; ++j)
                        if (j < have) p[j] = dst[(size_t)j * dp + tid];
                }
            }
            token = *reinterpret_cast<const uint32_t*>(line);
        }
        float acc_a[Q] = {}, acc_b[Q] = {};
        int ac = acap, bc = bcap;   // compared afresh in every pass, see k_bwi_lds
        asm volatile("" : "+s"(ac), "+s"(bc));
        if constexpr (Q == 4) unit_of(xbuf + (size_t)(feat_of[(OWN ? NT : 0) + tid] & 0xFFFFu) * 4, xa);
#pragma unroll
        for (int q = 0; q < KT / 4; q += Q == 4 ? 2 : 1) {
            if (q * 4 < ac) {
                if constexpr (Q == 4) gather8(acc_a, gw + q * 4, pk + q * 2, wt + q * 4, gw + q * 4 + 4, pk + q * 2 + 2, wt + q * 4 + 4, xa, ac, q * 4 + 4);
                else gather4_two(acc_a, gw[q * 4], gw[q * 4 + 1], gw[q * 4 + 2], gw[q * 4 + 3], pk[q * 2], pk[q * 2 + 1],
                                 wt[q * 4], wt[q * 4 + 1], wt[q * 4 + 2], wt[q * 4 + 3], xa);
            }
        }
        if constexpr (Q == 4) {   // OWN: the first list's sums leave before the second list begins
            tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            if (ov_n) more(acc_a, ov_share[tid], xa);
            if constexpr (OWN) {
                const uint32_t f = feat_of[tid] & 0xFFFFu;
#pragma unroll
                for (int j = 0; j < Q; ++j) outbuf[j * NF + f] = acc_a[j];
            }
            unit_of(xbuf + (size_t)(feat_of[(OWN ? NT : 0) + tid] >> 16) * 4, xb);
        }
#pragma unroll
        for (int n = 0; n < KT / 4; n += Q == 4 ? 2 : 1) {   // by twos from the list's own end
            const int q = Q == 4 ? KT / 4 - 1 - n : n;
            if (q * 4 >= KT - bc) {
                if constexpr (Q == 4) gather8(acc_b, gw + q * 4, pk + q * 2, wt + q * 4, gw + q * 4 - 4, pk + q * 2 - 2, wt + q * 4 - 4, xb, bc, KT - q * 4 + 3);
                else gather4_two(acc_b, gw[q * 4], gw[q * 4 + 1], gw[q * 4 + 2], gw[q * 4 + 3], pk[q * 2], pk[q * 2 + 1],
                                 wt[q * 4], wt[q * 4 + 1], wt[q * 4 + 2], wt[q * 4 + 3], xb);
            }
        }
        tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        if constexpr (Q == 2) {
            if (ov_n) {   // the same for the whole workgroup: the few lanes whose lists did not fit go on through LDS
                more(acc_a, ov_share[tid], xa);
                more(acc_b, ov_share[tid] >> 16, xb);
            }
            __syncthreads();   // every lane has taken its activations from the place of the sums
            const uint32_t f = feat_of[tid];
            outbuf[f & 0xFFFFu] = acc_a[0];
            outbuf[NF + (f & 0xFFFFu)] = acc_a[1];
            outbuf[f >> 16] = acc_b[0];
            outbuf[NF + (f >> 16)] = acc_b[1];
        } else {
            if (ov_n) more(acc_b, ov_share[tid] >> 16, xb);
            if constexpr (!OWN) __syncthreads();   // every lane has taken its activations from the place of the sums
            const uint32_t f = feat_of[tid];
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                if (!OWN) outbuf[j * NF + (f & 0xFFFFu)] = acc_a[j];
                outbuf[j * NF + (f >> 16)] = acc_b[j];
            }
        }
        if (ov_n > (uint32_t)NEAR2) {   // only a skewed connectivity gets here: what LDS does not hold, by atomics
            __syncthreads();
            for (uint32_t q = NEAR2 + tid; q < ov_n; q += NT) {
                const OvEntry o = ov[(size_t)ov0 + q];
                if (o.slot == PAD_SLOT) continue;
                const float wv = usl_load_f32<TS>(W, (size_t)o.slot);
                float u[Q];
                unit_of(row + (size_t)o.label * Q, u);
                float t = ovgw[(size_t)ov0 + q];
                uint32_t dd = (uint32_t)d;
                asm volatile("" : "+s"(dd));   // (its reciprocal is taken here, not kept in a register)
                const size_t xf = cut.S > 1 ? o.feature % dd : o.feature;
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    unsafeAtomicAdd(&outbuf[j * NF + o.feature], wv * u[j]);
                    if (j < have) t = fmaf(usl_load_f32<TS>(xrow, Q == 4 ? xf * Q + j : (size_t)j * x_stride + xf), u[j], t);
                }
                ovgw[(size_t)ov0 + q] = t;
            }
        }
        __syncthreads();
        if (Q == 2 || cut.S == 1) {   // the block's sums leave as contiguous runs (rows of dp floats, dp a multiple of 4)
#pragma unroll
            for (int u = 0; u < Q / 2; ++u) {
                const int v = (int)tid + u * NT;
                if (v < have * (NF / 4) && v % (NF / 4) * 4 < nf) {
                    const float4 t = reinterpret_cast<const float4*>(outbuf)[v];
                    reinterpret_cast<float4*>(dst + (size_t)(v / (NF / 4)) * dp)[v % (NF / 4)] =
                        make_float4(prior[u].x + t.x, prior[u].y + t.y, prior[u].z + t.z, prior[u].w + t.w);
                }
            }
        } else if ((int)tid < d) {    // ... those of the window's runs added up (d <= NT where there is more than one run)
            const float* p = &prior[0].x;
#pragma unroll
            for (int j = 0; j < Q; ++j)
                if (j < have) {
                    float t = 0.f;
                    for (int r = 0; r < cut.S; ++r) t += outbuf[j * NF + r * d + tid];
                    dst[(size_t)j * dp + tid] = p[j] + t;
                }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("" : "+v"(token));
    // Every slot's sum leaves for its place in stage (rk, ovrk: the workgroup's connections in the order of their
    // flat slots, see k_lf_seg_place), through LDS, which is free now: whole lines.  Written to grad_W[slot] from here
    // they would be 4 bytes each into lines that 16 workgroups share (0.29 ms at m = 500k, a fifth of this kernel); the
    // Adam kernel picks them up through pos instead, and finds neighbours there.  As many places at a time as LDS
    // holds below ov_sum (all of them, unless the connectivity is skewed).
    tid4 = threadIdx.x * 4u;   // taken afresh: addresses are rebuilt from it, not kept (and spilled)
    asm volatile("" : "+v"(tid4));
    float* to = stage + e0;   // (a later pass over the batch adds to the earlier ones)
    uint32_t places[KT / 2];
    if (one_go) load_words<KT>(rk + wg * KT * NT, tid4 / 4, places);
    else own_places(places);
    const uint32_t mine = threadIdx.x < ov_n ? (ovrk + (size_t)ov0)[threadIdx.x] : PAD_SLOT;
    // Behind it: the last pass's reads of LDS, the owners' last additions to ov_sum, and (the wait above) those to ovgw, whose
    // entries are handed out below by other lanes than theirs.
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KT / 4; ++q) {
        if (!used(4 * q)) continue;
#pragma unroll
        for (int t = 4 * q; t < 4 * q + 4; ++t) perm[place_of(places, t)] = gw[t];
    }
    const float near_sum = threadIdx.x < min((uint32_t)NEAR2, ov_n) ? ov_sum[threadIdx.x] : 0.f;
    if (one_go) {
        if (mine != PAD_SLOT) perm[mine] = threadIdx.x < (uint32_t)NEAR2 ? near_sum : ovgw[(size_t)ov0 + threadIdx.x];
        for (uint32_t q = NT + threadIdx.x; q < ov_n; q += NT) {
            const uint32_t place = (ovrk + (size_t)ov0)[q];
            if (place != PAD_SLOT) perm[place] = ovgw[(size_t)ov0 + q];
        }
        __syncthreads();
        for (uint32_t q = threadIdx.x * 4; q < n_ent; q += NT * 4) {
            const float4 v = *reinterpret_cast<const float4*>(perm + q);
            const f32x4_any sum = {v.x, v.y, v.z, v.w};
            if (q + 4 <= n_ent) {
                f32x4_any* at = reinterpret_cast<f32x4_any*>(to + q);
                *at = accumulate ? *at + sum : sum;
            } else {
                for (uint32_t u = 0; q + u < n_ent; ++u) to[q + u] = accumulate ? to[q + u] + sum[u] : sum[u];
            }
        }
    } else {
        auto leave = [&](uint32_t place, float sum) { if (place != PAD_SLOT) to[place] = accumulate ? to[place] + sum : sum; };
#pragma unroll 1
        for (int t = 0; t < KT; ++t)
            if (used(t)) leave((rk + (wg * KT + t) * NT)[threadIdx.x], perm[t * NT + threadIdx.x]);
        leave(mine, threadIdx.x < (uint32_t)NEAR2 ? near_sum : mine != PAD_SLOT ? ovgw[(size_t)ov0 + threadIdx.x] : 0.f);
        for (uint32_t q = NT + threadIdx.x; q < ov_n; q += NT) leave((ovrk + (size_t)ov0)[q], ovgw[(size_t)ov0 + q]);
    }
    }
}

// BOTH only names the kernel after the one whose sums it adds, so that a profile tells the two apart.
template <bool BOTH, int AT_ONCE>
__global__ void __launch_bounds__(256)
k_lf_reduce(usl_window_sums sums, const uint32_t* __restrict__ gate, const uint32_t* __restrict__ stale) {
    if (gate && *gate == 0) return;
    usl_add_up_windows<AT_ONCE>(sums, *stale != 0 /* the lists were built from other contents of idx: no number is better than a wrong one */,
                                blockIdx.x, gridDim.x);
}

}  // namespace

// ---- how a layer is cut up for either form --------------------------------------------------------------------

static Cut bwi_cut(const usl_ctx* c) { return bwi_cut(c->m, c->d, c->k, c->num_cu); }
static int both_q(const usl_ctx* c) { return both_q(c->m, c->d, c->k, c->num_cu); }
static Cut both_cut(const usl_ctx* c) { return both_cut(c->m, c->d, c->k, c->num_cu, both_q(c)); }

// The most that the partial sums of a pass over the batch may take: 16 GiB on a device with 128 GiB or more (every
// pass loads lists and weights anew: at m = 3M, d = 65536, b = 1024 the two products take 74 ms with passes of 4 GiB,
// 62 ms with passes of 16 GiB, 65 ms with one pass of 48 GiB), else 4 GiB.  USL_TUNE_LF_GIB overrides.
static size_t lf_partial_bytes() {
    if (const char* e = getenv("USL_TUNE_LF_GIB")) return (size_t)(atoi(e) > 0 ? atoi(e) : 1) << 30;
    static size_t cached = 0;
    if (!cached) {
        size_t free_b = 0, total_b = 0;
        cached = (hipMemGetInfo(&free_b, &total_b) == hipSuccess && total_b >= ((size_t)128 << 30)) ? (size_t)16 << 30 : (size_t)4 << 30;
    }
    return cached;
}

// where rk begins behind pos: 16-byte pieces
static size_t rk_at(size_t N) { return (N + 3) / 4 * 4; }
// runs of SEG slots in a window of the lists for both products
static int lf_runs(const usl_ctx* c, const Cut& cut) { return (int)(((int64_t)cut.wl * c->k + SEG - 1) / SEG); }

static int padded_d(const usl_ctx* c) { return (c->d + 3) / 4 * 4; }

// Is this layer one for the one-product form?  Lists of about 32 entries per (window, feature) from windows of 16384 to
// 32768 labels (k / d between 1/1024 and 1/512: longer windows do not fit LDS, with shorter ones the partial sums of
// the many windows outweigh the gain), whole feature blocks, 16-byte aligned rows of g, and enough (window, feature
// block) workgroups to fill the chip.  USL_TUNE_BWI=lds forces it where the shape allows at all, =l2 forbids it.
bool usl_bwi_lds_applies(const usl_ctx* c) {
    const int64_t lists = (int64_t)32 * c->d / c->k;   // labels that send that many connections into a feature
    if (!(c->d % NF == 0 && c->d <= 65536 && c->m % 4 == 0 && lists >= 2048 && lists <= WL && c->m * (int64_t)c->k < (int64_t)PAD_SLOT))
        return false;
    if (const char* e = getenv("USL_TUNE_BWI")) {
        if (!strcmp(e, "lds")) return true;
        if (!strcmp(e, "l2")) return false;
    }
    const Cut cut = bwi_cut(c);
    return lists >= 16384 && (int64_t)cut.nwin * cut.nfb * 4 >= (int64_t)c->num_cu * 3;
}

// ... and one for the kernel that computes both backward products from one pass of gathers?
// USL_TUNE_BOTH=on forces it where the shape allows at all, =off forbids it.
bool usl_both_lds_applies(const usl_ctx* c) {
    if (c->d > 65536 || c->m * (int64_t)c->k >= (int64_t)PAD_SLOT || c->no_order) return false;
    const Cut cut = both_cut(c);
    // the partial sums of a pass of 64 instances (the fewest a pass takes) must fit the allowance
    if ((size_t)cut.nwin * 64 * (size_t)padded_d(c) * 4 > lf_partial_bytes()) return false;
    if (const char* e = getenv("USL_TUNE_BOTH")) {
        if (!strcmp(e, "on")) return true;
        if (!strcmp(e, "off")) return false;
    }
    return true;
}

template <int KT>
static usl_status lf_build_t(usl_ctx* c, const int32_t* idx, int set, const Cut& cut) {
    auto& L = c->lf[set];
    const size_t N = (size_t)c->m * c->k;
    const int nwin = cut.nwin, nfb = cut.nfb, nwg = nwin * nfb;
    const size_t nbins = (size_t)nwin * cut.vd;
    const int Q = set == 1 ? both_q(c) : 1;
    {   // all of it in one allocation: thirteen of them were a third of the first call's time on a small layer
        size_t total = 0;
        auto share = [&](auto** to, size_t bytes) {   // twice: first the sizes, then the addresses
            *to = reinterpret_cast<std::remove_reference_t<decltype(*to)>>(static_cast<char*>(L.mem) + total);
            total += (bytes + 255) / 256 * 256;
        };
        for (int turn = 0; turn < 2; ++turn) {
            total = 0;
            share(&L.count, nbins * 4);
            share(&L.where, nbins * 4);
            share(&L.ovoff, nbins * 4);
            share(&L.feat, (size_t)nwg * 2 * NT * 2);
            share(&L.caps, (size_t)nwg * (NT / 64) * 4);
            share(&L.ov_base, ((size_t)nwg * 4 + 2) * 4);
            share(&L.ovr, (size_t)nwg * 2 * NT * 4);
            share(&L.lab, (size_t)nwg * pieces_of<KT>() * NT * 16);
            share(&L.slot, (set == 1 ? N : (size_t)nwg * KT * NT) * 4);   // by place, or by list
            share(&L.ent, N * 4);
            share(&L.ov, (N + nbins) * sizeof(OvEntry));   // worst case, + an empty place per list
            if (set == 1)   // pos [N] (and up to a multiple of 4), rk [nwg][KT][NT], ovrk [N + nbins], the counts of the runs [nwg][nseg]
                share(&L.pos, (rk_at(N) + (size_t)nwg * KT * NT + N + nbins + (size_t)nwg * lf_runs(c, cut)) * 4);
            if (turn == 0) USL_TRY(usl_reserve(c, &L.mem, &L.mem_cap, total));
        }
    }
    const bool own = set == 1 && both_own(Q, cut);
    const uint32_t small_wg = Q == 2 ? both_places<2, false>() : own ? both_places<4, true>() : both_places<4, false>();
    const int rounds = usl_order_rounds(c);
    uint32_t* ov_base = L.ov_base;                   // [nwg + 1]
    uint32_t* n_ov = ov_base + nwg + 1;              // [nwg]
    uint32_t* ent_base = n_ov + nwg;                 // [nwg + 1]
    uint32_t* n_ent = ent_base + nwg + 1;            // [nwg]
    const int nseg = lf_runs(c, cut);
    const int64_t total = (int64_t)nwin * nseg;
    // What only the building needs lies where the overflow entries come last: 8 bytes for every connection.
    uint32_t* slot_at = L.slot;
    uint16_t* feat_at = reinterpret_cast<uint16_t*>(L.ov);
    uint32_t* segcnt = set == 1 ? L.pos + rk_at(N) + (size_t)nwg * KT * NT + N + nbins : nullptr;
    if (set == 0) {
        slot_at = reinterpret_cast<uint32_t*>(feat_at + (N + 1) / 2 * 2);
        segcnt = slot_at + N;   // nwg * nseg words: fewer than N / 2 + nbins
    }
    USL_TRY(usl_idx_print_ready(c));
    const int print = set == 1 ? USL_PRINT_BOTH_PRODUCTS : USL_PRINT_ONE_PRODUCT;
    if (nfb > 1) {
        const dim3 sg((unsigned)((total + 31) / 32 * 8));
        hipLaunchKernelGGL(k_lf_seg_count, sg, dim3(256), 0, c->stream, idx, c->m, c->k, cut, nseg, total, segcnt);
        hipLaunchKernelGGL(k_lf_seg_scan, dim3((unsigned)nwg), dim3(256), 0, c->stream, segcnt, nseg, n_ent);
        hipLaunchKernelGGL(k_lf_scan, dim3(1), dim3(1024), 0, c->stream, n_ent, ent_base, nwg, nullptr, (size_t)0, nullptr, 0);
        hipLaunchKernelGGL(k_lf_seg_place, sg, dim3(256), 0, c->stream, idx, c->m, c->k, cut, nseg, total, segcnt, ent_base,
                           set == 1 ? L.pos : nullptr, slot_at, feat_at);
    }
    LfPlaces places;
    places.idx = idx;
    places.slot_at = slot_at;
    places.feat_at = feat_at;
    places.pos = set == 1 ? L.pos : nullptr;
    places.small_wg = set == 1 ? small_wg : 0;
    // LDS for a quarter more connections than a workgroup has on average, as far as there is room (beside 14 KiB of other things)
    const size_t mean = (size_t)cut.wl * c->k / nfb, want = mean + mean / 4 + 1024;
    places.staged = (int)(want < LF_STAGED ? want : LF_STAGED);
    const size_t lds = (size_t)places.staged * 4;
    USL_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(k_lf_plan<KT>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(k_lf_plan<KT>, dim3((unsigned)nwg), dim3(NT), lds, c->stream, places, c->m, c->k, c->d, cut, ent_base, L.count,
                       L.where, L.ovoff, L.feat, L.caps, n_ov, L.ovr, L.ent);
    hipLaunchKernelGGL(k_lf_scan, dim3(2), dim3(1024), 0, c->stream, n_ov, ov_base, nwg, reinterpret_cast<const uint32_t*>(idx), N,
                       c->idx_print, print);
    const uint32_t zero_label = set == 0 ? ZERO_LABEL : Q == 2 ? BothLayout<2, false>::zero_label : own ? BothLayout<4, true>::zero_label : BothLayout<4, false>::zero_label;
#define USL_LF_SCHED(GS)                                                                                                    \
    hipLaunchKernelGGL((k_lf_schedule<KT, GS>), dim3((unsigned)(nwg * 64 / (SG_NT / 32))), dim3(SG_NT), 0, c->stream, L.ent, \
                       ent_base, L.where, L.count, L.feat, L.caps, ov_base, L.ovoff, c->k, cut, zero_label, rounds,          \
                       L.lab, set == 1 ? nullptr : L.slot, reinterpret_cast<OvEntry*>(L.ov), set == 1 ? L.pos : nullptr, nfb > 1 ? L.slot : nullptr, small_wg,                                 \
                       set == 1 ? L.pos + rk_at(N) : nullptr, set == 1 ? L.pos + rk_at(N) + (size_t)nwg * KT * NT : nullptr)
    if (Q == 4) USL_LF_SCHED(16);
    else USL_LF_SCHED(32);
#undef USL_LF_SCHED
    USL_TRY(usl_check_launch(c, "register lists of the input gradient"));
    L.built_for = idx;
    return USL_OK;
}

// same address as when the lists were built: check that the contents are the same (else grad_x becomes NaN and usl_check
// reports it)
template <int KT>
static usl_status lf_ready(usl_ctx* c, const int32_t* idx, int set, const Cut& cut) {
    if (c->lf[set].built_for != idx) return lf_build_t<KT>(c, idx, set, cut);
    return set == 1 && c->print_done ? USL_OK : usl_idx_fingerprint(c, idx, set == 1 ? USL_PRINT_BOTH_PRODUCTS : USL_PRINT_ONE_PRODUCT, 0);
}

// Instances per pass over the batch: every pass loads the lists and the weights anew, and its partial sums are sets * G * d
// floats; as many as the allowance for partial sums admits, sized once for max_b, a multiple of `step`.
static int pass_rows(const usl_ctx* c, int sets, int step) {
    const size_t most = lf_partial_bytes() / ((size_t)sets * padded_d(c) * 4);
    int G = (int)(most > (size_t)c->max_b ? (size_t)c->max_b : most);
    if (const char* e = getenv("USL_TUNE_BWI_ROWS")) G = atoi(e) < G ? atoi(e) : G;   // tests: several passes on a small layer
    G = G < 64 ? 64 : G;
    G = G > c->max_b ? c->max_b : G;
    // several passes over the batch: only the last has a pass of the loop that is not full
    return G < c->max_b && G > step ? G / step * step : G;
}

// How the sums of `rows` instances are added up: see usl_add_up_windows for the lines.
static usl_window_sums window_sums(const usl_ctx* c, const float* partial, int sets, int rows, float* grad_x) {
    const int dp = padded_d(c);
    const size_t n4 = (size_t)rows * dp / 4, want = (n4 + 255) / 256, most = (size_t)c->num_cu * 8, blocks = want < most ? want : most;
    return {reinterpret_cast<const float4*>(partial), sets, n4, c->d, dp, dp == c->d && (uintptr_t)grad_x % 16 == 0, grad_x,
            (unsigned)((blocks + 7) / 8 * 8), blocks <= (size_t)c->num_cu ? 8 : blocks <= (size_t)c->num_cu * 2 ? 4 : 1};
}

static void lf_reduce(usl_ctx* c, const usl_window_sums& sums, bool both, const uint32_t* gate) {
#define USL_REDUCE(BOTH, AT_ONCE) \
    hipLaunchKernelGGL((k_lf_reduce<BOTH, AT_ONCE>), dim3(sums.blocks), dim3(256), 0, c->stream, sums, gate, usl_stale_word(c))
#define USL_REDUCE_B(BOTH)                                                                                                  \
    do {                                                                                                                    \
        if (sums.at_once == 8) USL_REDUCE(BOTH, 8);                                                                         \
        else if (sums.at_once == 4) USL_REDUCE(BOTH, 4);                                                                    \
        else USL_REDUCE(BOTH, 1);                                                                                           \
    } while (0)
    if (both) USL_REDUCE_B(true); else USL_REDUCE_B(false);
#undef USL_REDUCE_B
#undef USL_REDUCE
}

// The one-product form needs its row buffer at LDS address 0 (a label's byte offset is the address); all need the LDS.
template <typename KERNEL>
static usl_status lf_kernel_ready(usl_ctx* c, KERNEL kern, size_t lds) {
    hipFuncAttributes fa;
    USL_HIP(c, hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kern)));
    if (fa.sharedSizeBytes != 0)
        USL_FAIL(c, USL_EUNSUPPORTED, "backward_input (LDS form): the kernel has static LDS, its row buffer does not start at LDS address 0");
    USL_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    return USL_OK;
}

// grad_x[b][d] from g[b][m] (row-major).  gate as for the other dense kernels.
usl_status usl_bwi_lds_run(usl_ctx* c, const float* g, const int32_t* idx, const void* W, float* grad_x, int32_t b,
                           const uint32_t* gate) {
    auto& L = c->lf[0];
    const Cut cut = bwi_cut(c);
    USL_TRY(lf_ready<KT_BWI>(c, idx, 0, cut));
    const int G = pass_rows(c, cut.nwin, 1);
    USL_TRY(usl_reserve(c, (void**)&L.partial, &L.partial_cap, (size_t)cut.nwin * G * padded_d(c) * 4));
    const unsigned grid = (unsigned)(((cut.nwin + 7) / 8) * 8 * cut.nfb);
    static bool checked[2] = {false, false};
    for (int i0 = 0; i0 < b; i0 += G) {
        const int rows = b - i0 < G ? b - i0 : G;
#define USL_BWI(TS, WHICH)                                                                                                \
        do {                                                                                                              \
            if (!checked[WHICH]) USL_TRY(lf_kernel_ready(c, k_bwi_lds<TS>, LDS_BYTES));                                   \
            checked[WHICH] = true;                                                                                        \
            hipLaunchKernelGGL(k_bwi_lds<TS>, dim3(grid), dim3(NT), LDS_BYTES, c->stream, g + (size_t)i0 * c->m, (const TS*)W, \
                               c->m, c->k, rows, c->d, cut.wl, cut.nfb, cut.nwin, L.lab, L.slot, L.feat, L.caps, L.ov_base, \
                               reinterpret_cast<const OvEntry*>(L.ov), L.ovr, L.partial, gate);                           \
        } while (0)
        if (c->storage == USL_F32) USL_BWI(float, 0);
        else USL_BWI(uint16_t, 1);
#undef USL_BWI
        lf_reduce(c, window_sums(c, L.partial, cut.nwin, rows, grad_x + (size_t)i0 * c->d), false, gate);
    }
    return usl_check_launch(c, "backward_input (LDS form)");
}

// grad_x[b][d] and the weight gradient from g[b][m] and x[b][d].  The weight gradient is left in the order of the lists:
// slot f's is the sum over p < *parts of (*stage)[p * *part_stride + (*pos)[f]] (usl_launch_adam_staged takes it from
// there); both arrays belong to the context and hold until the next call or a change of idx.  The last pass's sums of the input
// gradient are handed over in out->sums: added up beside the weight gradient, not by a launch of their own before it.  A stale idx (see
// usl_check) poisons grad_x; *stale is the device word that says so, for whoever picks up the weight gradient.
usl_status usl_both_lds_run(usl_ctx* c, const float* g, const void* x, const int32_t* idx, const void* W, float* grad_x,
                            int32_t b, const uint32_t* gate, usl_staged* out) {
    auto& L = c->lf[1];
    const Cut cut = both_cut(c);
    const int Q = both_q(c), dp = padded_d(c);
    const size_t N = (size_t)c->m * c->k, nbins = (size_t)cut.nwin * cut.vd, rkn = (size_t)cut.nwin * cut.nfb * (Q == 4 ? KT_BOTH4 : KT_BOTH) * NT;
    if (Q == 4) USL_TRY(lf_ready<KT_BOTH4>(c, idx, 1, cut));
    else USL_TRY(lf_ready<KT_BOTH>(c, idx, 1, cut));
    int forced = 0;   // parts of the batch (tests)
    if (const char* e = getenv("USL_TUNE_BOTH_PARTS")) forced = atoi(e) > 0 ? atoi(e) : 1;
    const int G = pass_rows(c, both_chains(cut, c->num_cu), Q);
    const BothPlan plan = both_plan(cut, c->m, c->k, c->num_cu, b, G, Q, forced);
    const int parts = plan.parts, chains = plan.sets;
    const size_t sum_rows = (size_t)chains * (size_t)(b < G ? b : G);
    if (parts > L.most_parts || sum_rows > L.most_rows) {   // the first call (or another setting of a tuning aid): scratch for every batch that a later call can bring
        const BothMost most = both_most(cut, c->m, c->k, c->num_cu, c->max_b, G, Q, forced);
        if (most.parts > L.most_parts) L.most_parts = most.parts;
        if (most.rows > L.most_rows) L.most_rows = most.rows;
    }
    USL_TRY(usl_reserve(c, (void**)&L.partial, &L.partial_cap, L.most_rows * dp * 4));
    // per part: stage [N], the sums of the overflow entries beyond LDS [N + nbins]
    const size_t keep = (size_t)L.most_parts;
    USL_TRY(usl_reserve(c, (void**)&L.stage, &L.stage_cap, keep * (N + N + nbins) * 4));
    float* ovgw = L.stage + keep * N;
    const void* xs = nullptr;
    size_t x_stride = 0;
    USL_TRY(usl_activation_rows(c, x, b, Q == 4 ? 4 : 1, &xs, &x_stride));
    out->stale = usl_stale_word(c);
    out->sums.blocks = 0;
    const bool direct = chains == 1 && dp == c->d && (uintptr_t)grad_x % 16 == 0;   // nothing to add up
    static bool checked[6] = {false, false, false, false, false, false};
    const bool own = both_own(Q, cut);
    for (int i0 = 0; i0 < b; i0 += G) {
        const int rows = b - i0 < G ? b - i0 : G;
        const int per_part = ((rows + parts - 1) / parts + Q - 1) / Q * Q;
        // whole windows to an XCD where that leaves no XCD more rounds (of 32 compute units) than even shares
        const int64_t even = ((int64_t)chains * parts * cut.nfb + 7) / 8, whole = ((int64_t)chains * parts + 7) / 8 * cut.nfb;
        const dim3 grid((unsigned)(8 * ((whole + 31) / 32 == (even + 31) / 32 ? whole : even)));
#define USL_BOTH(TS, QQ, OWN, WHICH)                                                                                             \
        do {                                                                                                                \
            if (!checked[WHICH]) USL_TRY(lf_kernel_ready(c, k_both_lds<TS, QQ, OWN>, both_lds_bytes<QQ, OWN>()));                      \
            checked[WHICH] = true;                                                                                          \
            hipLaunchKernelGGL((k_both_lds<TS, QQ, OWN>), grid, dim3(NT), (both_lds_bytes<QQ, OWN>()), c->stream, g + (size_t)i0 * c->m, \
                               (const TS*)W, (const TS*)xs + (size_t)(QQ == 4 ? i0 / 4 : i0) * x_stride, x_stride, c->m, c->k, rows, c->d, \
                               dp, cut, L.lab, L.slot, L.feat, L.caps, L.ov_base, reinterpret_cast<const OvEntry*>(L.ov), L.ovr, \
                               direct ? grad_x + (size_t)i0 * c->d : L.partial, L.pos + rk_at(N), L.pos + rk_at(N) + rkn, L.ov_base + 2 * ((size_t)cut.nwin * cut.nfb) + 1, L.stage, \
                               ovgw, chains, parts, per_part, N, N + nbins, gate, i0 > 0 ? 1 : 0, direct ? out->stale : nullptr);                                         \
        } while (0)
        if (c->storage == USL_F32) { if (Q == 2) USL_BOTH(float, 2, false, 0); else if (own) USL_BOTH(float, 4, true, 1); else USL_BOTH(float, 4, false, 2); }
        else { if (Q == 2) USL_BOTH(uint16_t, 2, false, 3); else if (own) USL_BOTH(uint16_t, 4, true, 4); else USL_BOTH(uint16_t, 4, false, 5); }
#undef USL_BOTH
        if (direct) continue;
        const usl_window_sums sums = window_sums(c, L.partial, chains, rows, grad_x + (size_t)i0 * c->d);
        if (i0 + G < b) lf_reduce(c, sums, true, gate);   // the next pass takes the place of these
        else out->sums = sums;
    }
    out->stage = L.stage;
    out->pos = L.pos;
    out->parts = parts;
    out->part_stride = N;
    return usl_check_launch(c, "backward products (LDS form)");
}
