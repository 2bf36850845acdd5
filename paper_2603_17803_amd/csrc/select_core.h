// Block-level exact top-k selection on register-resident scores (device code, gfx950).
//
// Selection step (Section 2.3): the k highest scores of a row, equal scores won by the lower
// index, result in ascending index order.
//
// A block of 1024 threads holds the row as IPT consecutive scores per thread.  One pass bins every score *linearly in value*
// between the row's minimum and maximum into 2048 LDS counters (clamping, subtraction, scaling and truncation are all
// monotone, so bin order agrees with score order); a scan finds the bin b* that holds the k-th
// largest score.  Bins above b* are selected outright; inside b* (a handful of scores for any
// smooth distribution) the exact threshold key T and the number of entries equal to T that still
// belong to the result are found by ranking the candidates against each other, or -- when b*
// holds more candidates than the ranking buffer, e.g. under massive ties -- by an exact 4 x 8-bit
// radix select restricted to b*.  A final ordered compaction (block prefix scan over the
// contiguous per-thread chunks) writes the indices in ascending order, which also makes the
// lowest-index tie-break deterministic.
//
// A row is one block's work and a block has one compute unit, so what bounds this is instructions per score (four waves per
// SIMD take 16 cycles for each).  The scores therefore stay floats -- five instructions to bin one -- and only those of b*
// are mapped to order-preserving 32-bit keys; what is above b* and what is inside is kept as two bit masks per thread.
// (Every score carried as a key, mapped and mapped back for binning: 5.3 instead of 4.9 us for 32 rows of 4001 scores.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave_ops.h"

namespace selcore {

using waveops::wave_incl_scan;

constexpr int NT = 1024;        // threads per selecting block (default form)
constexpr int NB = 2048;        // value bins
constexpr int CMAX = 1024;      // candidates ranked pairwise

template <int NTH = NT>
struct SmemT {
    static constexpr int NW = NTH / 64;
    uint32_t hist[NB];
    __attribute__((aligned(16))) uint32_t cand[CMAX];
    uint32_t wave_a[16], wave_b[16];
    __attribute__((aligned(16))) uint32_t wave_kmax[16];
    __attribute__((aligned(16))) uint32_t wave_kmin[16];
    uint32_t cand_count, bstar, above, thr_key, thr_need;
    uint32_t digit, digit_above;
};
using Smem = SmemT<NT>;

// Monotone map fp32 -> uint32: larger float <=> larger key.  -0 maps to the key of +0; every
// NaN maps to key 0, below -inf.
__device__ __forceinline__ uint32_t order_key(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Scores are clamped to +-VMAX for binning, so that a difference of two is finite; what the clamp merges (infinities, NaN with
// -inf) shares a bin and is told apart by key.
constexpr float VMAX = 1.5e38f;
__device__ __forceinline__ float bin_value(float x) { return __builtin_amdgcn_fmed3f(x, -VMAX, VMAX); }     // a NaN becomes -VMAX

__device__ __forceinline__ int bin_of(float x, float hi, float scale) {
    return (int)fminf((hi - bin_value(x)) * scale, (float)(NB - 1));      // hi - v >= 0: non-increasing in the score
}

// Monotone unsigned image of a float that is not NaN, and its inverse.
__device__ __forceinline__ uint32_t plain_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float plain_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : ~key);
}

// Exclusive block scan of two counters at once.  The wave totals (at most 16) are scanned by every wave on its own (lane l
// reads total l % 16, four DPP steps inside the row of 16 lanes) instead of being read and conditionally added one by one.
template <int NTH>
__device__ __forceinline__ void block_excl_scan2(uint32_t a, uint32_t b, uint32_t& ea, uint32_t& eb, SmemT<NTH>& sm,
                                                 int lane, int wave) {
    constexpr int NW = NTH / 64;
    static_assert(NW >= 1 && NW <= 16, "one wave total per lane of a DPP row");
    const uint32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
    if (lane == 63) { sm.wave_a[wave] = ia; sm.wave_b[wave] = ib; }
    __syncthreads();
    uint32_t ta = (lane & 15) < NW ? sm.wave_a[lane & 15] : 0u, tb = (lane & 15) < NW ? sm.wave_b[lane & 15] : 0u;
    ta += waveops::dpp_or_zero<0x111, 0xF>(ta);  tb += waveops::dpp_or_zero<0x111, 0xF>(tb);     // row_shr:1
    ta += waveops::dpp_or_zero<0x112, 0xF>(ta);  tb += waveops::dpp_or_zero<0x112, 0xF>(tb);     // row_shr:2
    if (NW > 4) { ta += waveops::dpp_or_zero<0x114, 0xF>(ta);  tb += waveops::dpp_or_zero<0x114, 0xF>(tb); }    // row_shr:4
    if (NW > 8) { ta += waveops::dpp_or_zero<0x118, 0xF>(ta);  tb += waveops::dpp_or_zero<0x118, 0xF>(tb); }    // row_shr:8: totals of waves 0..l
    const int prev = wave > 0 ? wave - 1 : 0;
    const uint32_t pa = (uint32_t)__builtin_amdgcn_readlane((int)ta, prev), pb = (uint32_t)__builtin_amdgcn_readlane((int)tb, prev);
    ea = ia - a + (wave > 0 ? pa : 0u);
    eb = ib - b + (wave > 0 ? pb : 0u);
}

// x[e] is the score of index tid*IPT + e; slots at or beyond N must hold NaN, which ranks below every score.
// All NTH threads of the block must call this.  emit(pos, e) is called once for each of the k selected entries, by the thread
// that holds it: pos is its place in the result (ascending index order), e its slot in the thread's run.  STATIC_E: emit
// uses e to index registers, so the slots are walked unrolled; otherwise only the set ones are.
// meanwhile() is called by every thread after the histogram (what it loaded beside the row has had the time for that to
// arrive): what it writes to LDS is visible to every emit().
template <int IPT, int NTH = NT, bool STATIC_E = false, typename Emit, typename Meanwhile>
__device__ __forceinline__ void block_select(const float (&x)[IPT], int N, int k, SmemT<NTH>& sm, Emit emit, Meanwhile meanwhile) {
    constexpr int NW = NTH / 64;
    constexpr bool KEEP = IPT <= 32;                    // bins kept in registers between the histogram and the masks, not computed again
    constexpr int NBINS_KEPT = KEEP ? IPT : 1;
    constexpr int NM = (IPT + 31) / 32;                 // mask words per thread
    constexpr int MB = IPT < 32 ? IPT : 32;             // slots per mask word
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int base = tid * IPT;

    // row extrema of the binning value, from the slots that hold an entry
    float vmax = -VMAX, vmin = VMAX;
    if (base + IPT <= N) {
#pragma unroll
        for (int e = 0; e < IPT; ++e) {
            const float v = bin_value(x[e]);
            vmax = fmaxf(vmax, v);
            vmin = fminf(vmin, v);
        }
    } else {
#pragma unroll
        for (int e = 0; e < IPT; ++e) {
            const float v = bin_value(x[e]);
            vmax = fmaxf(vmax, v);                      // NaN slots cannot raise it
            vmin = fminf(vmin, base + e < N ? v : VMAX);
        }
    }
    uint32_t kmax = ~waveops::wave_min_u32(~plain_key(vmax));
    uint32_t kmin = waveops::wave_min_u32(plain_key(vmin));
    if (lane == 0) { sm.wave_kmax[wave] = kmax; sm.wave_kmin[wave] = kmin; }
#pragma unroll
    for (int i = 0; i < NB / NTH; ++i) sm.hist[tid + i * NTH] = 0;
#pragma unroll
    for (int i = 0; i < CMAX / NTH; ++i) sm.cand[tid + i * NTH] = 0;
    if (tid == 0) { sm.cand_count = 0; sm.thr_key = 0; sm.thr_need = 0xffffffffu; }
    __syncthreads();
    {
        const uint4* pmax = reinterpret_cast<const uint4*>(sm.wave_kmax);
        const uint4* pmin = reinterpret_cast<const uint4*>(sm.wave_kmin);
#pragma unroll
        for (int w = 0; w < (NW + 3) / 4; ++w) {
            const uint4 a = pmax[w], b = pmin[w];
            if (4 * w + 0 < NW) { kmax = max(kmax, a.x); kmin = min(kmin, b.x); }
            if (4 * w + 1 < NW) { kmax = max(kmax, a.y); kmin = min(kmin, b.y); }
            if (4 * w + 2 < NW) { kmax = max(kmax, a.z); kmin = min(kmin, b.z); }
            if (4 * w + 3 < NW) { kmax = max(kmax, a.w); kmin = min(kmin, b.w); }
        }
    }
    // an empty row (N = 0) leaves hi < lo, and the scale becomes 0
    const float hi = plain_value(kmax), lo = plain_value(kmin);
    const float range = hi - lo;
    const float scale = range > 0.f ? fminf((float)NB / range, 1.0e30f) : 0.f;

    // value histogram
    int bin[NBINS_KEPT];
    auto bin_at = [&](int e) __attribute__((always_inline)) { return KEEP ? bin[e] : bin_of(x[e], hi, scale); };
#pragma unroll
    for (int e = 0; e < IPT; ++e) {
        const int b = bin_of(x[e], hi, scale);
        if (KEEP) bin[e] = b;
        atomicAdd(&sm.hist[b], 1u);
    }
    meanwhile();
    __syncthreads();

    // bin b* holding the k-th largest: cumulative count from bin 0 (highest scores) first reaches k
    {
        constexpr int PER = NB / NTH;                   // consecutive bins per thread
        uint32_t hh[PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) { hh[i] = sm.hist[PER * tid + i]; sum += hh[i]; }
        uint32_t before, unused;
        block_excl_scan2<NTH>(sum, 0u, before, unused, sm, lane, wave);
        if (before < (uint32_t)k && (uint32_t)k <= before + sum) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (before < (uint32_t)k && (uint32_t)k <= before + hh[i]) { sm.bstar = PER * tid + i; sm.above = before; }
                before += hh[i];
            }
        }
    }
    __syncthreads();
    const int bstar = (int)sm.bstar;
    const uint32_t need = (uint32_t)k - sm.above;       // entries of bin b* that belong to the result
    const uint32_t c = sm.hist[bstar];

    // bit e of a word: slot e (+ 32 per word) lies above b* / inside it; a sign bit is shifted in per slot
    uint32_t take[NM], inside[NM], some_inside = 0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        uint32_t above = 0, upto = 0;
#pragma unroll
        for (int e = MB - 1; e >= 0; --e) {
            const int b = bin_at(m * 32 + e);
            above = __builtin_amdgcn_alignbit(above, (uint32_t)(b - bstar), 31);
            upto = __builtin_amdgcn_alignbit(upto, (uint32_t)(b - bstar - 1), 31);
        }
        take[m] = above;
        inside[m] = upto & ~above;
        some_inside |= inside[m];
    }

    if (need < c) {
        if (__builtin_expect(c <= (uint32_t)CMAX, 1)) {           // the massive-tie path is laid out off the straight line
            // rank the candidates of b* against each other
            if (some_inside) {
#pragma unroll
                for (int e = 0; e < IPT; ++e)
                    if ((inside[e / 32] >> (e & 31)) & 1u) sm.cand[atomicAdd(&sm.cand_count, 1u)] = order_key(x[e]);
            }
            __syncthreads();
            for (uint32_t t = tid; t < c; t += NTH) {
                const uint32_t mine = sm.cand[t];
                uint32_t gt = 0, eq = 0;
                // four at a time; the zeros behind the last one can only look equal to a zero, the lowest key, for which
                // gt + eq reaches `need` anyway
                for (uint32_t j = 0; j < c; j += 4) {
                    const uint4 other = *reinterpret_cast<const uint4*>(&sm.cand[j]);
                    gt += (other.x > mine) + (other.y > mine) + (other.z > mine) + (other.w > mine);
                    eq += (other.x == mine) + (other.y == mine) + (other.z == mine) + (other.w == mine);
                }
                if (gt < need && need <= gt + eq) { sm.thr_key = mine; sm.thr_need = need - gt; }
            }
            __syncthreads();
        } else {
            // exact radix select restricted to bin b* (hist[0..256) reused as digit counters)
            uint32_t prefix = 0, mask = 0, rem = need;
            for (int shift = 24; shift >= 0; shift -= 8) {
                __syncthreads();
                if (tid < 256) sm.hist[tid] = 0;
                __syncthreads();
#pragma unroll
                for (int e = 0; e < IPT; ++e) {
                    const uint32_t key = order_key(x[e]);
                    if (((inside[e / 32] >> (e & 31)) & 1u) && (key & mask) == prefix) atomicAdd(&sm.hist[(key >> shift) & 255u], 1u);
                }
                __syncthreads();
                if (wave == 0) {
                    const uint32_t h0 = sm.hist[4 * lane], h1 = sm.hist[4 * lane + 1], h2 = sm.hist[4 * lane + 2],
                                   h3 = sm.hist[4 * lane + 3];
                    const uint32_t tot = h0 + h1 + h2 + h3;
                    uint32_t incl = tot;
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const uint32_t v = __shfl_down(incl, off, 64);
                        if (lane + off < 64) incl += v;
                    }
                    uint32_t above = incl - tot;
                    const uint32_t hh[4] = {h0, h1, h2, h3};
#pragma unroll
                    for (int j = 3; j >= 0; --j) {
                        if (above < rem && rem <= above + hh[j]) { sm.digit = 4 * lane + j; sm.digit_above = above; }
                        above += hh[j];
                    }
                }
                __syncthreads();
                prefix |= sm.digit << shift;
                mask |= 0xffu << shift;
                rem -= sm.digit_above;
            }
            __syncthreads();
            if (tid == 0) { sm.thr_key = prefix; sm.thr_need = rem; }
            __syncthreads();
        }
    }
    const uint32_t T = sm.thr_key, need_eq = sm.thr_need;   // need == c: T = 0, every candidate is taken

    // ordered compaction.  A score is taken outright when it lies in a bin above b*, or in b* above the threshold key;
    // scores equal to the threshold key are taken in index order until need_eq of them are in.
    uint32_t same[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) same[m] = 0;
    if (some_inside) {
#pragma unroll
        for (int e = 0; e < IPT; ++e) {
            if ((inside[e / 32] >> (e & 31)) & 1u) {
                const uint32_t key = order_key(x[e]);
                take[e / 32] |= (uint32_t)(key > T) << (e & 31);
                same[e / 32] |= (uint32_t)(key == T) << (e & 31);
            }
        }
    }
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int m = 0; m < NM; ++m) { gt += __popc(take[m]); eq += __popc(same[m]); }
    uint32_t gt_before, eq_before;
    block_excl_scan2<NTH>(gt, eq, gt_before, eq_before, sm, lane, wave);
    uint32_t pos = gt_before + min(eq_before, need_eq);
    // the equal scores this thread still takes: its first (need_eq - eq_before) of them
    uint32_t room = need_eq > eq_before ? need_eq - eq_before : 0u;
#pragma unroll
    for (int m = 0; m < NM; ++m)
        for (; room && same[m]; --room) { take[m] |= same[m] & (0u - same[m]); same[m] &= same[m] - 1u; }
    if constexpr (STATIC_E) {
#pragma unroll
        for (int e = 0; e < IPT; ++e) {
            if ((take[e / 32] >> (e & 31)) & 1u) {
                if (pos < (uint32_t)k) emit(pos, e);                       // pos < k always holds; the guard keeps a slip in bounds
                ++pos;
            }
        }
    } else {
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            while (take[m]) {
                const int e = m * 32 + __ffs(take[m]) - 1;
                take[m] &= take[m] - 1u;
                if (pos < (uint32_t)k) emit(pos, e);
                ++pos;
            }
        }
    }
}

typedef float f32x4_row __attribute__((ext_vector_type(4), aligned(4)));    // rows of scores are 4-byte aligned; 16-byte loads need no more

// Loads IPT consecutive scores of a row (NaN in the slots beyond N).
template <int IPT>
__device__ __forceinline__ void load_scores(const float* __restrict__ row, int N, float (&x)[IPT]) {
    const int base = threadIdx.x * IPT;
    if (base + IPT <= N) {
#pragma unroll
        for (int e = 0; e < IPT / 4; ++e) {
            const f32x4_row v = reinterpret_cast<const f32x4_row*>(row + base)[e];
            x[4 * e] = v.x;
            x[4 * e + 1] = v.y;
            x[4 * e + 2] = v.z;
            x[4 * e + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < IPT; ++e) x[e] = (base + e < N) ? row[base + e] : __uint_as_float(0x7fc00000u);
    }
}

// The ids of a thread's IPT consecutive winners of M; slots beyond M repeat the last one.  (One by one, at a stride of IPT words
// between lanes, they cost a cache line per lane and load: 8 us for the 8192 winners of a 65536-entry row.)
typedef int i32x4_row __attribute__((ext_vector_type(4), aligned(4)));
template <int IPT>
__device__ __forceinline__ void load_winner_ids(const int32_t* __restrict__ ids, int M, int32_t (&id)[IPT]) {
    const int base = threadIdx.x * IPT;
    if (base + IPT <= M) {
#pragma unroll
        for (int e = 0; e < IPT / 4; ++e) {
            const i32x4_row v = reinterpret_cast<const i32x4_row*>(ids + base)[e];
            id[4 * e] = v.x;
            id[4 * e + 1] = v.y;
            id[4 * e + 2] = v.z;
            id[4 * e + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < IPT; ++e) id[e] = ids[min(base + e, M - 1)];
    }
}

// Loads the scores of a thread's IPT consecutive winners (of M, listed in ascending entry id).  kept: their scores as the
// slices wrote them beside the ids; without room for those (nullptr) they are gathered from the row.  Every load is clamped
// to a valid position instead of being branched around, so that all of a thread's loads are in flight together: behind a
// branch each, the eight of a 65536-entry row's second stage were eight pairs of dependent round trips, 12 of its 23 us.
template <int IPT>
__device__ __forceinline__ void load_winners(const float* __restrict__ row, const int32_t* __restrict__ ids,
                                             const float* __restrict__ kept, int M, float (&x)[IPT]) {
    if (kept) {
        load_scores<IPT>(kept, M, x);
        return;
    }
    const int base = threadIdx.x * IPT;
    int32_t id[IPT];
    load_winner_ids<IPT>(ids, M, id);
#pragma unroll
    for (int e = 0; e < IPT; ++e) x[e] = row[id[e]];
#pragma unroll
    for (int e = 0; e < IPT; ++e) x[e] = base + e < M ? x[e] : __uint_as_float(0x7fc00000u);
}

}  // namespace selcore
