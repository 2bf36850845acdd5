// Medoid-indexed retrieval helpers around the mapping step (Section 5.2, Tier 1, and Section 6.1):
//   cluster expansion -- the clusters activated through their medoids are merged (each once, ascending
//   id) and replaced by their member entries, the input of the entry-level mapping step;
//   submission order  -- the buckets built by the mapping step are drained head by head: batch b is the
//   b-th item of every bucket that has one, in ascending SSD id.
#include <type_traits>

#include "common.h"
#include "wave_ops.h"

namespace {

using waveops::wave_excl_scan;

constexpr int EXP_THREADS = 256;

// One workgroup per group, whatever the number of activated clusters: the picks set bits, the bits are walked in order by the
// threads that own them and every cluster's entries are copied by one thread, a memory round trip per entry.  For groups of
// more picks than the listed form below keeps in LDS.
// LDS: bitmap of activated clusters (Nc bits) + one partial sum per thread.
__global__ __launch_bounds__(EXP_THREADS) void expand_clusters_kernel(const int32_t* __restrict__ clusters, int Sc, int H, int Nc,
                                                                      const int32_t* __restrict__ cl_off,
                                                                      const int32_t* __restrict__ cl_entries, int E,
                                                                      int32_t* __restrict__ entries, int32_t* __restrict__ count,
                                                                      int cap_e, uint32_t* __restrict__ dev_flags) {
    extern __shared__ uint32_t smem[];
    const int nwords = (Nc + 31) / 32;
    uint32_t* bitmap = smem;
    uint32_t* wave_tot = smem + nwords;            // EXP_THREADS / 64 words
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t g = blockIdx.x;
    const int h = (int)(g % H);
    uint32_t flags = 0;
    for (int w = tid; w < nwords; w += EXP_THREADS) bitmap[w] = 0;
    __syncthreads();
    for (int s = tid; s < Sc; s += EXP_THREADS) {
        const int32_t c = clusters[g * Sc + s];
        if (c == -1) continue;
        if (c < 0 || c >= Nc) { flags |= SWARM_DEV_BAD_CLUSTER; continue; }
        atomicOr(&bitmap[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    // thread t owns a contiguous run of bitmap words, so that thread order is cluster order
    const int wpt = (nwords + EXP_THREADS - 1) / EXP_THREADS;
    const int w0 = min(tid * wpt, nwords), w1 = min(w0 + wpt, nwords);
    const int32_t* off = cl_off + (size_t)h * (Nc + 1);
    uint32_t mine = 0;
    for (int w = w0; w < w1; ++w) {
        uint32_t bits = bitmap[w];
        while (bits) {
            const int c = w * 32 + __ffs(bits) - 1;
            bits &= bits - 1;
            const int32_t lo = off[c], hi = off[c + 1];
            if (lo < 0 || hi < lo || hi > E) { flags |= SWARM_DEV_BAD_CLUSTER; continue; }
            mine += (uint32_t)(hi - lo);
        }
    }
    uint32_t wtot;
    uint32_t pos = wave_excl_scan(mine, &wtot);
    if (lane == 0) wave_tot[wave] = wtot;
    __syncthreads();
    uint32_t total = 0;
    for (int w = 0; w < EXP_THREADS / 64; ++w) {
        if (w < wave) pos += wave_tot[w];
        total += wave_tot[w];
    }
    const int32_t* ent = cl_entries + (size_t)h * E;
    int32_t* out = entries + g * cap_e;
    for (int w = w0; w < w1; ++w) {
        uint32_t bits = bitmap[w];
        while (bits) {
            const int c = w * 32 + __ffs(bits) - 1;
            bits &= bits - 1;
            const int32_t lo = off[c], hi = off[c + 1];
            if (lo < 0 || hi < lo || hi > E) continue;
            for (int32_t p = lo; p < hi; ++p, ++pos)
                if (pos < (uint32_t)cap_e) out[pos] = ent[p];
        }
    }
    if (total > (uint32_t)cap_e) { flags |= SWARM_DEV_CAP; total = cap_e; }
    if (tid == 0) count[g] = (int32_t)total;
    for (uint32_t p = total + tid; p < (uint32_t)cap_e; p += EXP_THREADS) out[p] = -1;
    if (flags) atomicOr(dev_flags, flags);
}

// The same for 65 to EXP_LIST picks per group.  What bounds it is the chain of dependent steps of a workgroup that
// is alone on its compute unit, so each step is one for all clusters: the place of an activated cluster among them comes from
// the popcounts below it (every pick computes it, equal picks write the same slot), all offset pairs are read together, their
// lengths scanned, and the entries are copied position by position, each finding its cluster by bisection.
// 8 x 32 of 1024 clusters into 512 entries: 13.7 -> 6.3 us (a chain of up to 16 loads per cluster before).
constexpr int EXP_LIST = 2048;
constexpr int EXP_PER = EXP_LIST / EXP_THREADS;

__global__ __launch_bounds__(EXP_THREADS) void expand_listed_kernel(const int32_t* __restrict__ clusters, int Sc, int H, int Nc,
                                                                    const int32_t* __restrict__ cl_off,
                                                                    const int32_t* __restrict__ cl_entries, int E,
                                                                    int32_t* __restrict__ entries, int32_t* __restrict__ count,
                                                                    int cap_e, uint32_t* __restrict__ dev_flags) {
    extern __shared__ uint32_t smem[];
    const int nwords = (Nc + 31) / 32;
    const int nlist = min(Sc, EXP_LIST);
    uint32_t* bitmap = smem;                       // nwords
    uint32_t* run_base = bitmap + nwords;          // activated clusters before each thread's run of words: EXP_THREADS
    uint32_t* list = run_base + EXP_THREADS;       // activated clusters, ascending, then the first entry of each: nlist
    uint32_t* start = list + nlist;                // first output position of each: nlist
    uint32_t* wave_tot = start + nlist;            // EXP_THREADS / 64
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t g = blockIdx.x;
    const int h = (int)(g % H);
    uint32_t flags = 0;

    int32_t pick[EXP_PER];
#pragma unroll
    for (int u = 0; u < EXP_PER; ++u) pick[u] = u * EXP_THREADS < Sc ? clusters[g * Sc + min(tid + u * EXP_THREADS, Sc - 1)] : -1;
    for (int w = tid; w < nwords; w += EXP_THREADS) bitmap[w] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < EXP_PER; ++u) {
        const bool ok = (uint32_t)pick[u] < (uint32_t)Nc;
        flags |= (!ok && pick[u] != -1) ? SWARM_DEV_BAD_CLUSTER : 0u;
        if (ok) atomicOr(&bitmap[pick[u] >> 5], 1u << (pick[u] & 31));
        else pick[u] = -1;
    }
    __syncthreads();

    auto block_excl_scan = [&](uint32_t v, uint32_t* total) __attribute__((always_inline)) {
        uint32_t wtot;
        uint32_t before = wave_excl_scan(v, &wtot);
        if (lane == 0) wave_tot[wave] = wtot;
        __syncthreads();
        uint32_t all = 0;
#pragma unroll
        for (int w = 0; w < EXP_THREADS / 64; ++w) {
            before += w < wave ? wave_tot[w] : 0u;
            all += wave_tot[w];
        }
        *total = all;
        return before;
    };
    const int wpt = (nwords + EXP_THREADS - 1) / EXP_THREADS;      // words of a thread's run
    const int w0 = min(tid * wpt, nwords), w1 = min(w0 + wpt, nwords);
    uint32_t mine = 0;
    for (int w = w0; w < w1; ++w) mine += (uint32_t)__popc(bitmap[w]);
    uint32_t m;
    run_base[tid] = block_excl_scan(mine, &m);                     // m <= min(Sc, Nc): distinct picks
    __syncthreads();
#pragma unroll
    for (int u = 0; u < EXP_PER; ++u) {
        if (pick[u] < 0) continue;
        const int w = pick[u] >> 5, run = w / wpt;
        uint32_t at = run_base[run];
        for (int v = run * wpt; v < w; ++v) at += (uint32_t)__popc(bitmap[v]);
        at += (uint32_t)__popc(bitmap[w] & ((1u << (pick[u] & 31)) - 1u));
        list[at] = (uint32_t)pick[u];
    }
    __syncthreads();

    // thread t owns the listed clusters [t * per, +per): their offset pairs all at once, then the running lengths
    const int per = (nlist + EXP_THREADS - 1) / EXP_THREADS;
    const int32_t* off = cl_off + (size_t)h * (Nc + 1);
    int32_t lo[EXP_PER], hi[EXP_PER];
#pragma unroll
    for (int u = 0; u < EXP_PER; ++u) {
        const uint32_t i = (uint32_t)(tid * per + u);
        const bool in = u < per && i < m;
        const uint32_t c = in ? list[i] : 0u;
        lo[u] = in ? off[c] : 0;
        hi[u] = in ? off[c + 1] : 0;
    }
    uint32_t len = 0;
#pragma unroll
    for (int u = 0; u < EXP_PER; ++u) {
        if (lo[u] < 0 || hi[u] < lo[u] || hi[u] > E) { flags |= SWARM_DEV_BAD_CLUSTER; hi[u] = lo[u]; }
        len += (uint32_t)(hi[u] - lo[u]);
    }
    uint32_t total;
    uint32_t pos = block_excl_scan(len, &total);
#pragma unroll
    for (int u = 0; u < EXP_PER; ++u) {
        const uint32_t i = (uint32_t)(tid * per + u);
        if (u < per && i < m) {
            list[i] = (uint32_t)lo[u];
            start[i] = pos;
        }
        pos += (uint32_t)(hi[u] - lo[u]);
    }
    __syncthreads();

    if (total > (uint32_t)cap_e) { flags |= SWARM_DEV_CAP; total = (uint32_t)cap_e; }
    const int32_t* ent = cl_entries + (size_t)h * E;
    int32_t* out = entries + g * cap_e;
    const int top = m > 1 ? 31 - __clz((int)(m - 1)) : -1;          // highest bit of the last list position
    constexpr int AHEAD = 4;
    for (uint32_t p0 = tid; p0 < total; p0 += AHEAD * EXP_THREADS) {
        uint32_t at[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) at[u] = 0;
        // the last cluster that starts at or before the position (an empty one shares its successor's start)
        for (int b = top; b >= 0; --b) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const uint32_t probe = at[u] | (1u << b);
                if (probe < m && start[probe] <= p0 + u * EXP_THREADS) at[u] = probe;
            }
        }
        int32_t v[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const uint32_t p = p0 + u * EXP_THREADS;
            v[u] = p < total ? ent[list[at[u]] + (p - start[at[u]])] : 0;
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
            if (p0 + u * EXP_THREADS < total) out[p0 + u * EXP_THREADS] = v[u];
    }
    if (tid == 0) count[g] = (int32_t)total;
    for (uint32_t p = total + tid; p < (uint32_t)cap_e; p += EXP_THREADS) out[p] = -1;
    if (flags) atomicOr(dev_flags, flags);
}

// The same for up to 64 picks, one per lane: every wave finds out for itself where each activated cluster goes, so that no
// barrier and no bitmap is left.  Picks that come in ascending order, as a selection lists them, need a scan of their lengths;
// others are ranked against each other through the wave's lists.  NT: one wave per group where the groups alone fill the device,
// four for the copying where they do not.
// 8 groups of 32 of 1024 clusters into up to 512 entries: 5.5 us by the listed form, 3.9 us (ascending) and 4.7 us; 4096 groups
// of 16, clusters of up to 8: 15.4, 4.6 and 5.5 us (11.1 us as one thread per run of clusters, the form above all of these).
constexpr int EXP_FEW = 64;

template <int NT>
__global__ __launch_bounds__(NT) void expand_few_kernel(const int32_t* __restrict__ clusters, int Sc, int H, int Nc,
                                                        const int32_t* __restrict__ cl_off, const int32_t* __restrict__ cl_entries, int E,
                                                        int32_t* __restrict__ entries, int32_t* __restrict__ count, int cap_e,
                                                        uint32_t* __restrict__ dev_flags) {
    __shared__ __attribute__((aligned(16))) int32_t s_first[NT / 64][EXP_FEW];      // first entry of each activated cluster, ascending cluster id
    __shared__ __attribute__((aligned(16))) uint32_t s_start[NT / 64][EXP_FEW];     // and its first output position
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t g = blockIdx.x;
    const int h = (int)(g % H);
    int32_t* first = s_first[wave];
    uint32_t* start = s_start[wave];

    const int32_t pick = lane < Sc ? clusters[g * Sc + lane] : -1;
    const bool ok = (uint32_t)pick < (uint32_t)Nc;
    uint32_t flags = (!ok && pick != -1) ? SWARM_DEV_BAD_CLUSTER : 0u;
    const int32_t* off = cl_off + (size_t)h * (Nc + 1) + (ok ? pick : 0);
    const int32_t lo = off[0];
    int32_t hi = off[1];
    constexpr int32_t BEHIND = 0x7fffffff;                   // every cluster
    int32_t c = ok ? pick : BEHIND;
    const int32_t prev = __shfl_up(c, 1, 64);
    const bool sorted = __ballot(lane > 0 && ok && prev >= c) == 0;
    if (!sorted) {                                           // of equal picks the first
        first[lane] = c;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        bool again = false;
        for (int j0 = 0; j0 < Sc; j0 += 16) {                // reads past Sc stay within the list and meet BEHIND
#pragma unroll
            for (int j = j0; j < j0 + 16; j += 4) {
                const int4 o = *reinterpret_cast<const int4*>(first + j);
                again |= (o.x == c && j < lane) | (o.y == c && j + 1 < lane) | (o.z == c && j + 2 < lane) | (o.w == c && j + 3 < lane);
            }
        }
        if (again) c = BEHIND;
    }
    const bool use = c != BEHIND;
    const bool sound = lo >= 0 && hi >= lo && hi <= E;
    if (use && !sound) flags |= SWARM_DEV_BAD_CLUSTER;
    if (!use || !sound) hi = lo;
    const uint32_t len = (uint32_t)(hi - lo);
    uint32_t total, rank = (uint32_t)lane;                   // in order the valid picks come first
    uint32_t at = wave_excl_scan(len, &total);
    const uint32_t m = (uint32_t)__popcll(__ballot(use));
    if (!sorted) {
        first[lane] = c;
        start[lane] = len;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        rank = at = 0;
        for (int j0 = 0; j0 < Sc; j0 += 16) {
#pragma unroll
            for (int j = j0; j < j0 + 16; j += 4) {
                const int4 o = *reinterpret_cast<const int4*>(first + j);
                const uint4 n = *reinterpret_cast<const uint4*>(start + j);
                rank += (o.x < c) + (o.y < c) + (o.z < c) + (o.w < c);
                at += (o.x < c ? n.x : 0u) + (o.y < c ? n.y : 0u) + (o.z < c ? n.z : 0u) + (o.w < c ? n.w : 0u);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (use) { first[rank] = lo; start[rank] = at; }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's own lists: it alone reads them

    if (total > (uint32_t)cap_e) { flags |= SWARM_DEV_CAP; total = (uint32_t)cap_e; }
    const int32_t* ent = cl_entries + (size_t)h * E;
    int32_t* out = entries + g * cap_e;
    auto copy = [&](auto ahead_tag) __attribute__((always_inline)) {
        constexpr int AHEAD = decltype(ahead_tag)::value;    // positions in flight per thread
        for (uint32_t p0 = tid; p0 < total; p0 += AHEAD * NT) {
            uint32_t i[AHEAD];                               // the last cluster that starts at or before a position
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) i[u] = 0;
#pragma unroll
            for (uint32_t b = EXP_FEW / 2; b; b >>= 1) {
                if (b >= m) continue;
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const uint32_t probe = i[u] | b;
                    if (probe < m && start[probe] <= p0 + u * NT) i[u] = probe;
                }
            }
            int32_t v[AHEAD];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const uint32_t p = p0 + u * NT;
                v[u] = p < total ? ent[first[i[u]] + (int32_t)(p - start[i[u]])] : 0;
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u)
                if (p0 + u * NT < total) out[p0 + u * NT] = v[u];
        }
    };
    if (total <= NT) copy(std::integral_constant<int, 1>{});
    else copy(std::integral_constant<int, 4>{});
    if (tid == 0) count[g] = (int32_t)total;
    for (uint32_t p = total + tid; p < (uint32_t)cap_e; p += NT) out[p] = -1;
    if (wave == 0 && flags) atomicOr(dev_flags, flags);
}

// One workgroup per group, one thread per routed item: the item at position pos of bucket d goes to
// rank = sum over buckets of min(length, pos) + number of lower-numbered buckets longer than pos.
__global__ __launch_bounds__(256) void submission_order_kernel(const int32_t* __restrict__ q_off, const int32_t* __restrict__ q_cluster,
                                                               int D, int cap, int32_t* __restrict__ order,
                                                               int32_t* __restrict__ batch_off, int32_t* __restrict__ nb,
                                                               uint32_t* __restrict__ dev_flags) {
    __shared__ int32_t off[65];
    const int64_t g = blockIdx.x;
    for (int d = threadIdx.x; d <= D; d += 256) off[d] = q_off[g * (D + 1) + d];
    __syncthreads();
    // offsets that are not a non-decreasing sequence from 0 to at most cap would send ranks out of range:
    // such a group gets an empty order and a flag (every thread takes the same decision)
    bool bad = off[0] != 0 || off[D] > cap;
    for (int e = 0; e < D; ++e) bad |= off[e + 1] < off[e];
    if (bad) {
        for (int32_t p = threadIdx.x; p < cap; p += 256) order[g * cap + p] = -1;
        for (int32_t b = threadIdx.x; b <= cap; b += 256) batch_off[g * (cap + 1) + b] = 0;
        if (threadIdx.x == 0) { nb[g] = 0; atomicOr(dev_flags, SWARM_DEV_BAD_OFFSETS); }
        return;
    }
    const int32_t total = off[D];
    for (int32_t p = threadIdx.x; p < cap; p += 256) {
        if (p >= total) { order[g * cap + p] = -1; continue; }
        int d = 0;
        while (d + 1 < D && off[d + 1] <= p) ++d;
        const int32_t pos = p - off[d];
        int32_t rank = 0;
        for (int e = 0; e < D; ++e) {
            const int32_t len = off[e + 1] - off[e];
            rank += min(len, pos) + ((e < d && len > pos) ? 1 : 0);
        }
        order[g * cap + rank] = q_cluster[g * cap + p];
    }
    int32_t longest = 0;
    for (int e = 0; e < D; ++e) longest = max(longest, off[e + 1] - off[e]);
    for (int32_t b = threadIdx.x; b <= cap; b += 256) {
        int32_t start = 0;
        for (int e = 0; e < D; ++e) start += min(off[e + 1] - off[e], b);
        batch_off[g * (cap + 1) + b] = min(start, total);
    }
    if (threadIdx.x == 0) nb[g] = longest;
}

}  // namespace

swarm_status launch_expand_clusters(swarm_ctx* ctx, const int32_t* clusters, int64_t groups, int Sc, int H, int Nc,
                                    const int32_t* cl_off, const int32_t* cl_entries, int E, int32_t* entries, int32_t* count,
                                    int cap_e) {
    if (Sc <= EXP_FEW) {
        const bool many = groups >= (cap_e > 512 ? 2048 : 1024);     // four to a compute unit, more where there is more to copy
        hipLaunchKernelGGL((many ? expand_few_kernel<64> : expand_few_kernel<EXP_THREADS>), dim3((unsigned)groups), dim3(many ? 64 : EXP_THREADS), 0,
                           ctx->stream, clusters, Sc, H, Nc, cl_off, cl_entries, E, entries, count, cap_e, ctx->dev_flags);
        return swarm_check_launch(ctx, "expand_few_kernel");
    }
    if (Sc <= EXP_LIST) {                          // bitmap and list stay below 64 KiB of LDS at the largest Nc
        const size_t lds = ((size_t)(Nc + 31) / 32 + EXP_THREADS + 2 * (size_t)Sc + EXP_THREADS / 64) * 4;
        hipLaunchKernelGGL(expand_listed_kernel, dim3((unsigned)groups), dim3(EXP_THREADS), lds, ctx->stream, clusters, Sc, H, Nc,
                           cl_off, cl_entries, E, entries, count, cap_e, ctx->dev_flags);
        return swarm_check_launch(ctx, "expand_listed_kernel");
    }
    const size_t lds = ((size_t)(Nc + 31) / 32 + EXP_THREADS / 64) * 4;
    hipLaunchKernelGGL(expand_clusters_kernel, dim3((unsigned)groups), dim3(EXP_THREADS), lds, ctx->stream, clusters, Sc, H, Nc,
                       cl_off, cl_entries, E, entries, count, cap_e, ctx->dev_flags);
    return swarm_check_launch(ctx, "expand_clusters_kernel");
}

swarm_status launch_submission_order(swarm_ctx* ctx, const int32_t* q_off, const int32_t* q_cluster, int64_t groups, int D, int cap,
                                     int32_t* order, int32_t* batch_off, int32_t* nb) {
    hipLaunchKernelGGL(submission_order_kernel, dim3((unsigned)groups), dim3(256), 0, ctx->stream, q_off, q_cluster, D, cap, order,
                       batch_off, nb, ctx->dev_flags);
    return swarm_check_launch(ctx, "submission_order_kernel");
}
