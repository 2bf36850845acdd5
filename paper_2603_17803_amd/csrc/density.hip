// Co-activation density and medoid queue (Section 5.1: co-activation probability of Step 1, distance
// of Step 2, density and descending medoid queue of Algorithm 1's Step 3), one streaming pass over the
// count matrix per quantity.
//
//   total  = sum of all C[k][l];  P(i,j) = C[i][j] / total;  d(i,j) = 1 - P(i,j)   (fp64)
//   rho[i] = number of j with d(i,j) <= tau
// d is a non-increasing function of the integer count (one correctly rounded division, one
// subtraction), so "d <= tau" is "count >= c*" for a single integer c* per head.  c* is found by
// a search with exactly the fp64 expression above; the pass over C is then an integer
// compare-and-count at memory speed, and takes the same decisions as evaluating d per element.
#include "common.h"
#include "wave_ops.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

typedef int v4i_row __attribute__((ext_vector_type(4), aligned(4)));    // rows of C are 4-byte aligned when N is odd; 16-byte loads need no more

constexpr int ROWS_PER_BLOCK = 4;        // one wave per row of C

__global__ void totals_init_kernel(int64_t* __restrict__ totals, const int64_t* __restrict__ totals_in, int H) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h < H) totals[h] = totals_in ? totals_in[h] : 0;
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;                               // valid in lane 0
}

// Calls f(count) for every element of a row, 16-byte loads four deep.  Both sweeps of C are bound by memory, and a wave
// with a single load in flight (or with 4-byte loads, which rows of odd length used to take) leaves half of it unused:
// 8 x 6001 x 6001 counts took 337 us summed and 352 us compared, against 167 us for their bytes.
template <typename F>
__device__ __forceinline__ void for_each_count(const int32_t* __restrict__ r, int N, int lane, F f) {
    const int n4 = N >> 2;
    auto at = [&](int i) __attribute__((always_inline)) { return (v4i)__builtin_nontemporal_load(reinterpret_cast<const v4i_row*>(r) + i); };
    int i = lane;
    for (; i + 192 < n4; i += 256) {
        const v4i a = at(i), b = at(i + 64), c = at(i + 128), d = at(i + 192);
        f(a.x); f(a.y); f(a.z); f(a.w); f(b.x); f(b.y); f(b.z); f(b.w);
        f(c.x); f(c.y); f(c.z); f(c.w); f(d.x); f(d.y); f(d.z); f(d.w);
    }
    for (; i < n4; i += 64) {
        const v4i a = at(i);
        f(a.x); f(a.y); f(a.z); f(a.w);
    }
    if (lane < (N & 3)) f(r[4 * n4 + lane]);
}

// grand total per head: every wave sums rows, the workgroup adds one partial total to the head's total
// (few atomics per address: thousands of them on eight addresses cost more than the sweep itself)
__global__ __launch_bounds__(256) void row_total_kernel(const int32_t* __restrict__ C, int N, int64_t* __restrict__ totals) {
    __shared__ int64_t part[ROWS_PER_BLOCK];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = blockIdx.y;
    int64_t s = 0;
    for (int row = blockIdx.x * ROWS_PER_BLOCK + wave; row < N; row += gridDim.x * ROWS_PER_BLOCK)
        for_each_count(C + ((size_t)h * N + row) * N, N, lane, [&](int32_t v) __attribute__((always_inline)) { s += v; });
    s = wave_sum_i64(s);
    if (lane == 0) part[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
#pragma unroll
        for (int w = 0; w < ROWS_PER_BLOCK; ++w) t += part[w];
        atomicAdd(reinterpret_cast<unsigned long long*>(totals + h), (unsigned long long)t);
    }
}

// Smallest count c in [0, 2^31) whose distance passes the radius test; 2^31 when none does.  All 64 lanes of a wave call
// this together: each round tests 64 candidates at once, six rounds where a bisection takes 31 divisions one after the
// other (every workgroup of the sweep over C needs the threshold before its first comparison).
__device__ __forceinline__ int64_t count_threshold(int64_t total, double tau, bool strict) {
    constexpr int64_t NONE = (int64_t)1 << 31;
    if (total == 0) return NONE;                         // P undefined: no pair counts
    const double t = (double)total;
    const int lane = threadIdx.x & 63;
    int64_t lo = 0;                                      // the answer lies in [lo, lo + 64 * width]
#pragma unroll
    for (int shift = 30; shift >= 0; shift -= 6) {
        const int64_t width = (int64_t)1 << shift;
        const int64_t c = lo + (int64_t)(lane + 1) * width - 1;          // the last count of this lane's interval
        const double d = 1.0 - (double)c / t;
        const uint64_t pass = __ballot(strict ? d < tau : d <= tau);     // d falls as c grows: once a lane passes, all later ones do
        if (!pass) return NONE;                          // only in the first round, whose intervals cover [0, 2^36)
        lo += (int64_t)(__ffsll((unsigned long long)pass) - 1) * width;
    }
    return lo < NONE ? lo : NONE;
}

__global__ __launch_bounds__(256) void density_count_kernel(const int32_t* __restrict__ C, int N, const int64_t* __restrict__ totals,
                                                            double tau, uint32_t flags, int32_t* __restrict__ rho) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = blockIdx.y;
    const int64_t cstar = count_threshold(totals[h], tau, flags & SWARM_RHO_STRICT);
    for (int row = blockIdx.x * ROWS_PER_BLOCK + wave; row < N; row += gridDim.x * ROWS_PER_BLOCK) {
        const int32_t* r = C + ((size_t)h * N + row) * N;
        int32_t count = 0;
        if (cstar <= 0x7fffffffll) {
            const int32_t c32 = (int32_t)cstar;
            for_each_count(r, N, lane, [&](int32_t v) __attribute__((always_inline)) { count += v >= c32; });
            if ((flags & SWARM_RHO_EXCLUDE_SELF) && lane == 0) count -= r[row] >= c32;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) count += __shfl_down(count, off, 64);
        if (lane == 0) rho[(size_t)h * N + row] = count;
    }
}

// Grand total of A^T A per head straight from the trace, and the threshold that goes with it, for a
// build that counts the density in its own epilogue: total = sum over trace rows of the square of the
// row's number of activated entries (each of a row's activated pairs adds one to C).
__global__ __launch_bounds__(1024) void trace_total_threshold_kernel(const int32_t* __restrict__ row_count, int slabs, int nrows, double tau,
                                                                     uint32_t flags, int64_t* __restrict__ totals,
                                                                     int64_t* __restrict__ cstar) {
    __shared__ int64_t part[16];
    const int h = blockIdx.x;
    const size_t slab = (size_t)gridDim.x * nrows;
    int64_t sum = 0;
    for (int r = threadIdx.x; r < nrows; r += 1024) {
        const int32_t* c = row_count + (size_t)h * nrows + r;
        int64_t n = 0;
#pragma unroll 8
        for (int s = 0; s < slabs; ++s) n += c[s * slab];
        sum += n * n;
    }
    sum = wave_sum_i64(sum);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x < 64) {
        int64_t total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) total += part[w];
        const int64_t c = count_threshold(total, tau, flags & SWARM_RHO_STRICT);
        if (threadIdx.x == 0) { totals[h] = total; cstar[h] = c; }
    }
}

// j = i left out of the density: one less where the diagonal element itself reaches the threshold
__global__ void rho_exclude_self_kernel(const int32_t* __restrict__ C, int N, const int64_t* __restrict__ cstar, int32_t* __restrict__ rho) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, h = blockIdx.y;
    if (i >= N) return;
    if ((int64_t)C[((size_t)h * N + i) * N + i] >= cstar[h]) rho[(size_t)h * N + i] -= 1;
}

// The queue without scratch (a capture that finds none and a device without the room, for more entries than one workgroup
// sorts): position of entry i = entries with a higher density + entries with the same density and a lower id: N^2
// comparisons per head, tiled through LDS.  A workgroup ranks 256 entries;
// its four quarters (256 threads each) take a quarter of every staged tile of 1024 densities, and the
// partial ranks meet in LDS: four times the waves per compute unit of one thread per entry.
constexpr int RANK_ENTRIES = 256, RANK_PARTS = 4, RANK_TILE = 1024;

__global__ __launch_bounds__(RANK_ENTRIES * RANK_PARTS) void medoid_rank_kernel(const int32_t* __restrict__ rho, int N,
                                                                                  int32_t* __restrict__ queue) {
    __shared__ int32_t tile[RANK_TILE];
    __shared__ int32_t partial[RANK_PARTS - 1][RANK_ENTRIES];
    const int h = blockIdx.y;
    const int32_t* rh = rho + (size_t)h * N;
    const int e = threadIdx.x % RANK_ENTRIES, part = threadIdx.x / RANK_ENTRIES;
    const int i = blockIdx.x * RANK_ENTRIES + e;
    const int32_t mine = i < N ? rh[i] : 0;
    constexpr int SUB = RANK_TILE / RANK_PARTS;
    int32_t rank = 0;
    for (int j0 = 0; j0 < N; j0 += RANK_TILE) {
        __syncthreads();
        tile[threadIdx.x] = (j0 + (int)threadIdx.x < N) ? rh[j0 + threadIdx.x] : -1;
        __syncthreads();
        // this quarter's slice [s0, s0 + lim) of the tile; entries below i win ties, entries above lose them:
        // count (rho_j >= mine) for j < i and (rho_j > mine) for j > i, split at j = i
        const int s0 = part * SUB;
        const int lim = max(0, min(SUB, N - j0 - s0));
        const int below = max(0, min(lim, i - j0 - s0));
        const int32_t* t = tile + s0;
#pragma unroll 8
        for (int u = 0; u < below; ++u) rank += t[u] >= mine;
#pragma unroll 8
        for (int u = below; u < lim; ++u) rank += t[u] > mine;
    }
    if (part > 0) partial[part - 1][e] = rank;
    __syncthreads();
    if (part == 0 && i < N) {
#pragma unroll
        for (int p = 0; p < RANK_PARTS - 1; ++p) rank += partial[p][e];
        queue[(size_t)h * N + rank] = i;
    }
}

// The same order as a stable radix sort of the ids by N - rho, ascending: comparing all pairs grows with N^2 (one
// head of 65536 entries 352 us), two passes over the ids are four short launches (34 us; 18 of them a move that waits for its counts).
// A pass moves the ids only and looks their densities up; digits of at most 9 bits, so up to 2^18 entries take two passes.
// One workgroup per SORT_BLOCK places of the list, each wave a contiguous part of it.
constexpr int SORT_THREADS = 256, SORT_STEPS = 8, SORT_BLOCK = SORT_THREADS * SORT_STEPS, SORT_BITS = 9;

// The entry at place p of the list (src null: the list is in ascending id) and its digit; -1 past the end.
__device__ __forceinline__ int sort_digit(const int32_t* __restrict__ rho, const int32_t* __restrict__ src, int N, int p, int shift, int mask, int& id) {
    id = p < N ? (src ? src[p] : p) : 0;
    return p < N ? ((N - rho[id]) >> shift) & mask : -1;
}

__global__ __launch_bounds__(SORT_THREADS) void rank_count_kernel(const int32_t* __restrict__ rho, const int32_t* __restrict__ src, int N, int shift, int bits,
                                                                  uint32_t* __restrict__ counts) {
    __shared__ uint32_t hist[1 << SORT_BITS];
    const int bins = 1 << bits, h = blockIdx.y;
    for (int d = threadIdx.x; d < bins; d += SORT_THREADS) hist[d] = 0u;
    __syncthreads();
    const int32_t *rh = rho + (size_t)h * N, *sh = src ? src + (size_t)h * N : nullptr;
#pragma unroll
    for (int s = 0; s < SORT_STEPS; ++s) {
        int id;
        const int d = sort_digit(rh, sh, N, blockIdx.x * SORT_BLOCK + s * SORT_THREADS + threadIdx.x, shift, bins - 1, id);
        if (d >= 0) atomicAdd(&hist[d], 1u);
    }
    __syncthreads();
    uint32_t* out = counts + ((size_t)h * gridDim.x + blockIdx.x) * bins;
    for (int d = threadIdx.x; d < bins; d += SORT_THREADS) out[d] = hist[d];
}

// Lanes of the wave with the same digit (`on` lanes only), a ballot per digit bit.
__device__ __forceinline__ uint64_t same_digit(int digit, bool on, int bits) {
    uint64_t same = __ballot(on);
    for (int b = 0; b < bits; ++b) {
        const bool bit = (digit >> b) & 1;
        const uint64_t with = __ballot(bit);
        same &= bit ? with : ~with;
    }
    return same;
}

// How many entries of the wave with its digit come before this one: those of earlier steps, which `seen` (the wave's own) counts per
// digit, and those on lower lanes.  A counter is added to by one lane of each digit: equal densities are the rule, and an atomic per
// lane would queue on their counter.
__device__ __forceinline__ uint32_t rank_in_wave(int digit, bool on, int bits, uint32_t* seen) {
    const uint64_t same = same_digit(digit, on, bits);
    const uint32_t below = (uint32_t)__popcll(same & ((1ull << (threadIdx.x & 63)) - 1ull));
    uint32_t r = 0;
    if (on) {
        r = seen[digit];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (below == 0) seen[digit] = r + (uint32_t)__popcll(same);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return r + below;
}

// Where a digit's entries of this workgroup go: behind all smaller digits and the same digit of the workgroups before, whose counts
// every workgroup adds up for itself.
__global__ __launch_bounds__(SORT_THREADS) void rank_move_kernel(const int32_t* __restrict__ rho, const int32_t* __restrict__ src, int N, int shift, int bits,
                                                                 const uint32_t* __restrict__ counts, int32_t* __restrict__ dst) {
    constexpr int WAVES = SORT_THREADS / 64, PER = (1 << SORT_BITS) / SORT_THREADS;
    __shared__ uint32_t at[WAVES][1 << SORT_BITS], wave_total[WAVES];
    const int bins = 1 << bits, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t *rh = rho + (size_t)h * N, *sh = src ? src + (size_t)h * N : nullptr;
    int id[SORT_STEPS], digit[SORT_STEPS];
#pragma unroll
    for (int s = 0; s < SORT_STEPS; ++s)
        digit[s] = sort_digit(rh, sh, N, blockIdx.x * SORT_BLOCK + (wave * SORT_STEPS + s) * 64 + lane, shift, bins - 1, id[s]);
    // PER consecutive digits per thread
    uint32_t all[PER], before[PER], sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        all[u] = before[u] = 0u;
        const int d = tid * PER + u;
        if (d < bins) {
            const uint32_t* c = counts + (size_t)h * gridDim.x * bins + d;
#pragma unroll 8
            for (uint32_t b = 0; b < gridDim.x; ++b) {
                const uint32_t n = c[(size_t)b * bins];
                all[u] += n;
                before[u] += b < blockIdx.x ? n : 0u;
            }
        }
        sum += all[u];
    }
    for (int d = lane; d < bins; d += 64) at[wave][d] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t place[SORT_STEPS];
#pragma unroll
    for (int s = 0; s < SORT_STEPS; ++s) place[s] = rank_in_wave(digit[s], digit[s] >= 0, bits, at[wave]);
    uint32_t total;
    uint32_t first = waveops::wave_excl_scan(sum, &total);
    if (lane == 0) wave_total[wave] = total;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) first += w < wave ? wave_total[w] : 0u;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int d = tid * PER + u;
        if (d < bins) {
            uint32_t p = first + before[u];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t n = at[w][d];
                at[w][d] = p;
                p += n;
            }
        }
        first += all[u];
    }
    __syncthreads();
    int32_t* out = dst + (size_t)h * N;
#pragma unroll
    for (int s = 0; s < SORT_STEPS; ++s)
        if (digit[s] >= 0) {
            const uint32_t p = at[wave][digit[s]] + place[s];
            if (p < (uint32_t)N) out[p] = id[s];                       // always holds
        }
}

// A head that fits one workgroup is sorted in LDS, all passes in one launch: key << 13 | id per entry, 7 bits a pass.  8 heads of
// 6001 entries 13 us (all pairs 36, the four launches above 30); the density calls of 1000 to 8192 entries lost 4 to 35 us.
constexpr int SMALL_MAX = 8192, SMALL_THREADS = 1024, SMALL_BITS = 7;

template <int STEPS>
__global__ __launch_bounds__(SMALL_THREADS) void rank_small_kernel(const int32_t* __restrict__ rho, int N, int passes, int32_t* __restrict__ queue) {
    constexpr int WAVES = SMALL_THREADS / 64, BINS = 1 << SMALL_BITS;
    __shared__ uint32_t list[STEPS * SMALL_THREADS], at[WAVES][BINS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t* rh = rho + (size_t)blockIdx.x * N;
    const int p0 = wave * STEPS * 64 + lane;
    uint32_t x[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const int i = p0 + s * 64;
        x[s] = i < N ? (uint32_t)(N - rh[i]) << 13 | (uint32_t)i : 0u;
    }
    for (int pass = 0; pass < passes; ++pass) {
#pragma unroll
        for (int u = 0; u < BINS / 64; ++u) at[wave][u * 64 + lane] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32_t place[STEPS];
        int digit[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            digit[s] = (int)(x[s] >> (13 + pass * SMALL_BITS)) & (BINS - 1);
            place[s] = rank_in_wave(digit[s], p0 + s * 64 < N, SMALL_BITS, at[wave]);
        }
        __syncthreads();
        if (wave == 0) {                                      // two digits per lane: the waves' counts become their first places
            uint32_t n[2][WAVES], sum[2] = {0u, 0u};
#pragma unroll
            for (int w = 0; w < WAVES; ++w)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    n[u][w] = at[w][2 * lane + u];
                    sum[u] += n[u][w];
                }
            uint32_t total;
            uint32_t p = waveops::wave_excl_scan(sum[0] + sum[1], &total);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < WAVES; ++w) {
                    at[w][2 * lane + u] = p;
                    p += n[u][w];
                }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (p0 + s * 64 < N) {
                const uint32_t p = at[wave][digit[s]] + place[s];
                if (p < (uint32_t)N) list[p] = x[s];                   // always holds
            }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < STEPS; ++s) x[s] = p0 + s * 64 < N ? list[p0 + s * 64] : 0u;
    }
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
        if (p0 + s * 64 < N) queue[(size_t)blockIdx.x * N + p0 + s * 64] = (int32_t)(x[s] & 8191u);
}

}  // namespace

swarm_status launch_density(swarm_ctx* ctx, const int32_t* C, int H, int N, const int64_t* totals_in, double tau,
                            uint32_t flags, int32_t* rho, int32_t* queue, int64_t* totals) {
    hipLaunchKernelGGL(totals_init_kernel, dim3((unsigned)((H + 63) / 64)), dim3(64), 0, ctx->stream, totals, totals_in, H);
    swarm_status st = swarm_check_launch(ctx, "totals_init_kernel");
    if (st != SWARM_OK) return st;
    // both sweeps stride over the rows with at most 512 workgroups per head: enough to fill the device, few enough that
    // the totals' atomics and the search for the threshold do not count
    const unsigned nblk = (unsigned)((N + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK);
    const dim3 grid(nblk < 512u ? nblk : 512u, (unsigned)H);
    if (!totals_in) {
        hipLaunchKernelGGL(row_total_kernel, grid, dim3(256), 0, ctx->stream, C, N, totals);
        st = swarm_check_launch(ctx, "row_total_kernel");
        if (st != SWARM_OK) return st;
    }
    hipLaunchKernelGGL(density_count_kernel, grid, dim3(256), 0, ctx->stream, C, N, totals, tau, flags, rho);
    st = swarm_check_launch(ctx, "density_count_kernel");
    if (st != SWARM_OK || !queue) return st;
    return launch_medoid_rank(ctx, rho, H, N, queue);
}

// Scratch of the sort: a list of ids and, per workgroup, the digits' counts.
static size_t rank_scratch_words(int H, int N) {
    return (size_t)H * N + (((size_t)H * ((N + SORT_BLOCK - 1) / SORT_BLOCK)) << SORT_BITS);
}

swarm_status launch_medoid_rank(swarm_ctx* ctx, const int32_t* rho, int H, int N, int32_t* queue) {
    int width = 1;                                            // bits of the largest key, N
    while (N >> width) ++width;
    if (N <= SMALL_MAX) {
        const int passes = (width + SMALL_BITS - 1) / SMALL_BITS;
        using kernel_t = void (*)(const int32_t*, int, int, int32_t*);
        const kernel_t kernel = N <= SMALL_THREADS ? rank_small_kernel<1> : N <= 2 * SMALL_THREADS ? rank_small_kernel<2>
                              : N <= 4 * SMALL_THREADS ? rank_small_kernel<4> : rank_small_kernel<8>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)H), dim3(SMALL_THREADS), 0, ctx->stream, rho, N, passes, queue);
        ctx->queue_way = SWARM_WAY_QUEUE_LDS;
        return swarm_check_launch(ctx, "rank_small_kernel");
    }
    bool sorted;
    const swarm_status st = swarm_try_grow(ctx, reinterpret_cast<void**>(&ctx->rank), &ctx->rank_bytes, rank_scratch_words(H, N) * 4, &sorted);
    if (st != SWARM_OK) return st;
    if (!sorted) {
        hipLaunchKernelGGL(medoid_rank_kernel, dim3((unsigned)((N + RANK_ENTRIES - 1) / RANK_ENTRIES), (unsigned)H),
                           dim3(RANK_ENTRIES * RANK_PARTS), 0, ctx->stream, rho, N, queue);
        ctx->queue_way = SWARM_WAY_QUEUE_COMPARED;
        return swarm_check_launch(ctx, "medoid_rank_kernel");
    }
    int32_t* ids = ctx->rank;
    uint32_t* counts = reinterpret_cast<uint32_t*>(ctx->rank + (size_t)H * N);
    const int passes = (width + SORT_BITS - 1) / SORT_BITS, bits = (width + passes - 1) / passes;
    const dim3 grid((unsigned)((N + SORT_BLOCK - 1) / SORT_BLOCK), (unsigned)H);
    const int32_t* src = nullptr;
    for (int p = 0; p < passes; ++p) {
        int32_t* dst = (passes - 1 - p) % 2 ? ids : queue;    // the last pass writes the queue
        hipLaunchKernelGGL(rank_count_kernel, grid, dim3(SORT_THREADS), 0, ctx->stream, rho, src, N, p * bits, bits, counts);
        hipLaunchKernelGGL(rank_move_kernel, grid, dim3(SORT_THREADS), 0, ctx->stream, rho, src, N, p * bits, bits, counts, dst);
        src = dst;
    }
    ctx->queue_way = SWARM_WAY_QUEUE_SORTED;
    return swarm_check_launch(ctx, "rank_move_kernel");
}

swarm_status launch_trace_totals_thresholds(swarm_ctx* ctx, const int32_t* row_count, int slabs, int H, int nrows, double tau, uint32_t flags,
                                            int64_t* totals, int64_t* cstar) {
    hipLaunchKernelGGL(trace_total_threshold_kernel, dim3((unsigned)H), dim3(1024), 0, ctx->stream, row_count, slabs, nrows, tau, flags,
                       totals, cstar);
    return swarm_check_launch(ctx, "trace_total_threshold_kernel");
}

swarm_status launch_rho_exclude_self(swarm_ctx* ctx, const int32_t* C, int H, int N, const int64_t* cstar, int32_t* rho) {
    hipLaunchKernelGGL(rho_exclude_self_kernel, dim3((unsigned)((N + 255) / 256), (unsigned)H), dim3(256), 0, ctx->stream, C, N, cstar,
                       rho);
    return swarm_check_launch(ctx, "rho_exclude_self_kernel");
}
