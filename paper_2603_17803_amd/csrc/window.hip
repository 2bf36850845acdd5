// Cluster maintenance over the local window (Section 6.2): for every newly generated entry e and every
// cluster medoid m_i, f(e, m_i) = number of the window's W steps in which both are activated,
// d = 1 - f / W (fp64), and e joins every cluster with d < tau; a joining entry goes to the cluster's
// next SSD, (id_i + |C_i| + 1) mod D, with |C_i| growing as entries join in the order given.
//
// f is a thin (new entries x medoids) slice of the window's A^T A.  The window's trace is built as
// bits (the same builder as for the full co-activation matrix), so a count is a handful of
// AND + popcount operations on the two entries' 16-byte words.
#include <type_traits>

#include "common.h"

namespace {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int WIN_MAX_RUNS = 16;      // window length up to 2048 steps held in registers
constexpr int WIN_PER_SEG = 8;            // new entries of a run and pass

// A workgroup owns 32 clusters of a head and walks all new entries, 2 NW runs of up to 8 of them at a time: lane l of a wave
// holds the trace words of medoid l % 32 in registers, its half of the wave takes one run, the words of a new entry are the
// same for the whole half (one broadcast load each).  A new entry's place depends on how many entries before it joined the
// cluster: each half wave counts the joiners of its run, the counts meet in LDS and every half adds up those before it.
// So membership, counts and places leave in one pass.  Before, one thread per cluster walked the entries in order in a
// kernel of its own, a load latency per entry: 67 us for 256 entries x 8 x 1024 clusters, beside 23 us for the counts.
// What is left is writing: 9 bytes per pair, in half-wave rows of 128 bytes.
// Without places nothing ties the new entries together: they are dealt to gridDim.z workgroups of `share` entries each, so
// that few clusters do not leave the device idle.  With places (PLACE) one workgroup walks them all.
// WIDE: positions of new entries in 64 bits, for lists whose last pass could end past 2^31.  Signed 32-bit positions otherwise:
// unsigned ones that may pass 2^31 took 191 us where these take 183 (8192 new entries, 64 clusters, places), counting down as much.
template <int NR, int NW, bool PLACE, bool WIDE>
__global__ __launch_bounds__(64 * NW) void window_kernel(const v4u* __restrict__ bits, int nruns, int Npad, int N, int W,
                                                                const int32_t* __restrict__ new_ids, int n_new, int share,
                                                                const int32_t* __restrict__ medoids, int Nc, double tau,
                                                                const int32_t* __restrict__ primary, const int32_t* __restrict__ size, int D,
                                                                int32_t* __restrict__ f_out, uint8_t* __restrict__ member,
                                                                int32_t* __restrict__ disk, uint32_t* __restrict__ dev_flags) {
    using pos_t = std::conditional_t<WIDE, int64_t, int>;
    constexpr int SEGS = 2 * NW;                               // runs of consecutive new entries, one per half wave
    __shared__ uint32_t joined[SEGS][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cl = lane & 31, seg = wave * 2 + (lane >> 5);
    const int h = blockIdx.y;
    const int c = blockIdx.x * 32 + cl;
    const bool c_in = c < Nc;
    const v4u* hb = bits + (size_t)h * nruns * Npad;
    const v4u zero = {0u, 0u, 0u, 0u};

    const int32_t m = c_in ? medoids[(size_t)h * Nc + c] : 0;
    const bool m_ok = m >= 0 && m < N;
    bool bad = !m_ok;
    v4u mw[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) mw[r] = (r < nruns && m_ok) ? hb[(size_t)r * Npad + m] : zero;

    // d = 1 - f / W falls as f grows, so "d < tau" is "f >= fstar": the smallest passing f in [0, W], W + 1 when none passes;
    // 64 candidates per round, the same fp64 expression as per pair
    int fstar = 0;
#pragma unroll
    for (int width = 64; width >= 1; width /= 64) {
        const int f = fstar + (lane + 1) * width - 1;
        const uint64_t pass = __ballot(1.0 - (double)f / (double)W < tau);
        fstar = pass ? fstar + (__ffsll((unsigned long long)pass) - 1) * width : W + 1;
        if (!pass) break;
    }

    int64_t base64 = 0;
    if (PLACE && c_in) base64 = (int64_t)primary[(size_t)h * Nc + c] + size[(size_t)h * Nc + c] + 1;
    const uint32_t base = (PLACE && base64 >= 0) ? (uint32_t)(base64 % D) : 0u;

    // new entries per run: as few as let one pass hold all of this workgroup's, at most WIN_PER_SEG
    const int per = (int)min((pos_t)WIN_PER_SEG, ((PLACE ? n_new : share) + (pos_t)(SEGS - 1)) / SEGS);
    const pos_t a_begin = PLACE ? 0 : (pos_t)blockIdx.z * share, a_end = PLACE ? n_new : min((pos_t)n_new, a_begin + share);
    uint32_t grown = 0;                                        // joiners of earlier passes
    for (pos_t a0 = a_begin; a0 < a_end; a0 += SEGS * per) {
        const pos_t first = a0 + seg * per;
        const int count = (int)min((pos_t)per, a_end - first);                        // <= 0: an empty run
        uint32_t joins = 0;
        constexpr int AHEAD = NR <= 2 ? 4 : NR <= 4 ? 2 : 1;   // new entries whose trace words are in flight together
        for (int e0 = 0; e0 < per; e0 += AHEAD) {
            int32_t id[AHEAD];
            v4u o[AHEAD][NR];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) id[u] = new_ids[(size_t)h * n_new + min(first + e0 + u, (pos_t)(n_new - 1))];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const bool e_ok = id[u] >= 0 && id[u] < N;
                bad |= !e_ok;
#pragma unroll
                for (int r = 0; r < NR; ++r) o[u][r] = (r < nruns && e_ok) ? hb[(size_t)r * Npad + id[u]] : zero;
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                int32_t f = 0;
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    f += __popc(mw[r].x & o[u][r].x) + __popc(mw[r].y & o[u][r].y) + __popc(mw[r].z & o[u][r].z) + __popc(mw[r].w & o[u][r].w);
                if (e0 + u < count) {
                    const bool join = f >= fstar;
                    joins |= (uint32_t)join << (e0 + u);
                    if (c_in) {
                        const size_t at = ((size_t)h * n_new + first + e0 + u) * Nc + c;
                        if (f_out) f_out[at] = f;
                        member[at] = join ? 1 : 0;
                    }
                }
            }
        }
        if (PLACE) {
            joined[seg][cl] = (uint32_t)__popc(joins);
            __syncthreads();
            uint32_t before = 0, all = 0;
#pragma unroll
            for (int s = 0; s < SEGS; ++s) {
                const uint32_t v = joined[s][cl];
                before += s < seg ? v : 0u;
                all += v;
            }
            __syncthreads();                                   // the counts have been read: the next pass may overwrite them
            if (c_in) {
                uint32_t g = grown + before;
                uint32_t place = (base + g) % (uint32_t)D;       // both below 2^31
                int32_t* dst = disk + ((size_t)h * n_new + first) * Nc + c;
#pragma unroll 1
                for (int e = 0; e < count; ++e, dst += Nc) {
                    int32_t v = -1;
                    if ((joins >> e) & 1u) {
                        v = base64 >= 0 ? (int32_t)place : (int32_t)((base64 + (int64_t)g) % D);   // a negative first SSD or size: the remainder as the language defines it
                        ++g;
                        place = place + 1 == (uint32_t)D ? 0u : place + 1;
                    }
                    *dst = v;
                }
            }
            grown += all;
        }
    }
    if (bad) atomicOr(dev_flags, SWARM_DEV_BAD_ENTRY);
}

}  // namespace

swarm_status launch_window(swarm_ctx* ctx, int nruns, int Npad, int N, int W, int H, const int32_t* new_ids, int n_new,
                           const int32_t* medoids, int Nc, double tau, const int32_t* primary, const int32_t* size, int D,
                           int32_t* f_out, uint8_t* member, int32_t* disk) {
    // Shares of the new entries when no places are asked for: one entry per half wave while that makes at most WGS workgroups
    // (two to a compute unit), larger ones otherwise.  8192 entries against 64 clusters of one head, window of 256 steps: 120 us on the two workgroups of
    // the clusters alone, 10.6 us on 512; 65536 entries 890 and 17 us (a workgroup per entry, as it once was: 23 and 106 us).
    constexpr int64_t WGS = 512;
    const int64_t blocks = (int64_t)((Nc + 31) / 32) * H;
    const int halves = nruns <= 8 ? 32 : 16;                   // half waves of a workgroup
    int64_t parts = disk ? 1 : WGS / blocks;
    const int64_t most = ((int64_t)n_new + halves - 1) / halves;
    parts = parts < 1 ? 1 : parts > most ? most : parts;
    const int share = (int)((n_new + parts - 1) / parts);
    const bool wide = n_new > (1 << 30);                       // below, no sum of a position and a pass or a share passes 2^31
    const dim3 grid((unsigned)((Nc + 31) / 32), (unsigned)H, (unsigned)(((int64_t)n_new + share - 1) / share));
#define SWARM_WINDOW(NR, NW) hipLaunchKernelGGL((wide ? (disk ? window_kernel<NR, NW, true, true> : window_kernel<NR, NW, false, true>) \
                                                      : (disk ? window_kernel<NR, NW, true, false> : window_kernel<NR, NW, false, false>)), grid, dim3(64 * NW), 0, ctx->stream, \
                                                reinterpret_cast<const v4u*>(ctx->trace), nruns, Npad, N, W, new_ids, n_new, share, medoids, Nc, tau, \
                                                primary, size, D, f_out, member, disk, ctx->dev_flags)
    if (nruns <= 2) SWARM_WINDOW(2, 16);
    else if (nruns <= 4) SWARM_WINDOW(4, 16);
    else if (nruns <= 8) SWARM_WINDOW(8, 16);
    else SWARM_WINDOW(WIN_MAX_RUNS, 8);                       // 64 registers of medoid words: half the waves, twice the registers
#undef SWARM_WINDOW
    return swarm_check_launch(ctx, "window_kernel");
}
