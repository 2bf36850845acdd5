// Co-activation counts of sparse traces (Section 5.1, Step 1: the same C = A^T A as coact.hip, the same integers).
//
// Row i of C is the sum of the selections of the trace rows that activate entry i: k increments for each of them, k^2 per
// trace row and head, where the dense product does N^2 multiply-adds whatever k is.  The increments are LDS atomics, and a
// compute unit takes one wave instruction of them every 4.2 cycles (4.8 on random addresses, however many lanes take part),
// some 13 increments a cycle against 16 thousand operations of the 4-bit matrix cores: from k = N / 64 down this is the shorter way.
//
// What bounds the obvious form (a workgroup per row of C, 128 KiB of counters) is the reading of the selections: each is read
// k times, 17 GB for 8192 of 1024 out of 65536 entries, which do not fit an L2 (3.9 ms without a single increment).  So the
// columns are cut into eight segments, one per XCD (workgroup b runs on XCD b % 8): an XCD meets only its segment's part of
// every selection, 2.7 MB of records that stay in its own L2, and a segment's 8192 counters leave room for four workgroups per
// compute unit.  Blocks of 32 columns (a line of C) are dealt to the segments, so that a run of neighbouring entries is spread evenly:
// with blocks of 64 a selection of whole pages of 64 entries takes 4.7 ms and not 4.4, with 16 the writing of C half as long again.
// Records have a fixed size -- the mean share of a segment, some standard deviations, and what completes a wave's division by
// whole records -- because walking ragged pieces costs more than the increments (pieces through a work list: 4.8 ms); the ids
// beyond it, rare unless the ids come in whole blocks, go to an overflow.
// 8192 selections of 1024 out of 65536 entries spread evenly: 5.4 to 5.8 ms by the dense product, 3.1 to 3.3 ms here with trace and records;
// on one device 3.33, without the writing of C 2.88, without the increments 3.33 (5.2 TB/s, what row pieces reach): they run side by side.
#include <numeric>
#include <type_traits>

#include "common.h"
#include "wave_ops.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_row __attribute__((ext_vector_type(4), aligned(4)));   // rows of C are 4-byte aligned when N is odd

constexpr int MAX_SEGMENTS = 8;       // one per XCD
constexpr int MAX_SEGMENT = 8192;     // columns of a segment: 32 KiB of counters
constexpr int BLOCK = 32;             // columns dealt to the segments together
constexpr int LIST_MAX_K = 1024;      // N / 64
constexpr int DUMMY_WORDS = 32;       // counters behind a segment's, taken by padding
constexpr int RT = 512;               // threads of a counting workgroup; with 256 the same within 2 %
constexpr int SLOTS = 128;            // workgroups of an XCD, four on each of its 32 compute units
constexpr int T_CAP = 1024;           // trace rows listed at a time
constexpr int QUEUE_STRIDE = 32;      // words from one XCD's counter of rows handed out to the next

// Each group of nseg blocks deals one to every segment, turned from group to group by a hash of its number: dealt in turn, entries at
// a distance of a multiple of 32 nseg fall to one segment, that is to one XCD of eight, and nearly all of them to the overflow (8192
// selections of 1024 out of every eighth 64 of 65536 entries took 18.3 ms; now 3.4).  Of all distances of up to a sixth of a segment's
// blocks, and 4 x 8192 to 65536 entries, this constant leaves the fullest segment at most 1 + 2.4 / sqrt(n) times its share of n blocks.
__host__ __device__ __forceinline__ uint32_t turn_of(uint32_t group) { return group * 0xf2ee4e45u >> 29; }
// Entries at a fixed distance would share a bank: the counters of each pair of blocks lie in an order of their own, place i at i ^ mix
// (every 64th entry in each of 8192 selections of 128 out of 8 x 8192 entries 1.07 -> 0.63 ms, where blocks turned by four words meet
// eight banks).
__host__ __device__ __forceinline__ uint32_t mix_of(uint32_t pair) { return pair * 0x9e3779b1u >> 26; }

// Columns of a segment: whole pairs of blocks, a counter on each of the 64 LDS banks.
__host__ __device__ __forceinline__ int seg_columns(int N, int nseg) { return (N + nseg * 64 - 1) / (nseg * 64) * 64; }

// Every selection becomes one record per segment: the byte offsets of its distinct valid ids' counters, 16 bits each, in L
// groups of eight, and the rest in the overflow.  Id p of a record is in group p % L, so that the lanes of a wave, a
// group each, meet neighbouring ids together (a run of entries then falls on distinct LDS banks).  One wave per
// selection: 30 us for 8192 of 1024.
__global__ __launch_bounds__(64) void list_build_kernel(const int32_t* __restrict__ idx, int64_t rows, int recs, int H, int k, int N, int nseg_log2,
                                                        int L, int ext_groups, uint4* __restrict__ lists, uint4* __restrict__ ext,
                                                        uint32_t* __restrict__ queue) {
    constexpr int PER = LIST_MAX_K / 64;
    __shared__ uint32_t piece[MAX_SEGMENTS];
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    const int lane = threadIdx.x;
    const int64_t r = blockIdx.x;                                       // row * H + head, as the selections lie in memory
    const int h = (int)(r % H);
    const int64_t row = r / H, t = (row & ~31ll) | trace_bit((int)(row & 31));       // records lie in the order of the trace's bits
    const int nseg = 1 << nseg_log2, cols = seg_columns(N, nseg);
    const int32_t* sel = idx + r * k;
    uint4* rec4 = reinterpret_cast<uint4*>(dyn);                        // the records, segment after segment
    uint16_t* rec = reinterpret_cast<uint16_t*>(dyn);
    uint32_t* seen = dyn + (L * 4 << nseg_log2);                        // N bits
    int32_t e[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) e[u] = u * 64 + lane < k ? sel[u * 64 + lane] : N;
    if (lane < MAX_SEGMENTS) piece[lane] = 0u;
    if (blockIdx.x == 0 && lane < 8) queue[lane * QUEUE_STRIDE] = 0u;     // for the counting kernel that follows
    for (int g = lane; g < L << nseg_log2; g += 64) {                   // padding everywhere, a bank of its own for every lane that meets it
        const uint32_t d = (uint32_t)(cols + (g & (DUMMY_WORDS - 1))) * 4 * 0x10001u;
        rec4[g] = make_uint4(d, d, d, d);
    }
    bool fine = true;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        int32_t prev = __shfl_up(e[u], 1, 64);
        if (lane == 0) prev = u ? __builtin_amdgcn_readlane(e[u ? u - 1 : 0], 63) : -1;
        if (u * 64 + lane < k) fine &= (uint32_t)e[u] < (uint32_t)N && prev < e[u];
        else e[u] = -1;
    }
    if (__ballot(!fine) != 0) {                                         // repeated, unsorted or invalid ids: the distinct valid ones stay
        for (int w = lane; w < (N + 31) / 32; w += 64) seen[w] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if ((uint32_t)e[u] >= (uint32_t)N || (atomicOr(&seen[e[u] >> 5], 1u << (e[u] & 31)) >> (e[u] & 31)) & 1u) e[u] = -1;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint32_t slots = 8u * L, cap = nseg > 1 ? slots - 1 : slots;
    const uint32_t inv = (65536u + L - 1) / L;                          // p / L for p < 1024
    // Records of neighbouring trace rows list an id as different ones of a group's first seven: lanes of a wave that add to one counter at
    // once wait for each other (the same 1024 entries in every row 4.2 -> 3.45 ms).
    const uint32_t turn = (uint32_t)t % 7u;
    auto slot = [&](uint32_t s, uint32_t p) __attribute__((always_inline)) {
        const uint32_t q = p * inv >> 16, turned = q + turn < 7u ? q + turn : q + turn - 7u;
        return s * slots + (p - q * L) * 8 + (q < 7u ? turned : 7u);
    };
    auto seg_of = [&](int32_t x) __attribute__((always_inline)) {
        const uint32_t block = (uint32_t)x / BLOCK;
        return (block + turn_of(block >> nseg_log2)) & (uint32_t)(nseg - 1);
    };
    auto counter_of = [&](int32_t x) __attribute__((always_inline)) {
        const uint32_t in_seg = ((uint32_t)x / BLOCK >> nseg_log2) * BLOCK + (uint32_t)x % BLOCK;
        return (uint16_t)((in_seg ^ mix_of(in_seg / 64)) * 4);
    };
    uint32_t place[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        place[u] = 0;
        if (e[u] >= 0) {
            place[u] = atomicAdd(&piece[seg_of(e[u])], 1u);
            if (place[u] < cap) rec[slot(seg_of(e[u]), place[u])] = counter_of(e[u]);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint32_t cnt = lane < nseg ? piece[lane] : 0u;
    if (__ballot(cnt > cap) != 0) {                                     // pieces that go on in the overflow, in whole groups
        const uint32_t ng = cnt > cap ? (cnt - cap + 7) / 8 : 0u;
        uint32_t total;
        const uint32_t off = waveops::wave_excl_scan(ng, &total);
        uint16_t* out = reinterpret_cast<uint16_t*>(ext + ((size_t)h * recs + t) * ext_groups);
        if (ng) {
            rec[slot(lane, slots - 1)] = (uint16_t)(1u | off << 1 | (ng - 1) << 9);        // odd, as no counter's offset is; off < 136, ng <= 128
            for (uint32_t p = cnt - cap; p < ng * 8; ++p) out[off * 8 + p] = (uint16_t)((cols + (lane & (DUMMY_WORDS - 1))) * 4);
            piece[lane] = off * 8;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (e[u] >= 0 && place[u] >= cap) out[piece[seg_of(e[u])] + place[u] - cap] = counter_of(e[u]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int g = lane; g < L << nseg_log2; g += 64) {
        const int s = g / L;
        lists[(((size_t)h * nseg + s) * recs + t) * L + (g - s * L)] = rec4[g];
    }
}

// Persistent workgroups: a workgroup takes rows of C one after the other, its XCD's segment of each.  While a row's records are
// summed, the trace rows of the next one are listed and the trace words of the one after are on their way, so a row costs two
// barriers.  The trace words of an entry's column (bits, see coact.hip) say which records to sum; a wave reads 64 / L records at
// once, a group of eight ids per lane.
// RHO: also counts, per row, the elements that reach the head's threshold (rho must be zero before).  SEG: more than one segment.
template <bool RHO, bool SEG>
__global__ __launch_bounds__(RT, 8) void coact_rows_kernel(const uint32_t* __restrict__ bits, const uint4* __restrict__ lists, int recs, int H, int N,
                                                           int Npad, int nruns, int nseg_log2, int L, int ext_groups, uint32_t* __restrict__ queue,
                                                           uint32_t row_step, uint32_t groups_inv, int32_t* __restrict__ C,
                                                           const int64_t* __restrict__ cstar, int32_t* __restrict__ rho) {
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    const int nseg = 1 << nseg_log2, cols = seg_columns(N, nseg);
    uint32_t* cnt = smem;                                                        // cols + DUMMY_WORDS counters
    uint16_t* tl = reinterpret_cast<uint16_t*>(smem + cols + DUMMY_WORDS);       // [2][T_CAP]
    __shared__ uint32_t tcount[2], fetched;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int seg = xcd & (nseg - 1), parts = 8 >> nseg_log2, part = xcd >> nseg_log2;
    const int nwords = nruns * 4, chunks = (nwords + RT - 1) / RT;
    const int lpw = 64 / L, my_list = lane / L, my_group = lane - my_list * L;   // lists a wave works on side by side
    for (int w = tid; w < (cols + DUMMY_WORDS) / 4; w += RT) reinterpret_cast<v4i*>(cnt)[w] = v4i{0, 0, 0, 0};
    if (tid < 2) tcount[tid] = 0;
    __syncthreads();

    // An XCD's rows are handed out one by one, each to the first workgroup that gets there: what a row costs differs by its entry's count,
    // and dealt beforehand, by equal rounds or rounds turned by a hash, often activated entries pile up on some workgroups (every 64th
    // entry in each of 8192 selections of 1024: 470 ms and 4.7, handed out 4.3; nine neighbours every 576 entries 9.6 and 3.9; any 1024
    // entries 5.8 and 4.2; ids spread evenly 3.45 and 3.1).  A workgroup's first two rows are known; the number of a later one is asked
    // for while two others are before it.  Where several XCDs share a segment, the rows are dealt to them as the blocks to the segments.
    // They are handed out in groups of eight (whose trace words share lines) spread over the head, not in order: where some region of the
    // entries is activated more than another, its increments then lie beside the other's writing (half a run, the rest of the ids in the
    // lower half of 65536: in order 3.97 ms, spread 3.16; pages of 64, as everywhere alike, 3.84 and 4.05).
    struct Place { int h, i, chunk, before, row; };            // before: rows of earlier heads
    auto begin = [&](Place& p, uint32_t place) __attribute__((always_inline)) {
        p.chunk = 0;
        p.i = (int)(place * (uint32_t)parts + ((part + turn_of(place)) & (uint32_t)(parts - 1))) - p.before;
        while (p.i >= N) { p.i -= N; p.before += N; ++p.h; }
        const uint32_t groups = (uint32_t)N / 8, x = (uint32_t)p.i / 8 * row_step;
        const int group = (int)(x - __umulhi(x, groups_inv) * groups);             // x modulo groups, or groups less
        p.row = (group < 0 ? group + (int)groups : group) * 8 + (p.i & 7);
    };
    uint32_t upcoming = slot + SLOTS;
    auto advance = [&](Place& p) __attribute__((always_inline)) {
        if (++p.chunk < chunks) return false;
        begin(p, upcoming);
        return true;
    };
    auto ask = [&]() __attribute__((always_inline)) {
        return 2 * SLOTS + __hip_atomic_fetch_add(queue + xcd * QUEUE_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const uint32_t word_off = ((uint32_t)(tid >> 2) * (uint32_t)Npad * 4 + (tid & 3)) * 4;       // bytes, inside a head's trace
    auto load_word = [&](const Place& p) __attribute__((always_inline)) -> uint32_t {
        if (p.chunk * RT + tid >= nwords || p.h >= H) return 0u;
        const char* base = reinterpret_cast<const char*>(bits) + (((size_t)p.h * nruns + p.chunk * (RT / 4)) * Npad + p.row) * 16;
        return *reinterpret_cast<const uint32_t*>(base + word_off);
    };
    // lists the records of the trace rows of this thread's word
    auto list_rows = [&](uint32_t word, int chunk, int buf) __attribute__((always_inline)) {
        if (word) {
            uint32_t at = atomicAdd(&tcount[buf], (uint32_t)__popc(word));
            const uint32_t t0 = (uint32_t)(chunk * RT + tid) * 32;
            while (word) {
                tl[buf * T_CAP + (at & (T_CAP - 1))] = (uint16_t)(t0 + __ffs(word) - 1);
                word &= word - 1;
                ++at;
            }
        }
    };
    auto add = [&](uint32_t at) __attribute__((always_inline)) {
        __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(cnt) + at), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    const uint32_t end = (uint32_t)cols * 4;
    auto add8 = [&](const uint4& x, uint32_t last) __attribute__((always_inline)) {
        add(x.x & 0xffffu); add(x.x >> 16);
        add(x.y & 0xffffu); add(x.y >> 16);
        add(x.z & 0xffffu); add(x.z >> 16);
        add(x.w & 0xffffu);
        if (__ballot(last < end) != 0) add(last);             // the last eighth of the slots is mostly padding
    };
    const uint32_t rec_bytes = (uint32_t)L * 16, group_off = (uint32_t)my_group * 16;
    const uint4* ext = lists + ((size_t)recs * H * L << nseg_log2);

    Place at{0, 0, 0, 0, 0};
    begin(at, slot);
    Place ahead = at;
    int buf = 0;
    uint32_t word = load_word(at);
    list_rows(word, 0, 0);
    const bool took_first = advance(ahead);
    uint32_t next = load_word(ahead);
    if (tid == 0) fetched = took_first ? ask() : upcoming;
    __syncthreads();
    upcoming = (uint32_t)__builtin_amdgcn_readfirstlane((int)fetched);
    __syncthreads();
    while (at.h < H) {
        const char* hl = reinterpret_cast<const char*>(lists + ((size_t)at.h * nseg + seg) * recs * L);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)tcount[buf]), word_now = word;
        list_rows(next, ahead.chunk, buf ^ 1);                // the rows of the step after this one listed, the words after those requested
        word = next;
        const Place after = ahead;
        const bool took = advance(ahead);
        next = load_word(ahead);
        uint32_t asked = 0;
        if (took && tid == 0) asked = ask();
        const int parts_of = n <= T_CAP ? 1 : (min(nwords - at.chunk * RT, RT) + 31) / 32;        // too many for the list: the words 32 at a time
        for (int s = 0; s < parts_of; ++s) {
            uint32_t m = n;
            if (parts_of > 1) {
                __syncthreads();
                if (tid == 0) tcount[buf] = 0;
                __syncthreads();
                if ((tid >> 5) == s) list_rows(word_now, at.chunk, buf);
                __syncthreads();
                m = (uint32_t)__builtin_amdgcn_readfirstlane((int)tcount[buf]);
            }
            constexpr int U = 3;                              // records in flight per lane; 2, 3, 4 and 6 within 2 %
            const uint16_t* t_of = tl + buf * T_CAP;
            const uint32_t step = (RT / 64) * lpw;
            if (my_list < lpw) {
                for (uint32_t p0 = wave * lpw; p0 < m; p0 += U * step) {
                    uint4 v[U];
                    uint32_t t[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        t[u] = t_of[min(p0 + u * step + my_list, m - 1)];
                        v[u] = *reinterpret_cast<const uint4*>(hl + (t[u] * rec_bytes + group_off));
                    }
                    // Pieces that go on: the lanes of a record read its overflow, for all records side by side, and the first of it
                    // before anything is added.
                    uint64_t goes_on = 0;
                    uint32_t rest[U];                          // groups of overflow from this lane's first on
                    const uint4* from[U];
                    uint4 y[U];
                    if (SEG) {
#pragma unroll
                        for (int u = 0; u < U; ++u) goes_on |= __ballot((v[u].w >> 16) & 1u);
                        if (__builtin_expect(goes_on != 0, 0)) {
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                const uint32_t x = (uint32_t)__shfl((int)(v[u].w >> 16), my_list * L + L - 1, 64);     // the record's last slot
                                const uint32_t ng = (x & 1u) && p0 + u * step + my_list < m ? (x >> 9) + 1 : 0u;
                                rest[u] = ng > (uint32_t)my_group ? ng - (uint32_t)my_group : 0u;
                                from[u] = ext + ((size_t)at.h * recs + t[u]) * ext_groups + ((x >> 1) & 0xffu) + my_group;
                                if (rest[u]) y[u] = *from[u];
                            }
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        uint32_t last = v[u].w >> 16;
                        if (SEG) last = last & 1u ? end : last;
                        if (p0 + u * step + my_list < m) add8(v[u], last);
                    }
                    if (SEG && __builtin_expect(goes_on != 0, 0)) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            if (rest[u]) add8(y[u], y[u].w >> 16);
                            for (uint32_t g = L; g < rest[u]; g += L) {
                                const uint4 z = from[u][g];
                                add8(z, z.w >> 16);
                            }
                        }
                    }
                }
            }
        }
        if (took && tid == 0) fetched = asked;
        __syncthreads();
        upcoming = (uint32_t)__builtin_amdgcn_readfirstlane((int)fetched);
        if (tid == 0) tcount[buf] = 0;
        buf ^= 1;
        if (after.chunk == 0) {
            // the row's segment leaves, its counters are cleared
            char* row = reinterpret_cast<char*>(C + ((size_t)at.h * N + at.row) * N);
            int32_t c32 = 0x7fffffff;
            if (RHO) {
                const int64_t c = cstar[at.h];
                if (c < 0x7fffffffll) c32 = (int32_t)c;
            }
            int near = 0;
            auto leave = [&](auto whole_tag) __attribute__((always_inline)) {
                constexpr bool WHOLE = decltype(whole_tag)::value;
                for (int w = tid; w < cols / 4; w += RT) {
                    const uint32_t group = (uint32_t)w / (BLOCK / 4), mix = mix_of((uint32_t)w / 16);
                    const uint32_t e = ((group << nseg_log2) + (((uint32_t)seg - turn_of(group)) & (uint32_t)(nseg - 1))) * BLOCK + (w & (BLOCK / 4 - 1)) * 4;
                    const uint32_t at_w = (uint32_t)w ^ (mix >> 2);
                    v4i v = reinterpret_cast<const v4i*>(cnt)[at_w];
                    v = mix & 1u ? v4i{v.y, v.x, v.w, v.z} : v;
                    v = mix & 2u ? v4i{v.z, v.w, v.x, v.y} : v;
                    reinterpret_cast<v4i*>(cnt)[at_w] = v4i{0, 0, 0, 0};
                    if (WHOLE || e + 4 <= (uint32_t)N) {
                        __builtin_nontemporal_store((v4i_row)v, reinterpret_cast<v4i_row*>(row + e * 4));
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (e + q < (uint32_t)N) reinterpret_cast<int32_t*>(row)[e + q] = v[q];
                    }
                    if (RHO) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) near += __popcll(__ballot(v[q] >= c32 && (WHOLE || e + q < (uint32_t)N)));
                    }
                }
            };
            if ((cols << nseg_log2) == N) leave(std::true_type{});
            else leave(std::false_type{});
            if (RHO && lane == 0 && near) atomicAdd(rho + (size_t)at.h * N + at.row, near);
        }
        at = after;
        __syncthreads();
    }
}

struct RowsPlan { int nseg_log2, L, ext_groups; };
RowsPlan plan_of(int N, int k) {
    RowsPlan p{0, 0, 0};
    while ((1 << p.nseg_log2) < MAX_SEGMENTS && N > (MAX_SEGMENT << p.nseg_log2)) ++p.nseg_log2;
    const int nseg = 1 << p.nseg_log2;
    int room = k;
    if (nseg > 1) {
        const int mean = (k + nseg - 1) / nseg;
        int s = 1;                                            // 2.5 standard deviations of ids that fall anywhere
        while (4 * s * s < 25 * mean) ++s;
        room = mean + s + 1;
    }
    p.L = 64 / (64 / ((room + 7) / 8));                       // as long as as many records fit a wave
    p.ext_groups = nseg > 1 ? (k + 7 * nseg) / 8 : 0;         // a single segment's record holds all of k
    return p;
}

}  // namespace

// Where the increments win, measured on both ways for N from 2048 to 65536, 1024 to 65535 trace rows, k from N / 44 to N / 128, and ids
// spread evenly, in pages, with a sink and a window, by Zipf's law, at fixed distances and the same in every row:
//  - k <= N / 64: at N / 44 three records to a wave become two (8192 rows 0.75 to 1.0 times as fast before rows were handed out);
//  - 6144 rows: below, the dense product waits for the writing of C as well (5120 rows 0.97 to 1.2);
//  - N >= 5120, or from 4096 on where more rows or shorter selections outweigh the two barriers of a row: spread ids, and with a sink,
//    32 x 4096^2, k = 64: 6144 rows 0.96 and 0.83, 8192 1.07 and 0.92, 16384 1.15 and 1.01; k = 32: 6144 rows 1.04 and 0.97, 8192 1.13
//    and 1.02; 21 x 5120^2, k = 80: 6144 rows 1.11 and 0.98, 8192 1.24 and 1.10;
//  - N a multiple of 16: a 64-byte piece of C shared by two XCDs is written twice (N = 12289: 0.85); so is every one of a C that itself starts inside
//    a piece (65536^2 14.8 ms, the dense product 8.6; 24576^2 1.97 and 1.2, 4 x 12288^2 1.92 and 1.1), unless one segment holds all
//    columns (8 x 8192^2 578 and 848 us).  Whole pieces that share a line are level or better (6144 rows, rows of 24592 563 and 634 us, of
//    16400 563 and 566; a C 64 bytes past a line, 24576^2 645 and 645, 4 x 12288^2 678 and 623);
//  - 2^29 counts: an entry that all of 8192 rows activate keeps one workgroup busy; handed out last it adds 40 us to 495 of 8 x 8192^2, 100 to
//    3250 of 65536^2, and would add as much to a smaller build.
// 8192 rows, k = N / 64, spread ids: 8 x 8192^2 733 -> 493 us, 4 x 12288^2 829 -> 541, 32768^2 1391 -> 803, 65536^2 5.7 -> 3.2 ms.  The worst
// that was found inside these bounds: pages of 64 from every ninth block of 40960 entries 0.90, the same ids in all of 6144 rows 0.96, and
// ids that were picked to fall to one segment 0.34.
// The ids of a segment and the trace rows have to fit 16 bits, a wave per selection one launch.
bool rows_route(int64_t rows, int H, int N, int k, const int32_t* C) {
    if (rows < 6144 || rows > 65535 || rows * H > (int64_t)1 << 25) return false;
    if (N < 4096 || N > MAX_SEGMENTS * MAX_SEGMENT || N % 16 != 0 || k > N / 64 || (int64_t)H * N * N < (int64_t)1 << 29) return false;
    if (N > MAX_SEGMENT && reinterpret_cast<uintptr_t>(C) % 64 != 0) return false;
    return N >= 5120 || rows >= 16384 || (rows >= 8192 && k <= N / 128);
}

// Scratch for the records, their overflow and the counters of rows handed out: at most 6 bytes per id and 300 per selection.
size_t rows_list_bytes(int64_t rows, int H, int k, int N) {
    const RowsPlan p = plan_of(N, k);
    const int64_t recs = (rows + 31) / 32 * 32;
    return (size_t)recs * H * ((((size_t)p.L << p.nseg_log2) + p.ext_groups) * 16) + 8 * QUEUE_STRIDE * 4;
}

swarm_status launch_coact_rows(swarm_ctx* ctx, const int32_t* idx, int64_t rows, int H, int k, int N, int Npad, int nruns, int32_t* C,
                               void* scratch, const int64_t* cstar, int32_t* rho) {
    const RowsPlan p = plan_of(N, k);
    const int recs = (int)((rows + 31) / 32 * 32);
    uint4* lists = static_cast<uint4*>(scratch);
    uint4* ext = lists + ((size_t)recs * H * p.L << p.nseg_log2);
    uint32_t* queue = reinterpret_cast<uint32_t*>(ext + (size_t)recs * H * p.ext_groups);
    hipLaunchKernelGGL(list_build_kernel, dim3((unsigned)(rows * H)), dim3(64),
                       ((size_t)p.L * 16 << p.nseg_log2) + (size_t)((N + 31) / 32) * 4, ctx->stream, idx, rows, recs, H, k, N, p.nseg_log2, p.L,
                       p.ext_groups, lists, ext, queue);
    swarm_status st = swarm_check_launch(ctx, "list_build_kernel");
    if (st != SWARM_OK) return st;
    // the groups of eight rows in steps of the golden section, without a common divisor: any stretch of them is spread over the head
    const uint32_t groups = (uint32_t)N / 8, groups_inv = (uint32_t)((((uint64_t)1 << 32) + groups - 1) / groups);
    uint32_t row_step = (uint32_t)(0.6180339887 * groups) | 1u;
    while (std::gcd(row_step, groups) != 1u) row_step += 2;
    const int lds = (seg_columns(N, 1 << p.nseg_log2) + DUMMY_WORDS) * 4 + 2 * T_CAP * 2;
    hipLaunchKernelGGL(p.nseg_log2 ? (cstar ? coact_rows_kernel<true, true> : coact_rows_kernel<false, true>)
                                   : (cstar ? coact_rows_kernel<true, false> : coact_rows_kernel<false, false>),
                       dim3(8 * SLOTS), dim3(RT), lds, ctx->stream, reinterpret_cast<const uint32_t*>(ctx->trace), lists, recs, H, N, Npad, nruns,
                       p.nseg_log2, p.L, p.ext_groups, queue, row_step, groups_inv, C, cstar, rho);
    ctx->count_way = SWARM_WAY_ROWS;
    return swarm_check_launch(ctx, "coact_rows_kernel");
}
