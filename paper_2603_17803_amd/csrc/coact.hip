// Activation trace and co-activation accumulation (Section 5.1, Step 1): C[i][j] = number of trace
// rows in which entries i and j are both activated, i.e. C = A^T A for the binary trace A.
//
// The trace is binary, so it is kept in memory as bits: for every head and every run of 128 trace
// rows one 16-byte word per entry, bits[h][run][entry], one bit per trace row of the run (rows 32w ..
// 32w+31 in dword w, in the order of trace_bit below).  Both operands of the product are entry panels of this one array.  On the way
// to the matrix cores the bits are expanded to 4-bit 0/1 operands -- the 128 tile rows by the workgroup, into LDS
// (contraction index contiguous), the 64 tile columns of a wave by the wave itself, in registers -- and the product
// runs on the 4-bit form of v_mfma_f32_32x32x64_f8f6f4, exact for these operands (see below).  Feeding expanded
// operands from memory instead would multiply the traffic through the L2 by four to eight; the bit form keeps a
// smaller tile affordable.
// C is symmetric, so only tiles on or above the diagonal are computed and each off-diagonal tile is
// stored twice (once transposed).
#include <stdlib.h>

#include <type_traits>

#include "common.h"

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_row __attribute__((ext_vector_type(4), aligned(4)));   // four counts of a row of C: rows are 4-byte aligned only when N is odd
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int TRACE_SPAN = 8192;   // entries one trace-building workgroup covers at most (128 KiB of LDS)
constexpr int TRACE_SPAN_MIN = 512;
constexpr int TRACE_THREADS = 1024;

// One workgroup per (run of 128 trace rows, head, span of entries): the 128 selections are merged
// into an LDS image of the run's bit words, which then leaves as one contiguous, fully written block
// (no separate clearing pass, no global atomics).
// The run's selections are one flat list of ids, VEC: taken four at a time (k a multiple of 4, idx 16-byte aligned), so that
// a division by k (a multiplication by its reciprocal, where that is exact) and a load serve four ids: 8192 rows of 1024
// ids over 65536 entries, counted, 109 -> 56 us (8 spans scan each id), 4096 rows of 256 over 8 x 8192 entries 24 -> 16 us.
// (The image as four planes of dwords, free of bank conflicts on consecutive ids: no gain, 7.1 -> 7.9 us on short runs.)
// COUNT: also count, per trace row, the bits this workgroup sets for the first time (= the row's number
// of distinct valid entries inside the span) into row_count[span][h][run * 128 + row], and clear rho for the build's epilogue.
template <bool COUNT, bool VEC>
__global__ __launch_bounds__(TRACE_THREADS) void trace_build_kernel(const int32_t* __restrict__ idx, int64_t rows, int H, int k, int N,
                                                           int Npad, int nruns, int max_span, uint32_t reciprocal, uint4* __restrict__ bits,
                                                           uint32_t* __restrict__ dev_flags, int32_t* __restrict__ row_count,
                                                           int32_t* __restrict__ rho) {
    extern __shared__ __attribute__((aligned(16))) uint32_t words[];          // [span][4], then 128 row counters when COUNT
    constexpr int Q = VEC ? 4 : 1;                                            // ids per list item
    constexpr int AHEAD = VEC ? 4 : 8;                                        // list items in flight per thread
    const int run = blockIdx.x, h = blockIdx.y;
    const int e0 = blockIdx.z * max_span;
    const int span = min(max_span, Npad - e0);
    uint32_t* fresh = words + span * 4;
    for (int i = threadIdx.x; i < span; i += TRACE_THREADS) reinterpret_cast<uint4*>(words)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (COUNT && threadIdx.x < 128) fresh[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t row0 = (int64_t)run * 128;
    const int nrows = (int)min((int64_t)128, rows - row0);                       // <= 0 for a run of pure padding
    bool bad = false;
    const uint32_t kq = (uint32_t)k / Q;
    const uint32_t total = nrows > 0 ? (uint32_t)nrows * kq : 0u;                // at most 2^31 (a window over 2^24 entries): unsigned, so that a step past the end does not wrap
    const int64_t row_stride = (int64_t)H * k;
    const int32_t* sel0 = idx + (row0 * H + h) * (int64_t)k;
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += AHEAD * TRACE_THREADS) {
        int32_t e[AHEAD][Q];
        int s[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const uint32_t i = min(i0 + u * TRACE_THREADS, total - 1);                  // past the end: a valid load that is not used
            s[u] = (int)(reciprocal ? __umulhi(i, reciprocal) : i / kq);
            const int32_t* p = sel0 + s[u] * row_stride + (i - (uint32_t)s[u] * kq) * Q;
            if constexpr (VEC) {
                const int4 v = *reinterpret_cast<const int4*>(p);
                e[u][0] = v.x; e[u][1] = v.y; e[u][2] = v.z; e[u][3] = v.w;
            } else {
                e[u][0] = *p;
            }
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (i0 + u * TRACE_THREADS >= total) continue;
            const uint32_t bit = 1u << trace_bit(s[u] & 31);
            uint32_t* row_words = words + (s[u] >> 5);
            uint32_t nfirst = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int32_t id = e[u][q];
                bad |= (uint32_t)id >= (uint32_t)N;
                if ((uint32_t)id < (uint32_t)N && (uint32_t)(id - e0) < (uint32_t)span) {
                    const uint32_t old = atomicOr(row_words + (id - e0) * 4, bit);
                    if (COUNT) nfirst += (old & bit) == 0u;
                }
            }
            if (COUNT) {
                // the lanes of a wave mostly work on one trace row (consecutive list items): one add per wave then
                const int s0 = __builtin_amdgcn_readfirstlane(s[u]);
                if (__builtin_amdgcn_ballot_w64(s[u] != s0) == 0) {
                    uint32_t sum = 0;
#pragma unroll
                    for (int b = 0; b < (VEC ? 3 : 1); ++b) sum += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((nfirst >> b) & 1u)) << b;
                    if (sum && (threadIdx.x & 63) == (unsigned)__builtin_ctzll(__builtin_amdgcn_ballot_w64(true))) atomicAdd(&fresh[s0], sum);
                } else if (nfirst) {
                    atomicAdd(&fresh[s[u]], nfirst);
                }
            }
        }
    }
    if (bad && blockIdx.z == 0) atomicOr(dev_flags, SWARM_DEV_BAD_ENTRY);
    __syncthreads();
    uint4* out = bits + ((size_t)h * nruns + run) * Npad + e0;
    for (int i = threadIdx.x; i < span; i += TRACE_THREADS) out[i] = reinterpret_cast<const uint4*>(words)[i];
    if (COUNT) {
        if (threadIdx.x < 128) row_count[(((size_t)blockIdx.z * H + h) * nruns + run) * 128 + threadIdx.x] = (int32_t)fresh[threadIdx.x];
        if (run == 0)
            for (int i = threadIdx.x; i < span && e0 + i < N; i += TRACE_THREADS) rho[(size_t)h * N + e0 + i] = 0;
    }
}

// Optional validation: flags a repeated entry inside one (row, head) selection.
__global__ void check_distinct_kernel(const int32_t* __restrict__ idx, int k, uint32_t* __restrict__ dev_flags) {
    const int32_t* sel = idx + (size_t)blockIdx.x * k;
    bool dup = false;
    for (int a = threadIdx.x; a < k; a += blockDim.x) {
        const int32_t e = sel[a];
        for (int b = 0; b < a; ++b) dup |= (sel[b] == e);
    }
    if (dup) atomicOr(dev_flags, SWARM_DEV_DUP_ENTRY);
}

// floor((old * decay_q16 + 2^15) / 2^16) with a 64-bit intermediate (one 64-bit multiply-add and a
// funnel shift; decay_q16 <= 65536, so the result fits int32).
__device__ __forceinline__ int32_t decayed(int32_t old, uint32_t decay_q16) {
    return (int32_t)(((int64_t)old * (int64_t)decay_q16 + 32768) >> 16);
}

// Updated count for the accumulating (MODE 1) and decayed (MODE 2) forms: v >= 0 is added to the old
// count or to its decayed value.  A sum that passes INT32_MAX wraps and sets `ovf`.
template <int MODE>
__device__ __forceinline__ int32_t updated_count(int32_t old, int32_t v, uint32_t decay_q16, bool& ovf) {
    const int32_t base = MODE == 1 ? old : decayed(old, decay_q16);
    const int32_t s = (int32_t)((uint32_t)base + (uint32_t)v);
    ovf |= s < base;
    return s;
}

constexpr int TM = 128;                        // C tile rows per workgroup
constexpr int TN = 128;                        // C tile columns per workgroup
constexpr int KC = 64;                         // contraction BYTES per chunk and operand row: 128 trace rows as 4-bit values, two MFMA k-steps of 64
constexpr int A_BYTES = TM * KC;               // A operand panel of one chunk in LDS: 8 KiB; two of them form the ring
constexpr int RAW_DEPTH = 4;                   // chunks of raw trace bits on their way from memory or waiting in LDS
constexpr int RAW_CHUNK = (TM + TN) * 16;      // one chunk of raw bits: the 16-byte run words of the tile's 128 rows, then of its 128 columns
constexpr int RAW_BASE = 2 * A_BYTES;          // the raw ring sits behind the operand ring
constexpr int SYRK_WAVES = 4;                  // 2 x 2 waves of 64 x 64
constexpr int TROW = 256 + 16;                 // epilogue staging row (64 counts), padded: the 16-byte slots of 8 consecutive lanes differ
constexpr int SYRK_LDS_BYTES = SYRK_WAVES * 32 * TROW;   // 34 KiB: the epilogue's staging (one 32-column block per wave) is the larger user
static_assert(SYRK_LDS_BYTES >= RAW_BASE + RAW_DEPTH * RAW_CHUNK, "operand ring and raw ring must fit");

// Operand rows in LDS are 64 bytes; 16-byte piece c of row r lives at slot c ^ swz(r).  Measured on
// gfx950: a 16-byte LDS read is served 16 consecutive lanes at a time across 64 four-byte banks, a
// 16-byte write 8 consecutive lanes at a time with only address bits 4..6 telling lanes apart.
// Fragment reads take one piece of 16 consecutive rows, so rows that agree in bits 0..1 need
// different swz; the expansion writes of 8 consecutive lanes cover 4 rows x 2 halves, so bit 0 of swz
// must follow bit 1 of the row.  swz = (bit1 ^ bit3) | bit2 << 1 does both.
__device__ __forceinline__ int lds_swz(int row) { return (((row >> 1) ^ (row >> 3)) & 1) | (((row >> 2) & 1) << 1); }
__device__ __forceinline__ int lds_off(int row, int piece) { return row * KC + ((piece ^ lds_swz(row)) << 4); }

// The matrix-core instruction is v_mfma_f32_32x32x64_f8f6f4 in its 4-bit form (E2M1): 0 and 1 are
// exact in it, products of them are exact, and the fp32 accumulators hold every integer up to 2^24
// exactly -- a call accumulates at most 2^24 trace rows, so the counts are exact, at twice the rate of
// the int8 instruction and with half the operand bytes.  Lane l of an operand holds row l%32, contraction
// indices [32 (l/32), +32) as 32 nibbles (16 bytes); 0.5, 1.0 and 2.0 are the nibbles 0b0001, 0b0010, 0b0100.
// No block scales (the unscaled form of the instruction: measured 3 % faster in the contraction loop than the scaled
// form with both scales 2^0, same results).
// Expansion of trace bits to nibbles: the rows of a 32-row group sit in their word so that the eight
// consecutive rows of an output dword are the same bit of the word's eight nibbles (trace_bit above),
// and a mask (with a shift where the bit has to move inside its nibble) is the whole expansion of eight rows.

// C tile of 128 x 128 per workgroup of 4 waves (2 x 2, each 64 x 64 = 2 x 2 MFMA tiles, 64 accumulator registers),
// four workgroups per compute unit, i.e. four waves per SIMD, each from a workgroup of its own.  A workgroup alternates
// between contracting (matrix cores) and writing its tile (memory); with equal demand on both, two workgroups per
// compute unit keep the busier of the two resources occupied two thirds of the time, four of them four fifths, and
// while one writes, every SIMD still has three waves feeding its matrix cores.  (Measured on one device with a model
// of this loop: two computing waves per SIMD run it at 69 % of the matrix cores' rate, one wave alone at 50 %.)
// The contraction runs in chunks of 128 trace rows (one 16-byte run word per entry).  Three stages, all in LDS:
//   raw ring   (RAW_DEPTH chunks)  the run words of the tile's 128 rows and 128 columns, loaded memory -> LDS directly
//              (buffer_load ... lds, 16 bytes per lane: one load per chunk and wave, no register ever holds data in
//              flight -- with four waves per SIMD there are none to spare for that)
//   row ring   (2 chunks)          the 128 rows expanded to 4-bit operands, thread t expands half of row t/2
//   fragments                      rows from the row ring (16-byte LDS reads), columns expanded in registers from the
//                                  lane's own 8 raw bytes per 32-column block
// One barrier per chunk hands over all three: before it a wave has waited for its own load of chunk d + 2, has written
// its share of chunk d + 1's rows and has read everything it needs of chunk d + 1's raw bits; after it the slot of
// chunk d + 1's raw bits is free for the load of chunk d + 1 + RAW_DEPTH, chunk d + 1's rows may be read, and the row
// buffer of chunk d may be overwritten (during chunk d + 1).
// Because the operands travel as bits, the small tile costs next to nothing in memory traffic.
// Workgroups are numbered so that the eight L2 slices (one per XCD, workgroups are dealt to them
// round-robin) each walk a contiguous run of the tile schedule.
// RHO (MODE 0): the epilogue also counts, for every row of C, the elements that reach the head's
// threshold cstar[h] (Algorithm 1, Step 3: the density of an entry is the number of entries within the
// radius, and "within the radius" is "count >= threshold", see the density pass).  A lane's register
// column of the direct tile gives the counts of the mirrored tile's rows, the mirrored tile's vectors
// give those of the direct tile's rows; a diagonal tile is computed in full, and by
// symmetry its column counts are its row counts.  Counts meet in LDS and leave as one
// atomic add per row and tile.
// FORM: STREAM (MODE 0) lets C leave in streaming stores, past the caches; STAGGER makes the workgroups of a compute unit finish
// one after the other; STAGGER | STREAM is both.  launch_coact_syrk says when.
// PART contracts one piece of the trace rows and leaves the tile's partial counts in `part`; FINISH adds a tile's pieces up in place
// of the contraction, a workgroup per wave of the other forms.
enum { PLAIN = 0, STREAM = 1, STAGGER = 2, PART = 4, FINISH = 8 };
typedef __attribute__((address_space(3))) void lds_void;

template <int MODE, bool RHO = false, int FORM = PLAIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void coact_syrk_kernel(const v4i* __restrict__ bits, int N, int Npad, int nruns, int32_t* __restrict__ C, uint32_t decay_q16,
                       int tiles_per_head, int total_tiles, int per_xcd, const int32_t* __restrict__ tile_order,
                       uint32_t* __restrict__ dev_flags, const int64_t* __restrict__ cstar, int32_t* __restrict__ rho,
                       v4f* __restrict__ part, int pieces, int piece_runs) {
    static_assert(!RHO || MODE == 0, "the fused density count belongs to the overwriting form");
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int xcd = blockIdx.x & 7, slot_id = blockIdx.x >> 3;
    // PART: the pieces of a tile one after the other, and per_xcd, total_tiles counts of pieces
    const int unit = FORM == FINISH ? blockIdx.x >> 2 : xcd * per_xcd + slot_id;
    if (FORM != FINISH && (slot_id >= per_xcd || unit >= total_tiles)) return;
    const int t = FORM == PART ? unit / pieces : unit;
    const int h = t / tiles_per_head;
    const int32_t packed = tile_order[t - h * tiles_per_head];
    const int ti = packed >> 16, tj = packed & 0xffff;       // tile row, tile column (tj >= ti)
    const bool diag = tj == ti;                              // a diagonal tile is computed in full: no mirror

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = FORM == FINISH ? (int)blockIdx.x & 3 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wy = wave >> 1, wx = wave & 1;
    const int frow = lane & 31, fhalf = lane >> 5;

    // memory -> raw ring.  A chunk's raw bits are 4 KiB, contiguous in memory in two pieces (rows, columns), and land in
    // LDS in the same order: waves 0 and 1 bring rows [64 w, +64) of the tile, waves 2 and 3 columns [64 (w - 2), +64); lane l
    // of a load carries 16 bytes to byte 16 l of the wave's KiB.  One buffer descriptor per run (its range is the run:
    // 16 Npad bytes), so an offset past the run would read zeros, not memory.
    const int first_run = FORM == PART ? (unit - t * pieces) * piece_runs : 0;
    const int runs = FORM == PART ? min(piece_runs, nruns - first_run) : nruns;        // even
    const char* panel = reinterpret_cast<const char*>(bits) + ((size_t)h * nruns + first_run) * Npad * 16;
    const uint32_t src_lane = (uint32_t)(((wave < 2 ? ti * TM + wave * 64 : tj * TN + (wave - 2) * 64) + lane) * 16);
    const int last_run = runs - 1;
    auto issue_load = [&](int run) __attribute__((always_inline)) {                   // clamped: a redundant reload past the end is harmless
        {
            const char* runp = panel + (size_t)min(run, last_run) * Npad * 16;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(runp), 0, Npad * 16, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(lds + RAW_BASE + (run % RAW_DEPTH) * RAW_CHUNK + wave * 1024), 16,
                                                     src_lane, 0, 0, 0);
        }
    };
    // raw ring -> registers.  Thread t owns half ahalf = t % 2 of row t / 2 of the row panel: 8 bytes, two pieces of 32 trace
    // rows.  Lane l of a fragment supplies row l % 32 with the contraction indices of lane half l / 32, and which 32 trace
    // rows of a chunk those are is free as long as both operands agree: k-step ks of lane half f is word 2 f + ks of the
    // run, so the two k-steps of a lane are 8 contiguous raw bytes.
    const int arow = tid >> 1, ahalf = tid & 1;
    const int rawa_off = RAW_BASE + arow * 16 + ahalf * 8;
    const int rawb_off = RAW_BASE + TM * 16 + (wx * 64 + frow) * 16 + fhalf * 8;
    v2i ba;                                        // raw bits of this thread's half row, next chunk
    v2i bw[2][2];                                  // raw column bits [chunk parity][column block] = {k-step 0, k-step 1}
    auto read_raw_a = [&](int run) __attribute__((always_inline)) {
        ba = *reinterpret_cast<const v2i*>(lds + (run % RAW_DEPTH) * RAW_CHUNK + rawa_off);
    };
    auto read_raw_b = [&](int set, int run) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) bw[set][j] = *reinterpret_cast<const v2i*>(lds + (run % RAW_DEPTH) * RAW_CHUNK + rawb_off + j * 512);
    };
    // registers -> row ring, in pieces of 16 contraction bytes (32 trace rows = one 32-bit word of the run).  A piece is
    // expanded one dword (8 trace rows) at a time and stored when complete.
    int st_off[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) st_off[p] = lds_off(arow, 2 * ahalf + p);
    v4i ex;
    // Row operand: the bit of trace row 8q + n of a 32-row word is bit q of nibble n, and for q = 0, 1, 2 it is left where
    // it is -- the nibbles 0b0001, 0b0010, 0b0100 are 0.5, 1 and 2 in E2M1 -- while the column operand (below) carries the
    // inverse factor at the same contraction index, so every product of two set bits is still exactly 1.  Only q = 3 (the
    // sign bit of its nibble) has to move.  Five vector operations per 32 trace rows instead of seven.
    auto expand_quarter = [&](int piece, int q) __attribute__((always_inline)) {
        const uint32_t w = (uint32_t)ba[piece];
        ex[q] = (int)(q == 3 ? (w >> 2) & 0x22222222u : w & (0x11111111u << q));
    };
    auto store_piece = [&](int buf, int piece) __attribute__((always_inline)) {
        *reinterpret_cast<v4i*>(lds + buf * A_BYTES + st_off[piece]) = ex;
    };

    v16f facc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) facc[i][j][r] = 0.f;

    // A fragment addressing: lane l reads row l%32 of an MFMA tile, the 16-byte piece 2 (l/32) + ks of its row.
    // The swizzle term is the same for rows 32 apart; the tile index is a constant byte offset.
    int fa_base[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fa_base[ks] = lds_off(wy * 64 + frow, 2 * fhalf + ks);
    v4i fa[2][2], fb[2];
    auto read_a = [&](int buf, int ks, int fs, int i) __attribute__((always_inline)) {
        fa[fs][i] = *reinterpret_cast<const v4i*>(lds + buf * A_BYTES + fa_base[ks] + i * 32 * KC);
    };
    // Column operand: 2, 1, 0.5 and 1 at q = 0, 1, 2, 3, the inverses of the row operand's factors (two shifts, four masks).
    // One set of fragment registers: a k-step's columns are expanded after the previous k-step's MFMAs have been issued.
    auto expand_b = [&](int set, int ks, int j) __attribute__((always_inline)) {
        const uint32_t w = (uint32_t)bw[set][j][ks], w2 = w >> 2;
        fb[j] = v4i{(int)((w << 2) & 0x44444444u), (int)(w & 0x22222222u), (int)(w2 & 0x11111111u), (int)(w2 & 0x22222222u)};
    };
    // no block scales: with both scales 0 the compiler emits the unscaled form of the instruction (scale 2^0)
    auto mfma = [&](int fs, int m) __attribute__((always_inline)) {
        const v4i a4 = fa[fs][m >> 1], b4 = fb[m & 1];
        const v8i a8 = {a4.x, a4.y, a4.z, a4.w, 0, 0, 0, 0}, b8 = {b4.x, b4.y, b4.z, b4.w, 0, 0, 0, 0};   // the 4-bit form reads 4 registers
        facc[m >> 1][m & 1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, facc[m >> 1][m & 1], 4, 4, 0, 0, 0, 0);
    };

    if constexpr (FORM != FINISH) {
    // start-up: chunks 0 .. RAW_DEPTH-1 on their way; chunk 0 expanded; chunk RAW_DEPTH into the slot of chunk 0
#pragma unroll
    for (int c = 0; c < RAW_DEPTH; ++c) issue_load(c);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    read_raw_a(0);
    read_raw_b(0, 0);
#pragma unroll
    for (int piece = 0; piece < 2; ++piece) {
#pragma unroll
        for (int q = 0; q < 4; ++q) expand_quarter(piece, q);
        store_piece(0, piece);
    }
    __syncthreads();
    issue_load(RAW_DEPTH);
#pragma unroll
    for (int i = 0; i < 2; ++i) read_a(0, 0, 0, i);
#pragma unroll
    for (int j = 0; j < 2; ++j) expand_b(0, 0, j);

    // Chunk d (parity `set`, passed as a literal) computes out of row buffer `set`.  First k-step: its four MFMAs, between
    // them the row fragments of the second k-step and this thread's share of chunk d + 1's rows (raw bits read at the top of
    // the chunk: they were published by the previous barrier); then the columns of the second k-step; the barrier; the load
    // of chunk d + 1 + RAW_DEPTH; the first row fragments of chunk d + 1, whose LDS latency the second k-step's MFMAs and
    // the SIMD's other waves cover; the columns of chunk d + 1's first k-step.
    auto chunk_body = [&](int d, int set) __attribute__((always_inline)) {
        const int nset = set ^ 1;
        read_raw_a(d + 1);
        read_raw_b(nset, d + 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            mfma(0, s);
            if (s < 2) read_a(set, 1, 1, s);
#pragma unroll
            for (int u = 2 * s; u < 2 * (s + 1); ++u) {
                expand_quarter(u >> 2, u & 3);
                if ((u & 3) == 3) store_piece(nset, u >> 2);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) expand_b(set, 1, j);
        // this wave's load of chunk d + 2 has landed; the RAW_DEPTH - 2 younger ones may still be in flight
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(RAW_DEPTH - 2) : "memory");
        __syncthreads();
        issue_load(d + 1 + RAW_DEPTH);
#pragma unroll
        for (int i = 0; i < 2; ++i) read_a(nset, 0, 0, i);            // after the last chunk this reads stale but valid LDS and is never used
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) mfma(1, s);
#pragma unroll
        for (int j = 0; j < 2; ++j) expand_b(nset, 0, j);
    };
    // The contraction outranks the other waves' epilogue stores.  STAGGER: of the workgroups that share a compute unit (an XCD's
    // workgroups are dealt to its 32 compute units in turn) each outranks the later ones.
    if constexpr ((FORM & STAGGER) != 0) {
        switch ((slot_id >> 5) & 3) {
            case 0: __builtin_amdgcn_s_setprio(3); break;
            case 1: __builtin_amdgcn_s_setprio(2); break;
            case 2: __builtin_amdgcn_s_setprio(1); break;
            default: __builtin_amdgcn_s_setprio(0);
        }
    } else {
        __builtin_amdgcn_s_setprio(2);
    }
    for (int d = 0; d < runs; d += 2) {                     // nruns is a multiple of 4
        chunk_body(d, 0);
        chunk_body(d + 1, 1);
    }
    // every load has landed before the staging below reuses the rings, and every wave has left the loop
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    __builtin_amdgcn_s_setprio(0);
    }
    if constexpr (FORM == PART) {
        v4f* out = part + ((size_t)unit * SYRK_WAVES + wave) * (16 * 64) + lane;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    out[((i * 2 + j) * 4 + q) * 64] = v4f{facc[i][j][4 * q], facc[i][j][4 * q + 1], facc[i][j][4 * q + 2], facc[i][j][4 * q + 3]};
        return;
    }
    if constexpr (FORM == FINISH) {
        // sums of integers up to 2^24: exact in any order
        for (int p = 0; p < pieces; ++p) {
            const v4f* in = part + (((size_t)t * pieces + p) * SYRK_WAVES + wave) * (16 * 64) + lane;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v4f v = in[((i * 2 + j) * 4 + q) * 64];
#pragma unroll
                        for (int r = 0; r < 4; ++r) facc[i][j][4 * q + r] += v[r];
                    }
        }
    }
    // 32x32 result layout: lane l, register r -> column l%32, row 8*(r/4) + 4*(l/32) + r%4.  One
    // register of a wave is therefore two whole 128-byte lines of the direct tile (32 consecutive
    // columns of two rows): the direct tile leaves straight from the accumulators in 4-byte stores,
    // with nothing to wait for.  In the mirrored tile a lane's register quadruple is 16 contiguous
    // bytes but the lines are spread over lanes, so that tile is re-laid out through the (now idle)
    // LDS and leaves in 16-byte stores that cover whole lines.
    // the counts as integers (exact: every partial sum is an integer below 2^24)
    v16i acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = (int32_t)facc[i][j][r];
    int32_t* Ch = C + (size_t)h * N * N;
    const int col_in = lane & 31, half = lane >> 5, row_in = half * 4;
    int8_t* tbuf = lds + (FORM == FINISH ? 0 : wave * (32 * TROW));
    const int gi_base = ti * TM + wy * 64;
    const int mrow = lane >> 4, c16 = lane & 15;             // mirrored tile: a store covers 4 rows of 64 columns, 16 bytes per lane
    // Addresses are a wave-uniform row pointer (scalar arithmetic) plus one per-lane element offset
    // that is the same for every store of a tile.
    // The lane part is a 32-bit BYTE offset, so that an access is "scalar base + 32-bit lane offset", the
    // addressing form that needs no per-store 64-bit vector arithmetic and no register pair per address.
    const uint32_t lane_direct = ((uint32_t)row_in * (uint32_t)N + col_in) * 4u;
    const uint32_t lane_mirror = ((uint32_t)mrow * (uint32_t)N + c16 * 4) * 4u;
    auto at = [](int32_t* base, uint32_t byte_off) __attribute__((always_inline)) {
        return reinterpret_cast<int32_t*>(reinterpret_cast<char*>(base) + byte_off);
    };
    // density counters behind everything else in LDS: 128 direct-tile rows, then 128 direct-tile columns
    uint32_t* cnt_row = reinterpret_cast<uint32_t*>(lds + (FORM == FINISH ? 32 * TROW : SYRK_LDS_BYTES));
    uint32_t* cnt_col = cnt_row + TM;
    int32_t c32 = 0x7fffffff;                              // counts never reach it (rows <= 2^24): "nothing is within the radius"
    if (RHO) {
        const int64_t c = cstar[h];
        if (c < 0x7fffffffll) c32 = (int32_t)c;
        for (int u = threadIdx.x; u < TM + TN; u += FORM == FINISH ? 64 : 256) cnt_row[u] = 0u;       // the columns' lie behind the rows'
        __syncthreads();                                   // the waves' counts meet in these counters
    }
    // 1 where v >= c32, 0 elsewhere, without a compare: counts lie in [0, 2^24] and c32 in [0, 2^31), so
    // (c32 - 1) - v cannot wrap and is negative exactly when v >= c32 (plain arithmetic: the compare form
    // kept its lane masks in scalar registers until those ran out)
    const int32_t c32m1 = c32 - 1;
    auto reaches = [&](int32_t v) __attribute__((always_inline)) { return (uint32_t)(c32m1 - v) >> 31; };
    uint32_t rowc[4] = {0u, 0u, 0u, 0u};
    bool ovf = false;
    auto combine = [&](int32_t old, int32_t v) __attribute__((always_inline)) {
        return updated_count<MODE == 0 ? 1 : MODE>(old, v, decay_q16, ovf);
    };
    auto put = [](int32_t v, int32_t* p) __attribute__((always_inline)) {
        if (FORM & STREAM) __builtin_nontemporal_store(v, p);
        else *p = v;
    };
    // four consecutive counts of a row, `cols` of them inside C (four unless the tile reaches past N)
    auto load_row = [](const int32_t* p, int cols) __attribute__((always_inline)) {
        if (cols >= 4) return (v4i) *reinterpret_cast<const v4i_row*>(p);
        return v4i{p[0], cols > 1 ? p[1] : 0, cols > 2 ? p[2] : 0, 0};
    };
    auto store_row = [](int32_t* p, v4i w, int cols) __attribute__((always_inline)) {
        if (cols >= 4) {
            if (FORM & STREAM) __builtin_nontemporal_store((v4i_row)w, reinterpret_cast<v4i_row*>(p));
            else *reinterpret_cast<v4i_row*>(p) = w;
        } else {
            p[0] = w.x;
            if (cols > 1) p[1] = w.y;
            if (cols > 2) p[2] = w.z;
        }
    };
    // GUARD: the tile reaches past N (only tiles of the last tile row / column when N is not a multiple of 128)
    auto emit = [&](auto guard_tag) __attribute__((always_inline)) {
        constexpr bool GUARD = decltype(guard_tag)::value;
        const int gj_wave = tj * TN + wx * 64;                                        // the wave's 64 x 64 block: rows gi_base.., columns gj_wave..
        if constexpr (MODE == 0) {
            // The direct tile first, the two 32-column blocks of a row back to back, so that the two
            // 128-byte halves of a 256-byte run reach the memory system together.
            int32_t* Cd = Ch + (size_t)gi_base * N + gj_wave;                         // wave-uniform
            const bool c0_ok = !GUARD || gj_wave + col_in < N, c1_ok = !GUARD || gj_wave + 32 + col_in < N;
            uint32_t colc0 = 0u, colc1 = 0u;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int urow = i * 32 + (r >> 2) * 8 + (r & 3);
                    int32_t* p = Cd + (size_t)urow * N;
                    if (!GUARD || gi_base + urow + row_in < N) {
                        if (c0_ok) put(acc[i][0][r], at(p, lane_direct));
                        if (c1_ok) put(acc[i][1][r], at(p + 32, lane_direct));
                        if (RHO && c0_ok) colc0 += reaches(acc[i][0][r]);
                        if (RHO && c1_ok) colc1 += reaches(acc[i][1][r]);
                    }
                }
            if (RHO) {
                atomicAdd(&cnt_col[wx * 64 + col_in], colc0);
                atomicAdd(&cnt_col[wx * 64 + 32 + col_in], colc1);
            }
        }
        // A block of 32 rows x 64 columns of C goes through the wave's LDS staging as rows: eight accesses of 16 bytes per
        // lane, each covering four rows.  The old counts are requested before the block is parked.
        auto row_block = [&](auto park, int grow, int gcol) __attribute__((always_inline)) {
            size_t off = (size_t)grow * N + gcol;                                     // wave-uniform
            if (RHO) asm volatile("" : "+s"(off));
            int32_t* Cb = Ch + off;
            const int cols = GUARD ? N - gcol - c16 * 4 : 4;                          // columns of this lane's vector inside C
            auto inside = [&](int s) __attribute__((always_inline)) { return !GUARD || (cols > 0 && grow + 4 * s + mrow < N); };
            v4i old[8];
            if (MODE != 0) {
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    if (inside(s)) old[s] = load_row(at(Cb + (size_t)(4 * s) * N, lane_mirror), cols);
            }
            park();
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                v4i w = *reinterpret_cast<const v4i*>(tbuf + (4 * s + mrow) * TROW + c16 * 16);
                if (inside(s)) {
                    if (RHO) {
                        // columns past N hold counts of padding entries; their counters are dropped
                        rowc[0] += reaches(w.x); rowc[1] += reaches(w.y); rowc[2] += reaches(w.z); rowc[3] += reaches(w.w);
                    }
                    if (MODE != 0) {
                        w.x = combine(old[s].x, w.x); w.y = combine(old[s].y, w.y); w.z = combine(old[s].z, w.z); w.w = combine(old[s].w, w.w);
                    }
                    store_row(at(Cb + (size_t)(4 * s) * N, lane_mirror), w, cols);
                }
            }
            // the LDS executes one wave's accesses in order: the next block may be parked right away
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        };
        if constexpr (MODE != 0) {
            // read-modify-write: the direct tile as row blocks too
#pragma unroll
            for (int i = 0; i < 2; ++i)
                row_block([&]() __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            *reinterpret_cast<int32_t*>(tbuf + ((r >> 2) * 8 + row_in + (r & 3)) * TROW + (j * 32 + col_in) * 4) = acc[i][j][r];
                }, gi_base + i * 32, gj_wave);
        }
        if (!diag) {                                                                  // the mirrored tile, parked as [column][row]
#pragma unroll
            for (int j = 0; j < 2; ++j)
                row_block([&]() __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int rq = 0; rq < 4; ++rq) {
                            const v4i v = {acc[i][j][rq * 4], acc[i][j][rq * 4 + 1], acc[i][j][rq * 4 + 2], acc[i][j][rq * 4 + 3]};
                            *reinterpret_cast<v4i*>(tbuf + col_in * TROW + (i * 32 + rq * 8 + row_in) * 4) = v;
                        }
                }, gj_wave + j * 32, gi_base);
        }
    };
    if ((ti + 1) * TM <= N && (tj + 1) * TN <= N) emit(std::false_type{});   // whole tile inside C: no per-store checks
    else emit(std::true_type{});
    if (MODE != 0 && ovf) atomicOr(dev_flags, SWARM_DEV_OVERFLOW);
    if (RHO) {
        if (!diag) {
#pragma unroll
            for (int c = 0; c < 4; ++c) atomicAdd(&cnt_row[wy * 64 + c16 * 4 + c], rowc[c]);
        }
        __syncthreads();
        int32_t* rh = rho + (size_t)h * N;
        for (int u = threadIdx.x; u < TM + TN; u += FORM == FINISH ? 64 : 256) {
            if (!diag && u < TM && ti * TM + u < N && cnt_row[u]) atomicAdd(rh + ti * TM + u, (int32_t)cnt_row[u]);
            if (u >= TM && tj * TN + u - TM < N && cnt_col[u - TM]) atomicAdd(rh + tj * TN + u - TM, (int32_t)cnt_col[u - TM]);
        }
    }
}

// The same counts without the matrix cores: C[i][j] = sum over the trace's 32-bit words of
// popcount(bits_i & bits_j), on the plain vector ALUs (v_and + v_bcnt, which adds the popcount to
// its accumulator).  A cross-check of the matrix-core path by an independent route, and its
// competitor: an eighth of the LDS traffic per trace row, but 2 ALU operations per 32 products
// where the matrix cores do 65536 per instruction.
// Workgroup = 64 x 64 tile of C on or above the diagonal, thread = 4 x 4 outputs (rows ty + 16 i,
// columns tx + 16 j), eight runs of 128 trace rows staged in LDS per pass.
constexpr int PT = 64, PRUNS = 8;

template <int MODE>
__global__ __launch_bounds__(256) void coact_popcount_kernel(const v4i* __restrict__ bits, int N, int Npad, int nruns,
                                                             int32_t* __restrict__ C, uint32_t decay_q16,
                                                             uint32_t* __restrict__ dev_flags) {
    __shared__ v4i sa[PRUNS][PT], sb[PRUNS][PT];
    const int h = blockIdx.z, ti = blockIdx.y, tj = blockIdx.x;
    if (tj < ti) return;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const v4i* panel = bits + (size_t)h * nruns * Npad;
    uint32_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0u;
    for (int r0 = 0; r0 < nruns; r0 += PRUNS) {
        __syncthreads();
        for (int u = tid; u < PRUNS * PT; u += 256) {
            const int r = r0 + u / PT, e = u % PT;
            const v4i zero = {0, 0, 0, 0};
            sa[u / PT][e] = r < nruns ? panel[(size_t)r * Npad + ti * PT + e] : zero;
            sb[u / PT][e] = r < nruns ? panel[(size_t)r * Npad + tj * PT + e] : zero;
        }
        __syncthreads();
#pragma unroll 2
        for (int r = 0; r < PRUNS; ++r) {
            v4i a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = sa[r][ty + 16 * i]; b[i] = sb[r][tx + 16 * i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] += __popc((uint32_t)(a[i].x & b[j].x)) + __popc((uint32_t)(a[i].y & b[j].y)) +
                                 __popc((uint32_t)(a[i].z & b[j].z)) + __popc((uint32_t)(a[i].w & b[j].w));
        }
    }
    int32_t* Ch = C + (size_t)h * N * N;
    bool ovf = false;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int gi = ti * PT + ty + 16 * i, gj = tj * PT + tx + 16 * j;
            if (gi >= N || gj >= N) continue;
            const int32_t v = (int32_t)acc[i][j];
            int32_t* p = Ch + (size_t)gi * N + gj;
            int32_t* q = Ch + (size_t)gj * N + gi;
            if (MODE == 0) { *p = v; if (ti != tj) *q = v; }
            else {
                *p = updated_count<MODE == 0 ? 1 : MODE>(*p, v, decay_q16, ovf);
                if (ti != tj) *q = updated_count<MODE == 0 ? 1 : MODE>(*q, v, decay_q16, ovf);
            }
        }
    if (MODE != 0 && ovf) atomicOr(dev_flags, SWARM_DEV_OVERFLOW);
}

}  // namespace

// Entries per trace-building workgroup.  A workgroup scans all selections of its run whatever its span, so spans are as
// long as they can be while there is a workgroup for every compute unit: a window of 256 steps over 8 heads of 8192
// entries takes 16.5 us as 16 workgroups and 6.5 us as 256; four workgroups per compute unit cost 24 against 16.5 us on
// 4096 steps (256 against 512 or 1024 threads each: 20 and 17 against 16.5 us).
static int trace_span(int nruns, int H, int Npad) {
    int span = TRACE_SPAN;
    while (span > TRACE_SPAN_MIN && (int64_t)nruns * H * ((Npad + span - 1) / span) < 256) span /= 2;
    return span;
}

int trace_slabs(int nruns, int H, int Npad) {
    const int span = trace_span(nruns, H, Npad);
    return (Npad + span - 1) / span;
}

// Room for the builder's row counts.  Their number, runs x heads x slabs, does not grow with the shape: shorter spans make more
// slabs.  But the spans are halved only while there are fewer than 256 workgroups, so it is either the number at full spans or
// below 512, and the larger of the two bounds grows with every argument.
size_t trace_count_words(int nruns, int H, int Npad) {
    const size_t full = (size_t)nruns * H * ((Npad + TRACE_SPAN - 1) / TRACE_SPAN);
    return (full > 512 ? full : 512) * 128;
}

swarm_status launch_trace_build(swarm_ctx* ctx, const int32_t* idx, int64_t rows, int H, int k, int N, int Npad,
                                int nruns, uint32_t flags, int32_t* row_count, int32_t* rho) {
    if (flags & SWARM_CHECK_IDX) {
        hipLaunchKernelGGL(check_distinct_kernel, dim3((unsigned)(rows * H)), dim3(256), 0, ctx->stream, idx, k,
                           ctx->dev_flags);
        const swarm_status st = swarm_check_launch(ctx, "check_distinct_kernel");
        if (st != SWARM_OK) return st;
    }
    using kernel_t = void (*)(const int32_t*, int64_t, int, int, int, int, int, int, uint32_t, uint4*, uint32_t*, int32_t*, int32_t*);
    static const kernel_t kernels[2][2] = {{trace_build_kernel<false, false>, trace_build_kernel<false, true>},
                                           {trace_build_kernel<true, false>, trace_build_kernel<true, true>}};
    if (!ctx->trace_lds_opt_in) {                          // per context: the attribute belongs to the device the context is bound to
        for (int c = 0; c < 2; ++c)
            for (int v = 0; v < 2; ++v) {
                const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernels[c][v]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         TRACE_SPAN * 16 + 512);
                if (e != hipSuccess) {
                    snprintf(ctx->err, sizeof(ctx->err), "coact: cannot opt in to %d bytes of LDS: %s", TRACE_SPAN * 16 + 512, hipGetErrorString(e));
                    return SWARM_EHIP;
                }
            }
        ctx->trace_lds_opt_in = true;
    }
    const int span = trace_span(nruns, H, Npad);
    const bool vec = (k & 3) == 0 && (reinterpret_cast<uintptr_t>(idx) & 15) == 0;
    const uint64_t kq = (uint64_t)(vec ? k / 4 : k);
    // ceil(2^32 / kq) divides every list position below 128 kq exactly as long as 128 kq^2 < 2^32; otherwise the kernel divides
    const uint32_t reciprocal = kq > 1 && 128 * kq * kq < (1ull << 32) ? (uint32_t)(((1ull << 32) + kq - 1) / kq) : 0u;
    const dim3 grid((unsigned)nruns, (unsigned)H, (unsigned)((Npad + span - 1) / span));
    const size_t lds_bytes = (size_t)(Npad < span ? Npad : span) * 16 + (row_count ? 512 : 0);
    hipLaunchKernelGGL(kernels[row_count ? 1 : 0][vec ? 1 : 0], grid, dim3(TRACE_THREADS), lds_bytes, ctx->stream, idx, rows, H, k, N, Npad, nruns, span,
                       reciprocal, reinterpret_cast<uint4*>(ctx->trace), ctx->dev_flags, row_count, rho);
    return swarm_check_launch(ctx, "trace_build_kernel");
}

// Order in which the tiles on or above the diagonal are handed out: super-blocks of 8 x 16 tiles
// (1024 x 2048 entries), so that the workgroups resident on one XCD share few panels in its L2.
// Tile (ti, tj) covers rows [128 ti, +128) and columns [128 tj, +128), tj >= ti.
static swarm_status tile_order_for(swarm_ctx* ctx, int ntm, const int32_t** out) {
    for (const auto& t : ctx->tile_orders)
        if (t.first == ntm) { *out = t.second; return SWARM_OK; }
    if (ctx->capturing) {
        snprintf(ctx->err, sizeof(ctx->err), "coact: first call with this N while recording; run the sequence once first");
        return SWARM_EINVAL;
    }
    const size_t count = (size_t)ntm * (ntm + 1) / 2;
    int32_t* host = static_cast<int32_t*>(malloc(count * sizeof(int32_t)));
    if (!host) {
        snprintf(ctx->err, sizeof(ctx->err), "out of host memory");
        return SWARM_ENOMEM;
    }
    size_t n = 0;
    for (int bi = 0; bi < ntm; bi += 8)
        for (int bj = bi / 16 * 16; bj < ntm; bj += 16)
            for (int ti = bi; ti < bi + 8 && ti < ntm; ++ti)
                for (int tj = (bj > ti ? bj : ti); tj < bj + 16 && tj < ntm; ++tj)
                    if (n < count) host[n++] = (ti << 16) | tj; else ++n;
    swarm_status st = SWARM_OK;
    int32_t* dev = nullptr;
    if (n != count) {
        snprintf(ctx->err, sizeof(ctx->err), "coact: tile order covers %zu of %zu tiles", n, count);
        st = SWARM_EINVAL;
    }
    if (st == SWARM_OK) {
        hipError_t e = hipMalloc(reinterpret_cast<void**>(&dev), count * sizeof(int32_t));
        if (e == hipSuccess) e = hipMemcpyAsync(dev, host, count * sizeof(int32_t), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e == hipSuccess) {
            try {
                ctx->tile_orders.emplace_back(ntm, dev);
            } catch (...) {
                e = hipErrorOutOfMemory;
            }
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            snprintf(ctx->err, sizeof(ctx->err), "coact: tile order set-up failed: %s", hipGetErrorString(e));
            if (dev) (void)hipFree(dev);
            st = SWARM_EHIP;
        }
    }
    free(host);
    *out = dev;
    return st;
}

// Whether the trace rows are contracted in pieces: so many that they fill the device, of 24 runs or more (8 to 32 measured alike),
// and only where the rows saved outweigh the partial counts (64 KiB a piece, written and read) and the second launch.  Whole and in
// pieces, decayed updates: 36 tiles, 4096 rows 20.2 and 20.7 us, 8192 30.7 and 26.0, 16384 51.7 and 30.4; 136 tiles, 8192 rows 34 and 33,
// 11000 42.9 and 34.7, 16384 55 and 40; 300 tiles, 12000 rows 65 and 66, 16384 75.7 and 71.7, 33000 130 and 104.  Overwriting: 36 tiles,
// 6144 rows 22.7 and 19.9, 8192 28.0 and 24.4; 136 tiles, 8192 rows 30 and 35 (left whole), 11000 38.6 and 34.4; 300 tiles, 33000 rows 122
// and 89.  With the density count 36 tiles, 6144 rows 34.4 and 32.3; 136 tiles, 11000 rows 61 and 58; 300 tiles, 33000 rows 154 and 124.
static bool split_rows(int64_t total, int nruns, int* pieces, int* piece_runs) {
    constexpr int MIN_RUNS = 24;
    if (total + 32 > 2 * (int64_t)nruns) return false;
    const int64_t fill = 1024 / total, most = fill < nruns / MIN_RUNS ? fill : nruns / MIN_RUNS;
    if (most < 2) return false;
    *piece_runs = (int)((nruns + 2 * most - 1) / (2 * most)) * 2;         // even
    *pieces = (nruns + *piece_runs - 1) / *piece_runs;                    // none of them empty
    return *pieces > 1;
}

// Whether a C that is not read leaves past the caches.  Cached, its lines push the trace out of them, a C larger than the last-level
// cache (256 MiB) all the more; streamed, it is on its way to memory from the first tile on, at the rate of the memory.  Times below in
// us, streamed and cached.
//  - Rows of C in whole 64-byte pieces: streamed (8 x 8192^2, 4096 rows 434 and 650; 2 x 2048^2, 2048 rows 17.3 and 19.0), but cached from
//    128 to 256 MiB where the trace leaves it room, C and twice the trace up to 278 MiB (8 x 2048^2, 2048 rows 42.6 and 37.5, 6144 rows
//    62.9 and 60.6; 60 x 1024^2, 2048 rows 63.4 and 60.6, 6144 rows 96 and 105, 16384 rows 230 and 273; 160 x 512^2, 2048 rows 49.5 and
//    47.6, 6144 rows 89 and 100; 600 x 256^2, 2048 rows 62.8 and 61.5, 6144 rows 140 and 177).
//  - Staggered, its writing lies beside the contraction of others, and the trace counts for more: cached from 80 MiB (20 << 20 counts) up
//    to 230 MiB of C and twice the trace (8 x 2048^2, 2048 rows 40.2 and 34.3, 16384 rows 116 and 118; 103 x 512^2, 2048 rows 40.0 and
//    38.2, 16384 rows 147 and 167; 400 x 256^2, 2048 rows 47.1 and 45.4, 6144 rows 94 and 105; 103 x 304^2, 2048 rows 37.1 and 38.2).
//  - Rows that start inside a 64-byte piece share it with their neighbour tiles, and streamed, each of the two writes it to memory by
//    itself: cached, except where the trace takes 64 MiB (90 x 700^2, 6144 rows 105 and 103, 16384 rows 231 and 263; 300 x 301^2, 6144
//    rows 163 and 177) or C is larger than the last-level cache and the contraction takes about as long as writing twice (8 x 4001^2,
//    6144 rows 268 and 209, 10240 rows 266 and 281; 12290^2, 6144 rows 291 and 247, 10240 rows 299 and 317), half as long where the
//    product of C and trace says that little of either stays (4 x 8190^2, 2048 rows 476 and 364, 6144 rows 440 and 502; 60 x 1500^2, 2048
//    rows 238 and 191, 6144 rows 232 and 302).  A small C of whole 16-byte vectors is better streamed (64 x 300^2, 2048 rows 25.7 and 26.9).
// Where C itself starts is not looked at: one of N % 16 == 0 that starts inside a piece is streamed like the others of its size.
static bool streams(int64_t elements, int N, int64_t trace_bytes, int64_t total, int nruns, bool stagger) {
    constexpr int64_t MIB = 1 << 20;
    const int64_t c_bytes = elements * 4, both = c_bytes + 2 * trace_bytes;
    if (N % 16 == 0) {
        if (stagger) return elements < 20 * MIB || both > 230 * MIB;
        return elements < 32 * MIB || elements > 64 * MIB || both > 278 * MIB;
    }
    if (N % 4 == 0 && elements < 8 * MIB) return true;
    if (c_bytes <= 256 * MIB) return trace_bytes >= 64 * MIB;
    const double contraction = 347.0 * total * nruns / elements;          // its time over that of writing C twice
    return contraction >= 0.85 || (contraction >= 0.45 && (double)c_bytes * trace_bytes >= 1.31e16);
}

swarm_status coact_reserve_tiles(swarm_ctx* ctx, int Npad) {
    if (swarm_capturing(ctx) || Npad / TM > 65535) return SWARM_OK;
    const int32_t* order;
    return tile_order_for(ctx, Npad / TM, &order);
}

// cstar and rho both null: plain update of C.  Both given (overwriting form only): the
// epilogue adds to rho[h][i] the number of elements of row i that reach cstar[h]; rho must be zero.
swarm_status launch_coact_syrk(swarm_ctx* ctx, int H, int N, int Npad, int nruns, int32_t* C, uint32_t decay_q16,
                               const int64_t* cstar, int32_t* rho) {
    const int ntm = Npad / TM;
    const int64_t tiles_per_head = (int64_t)ntm * (ntm + 1) / 2;
    const int64_t total = tiles_per_head * H;
    if (total > (int64_t)1 << 30 || ntm > 65535) {
        snprintf(ctx->err, sizeof(ctx->err), "coact: N=%d, H=%d give too many tiles for one launch", N, H);
        return SWARM_EINVAL;
    }
    const int32_t* tile_order = nullptr;
    swarm_status st = tile_order_for(ctx, ntm, &tile_order);
    if (st != SWARM_OK) return st;
    const int per_xcd = (int)((total + 7) / 8);
    const int mode = decay_q16 == 0u ? 0 : decay_q16 == 65536u ? 1 : 2;
    const bool fused = cstar != nullptr;
    if (fused && (!rho || mode != 0)) {
        snprintf(ctx->err, sizeof(ctx->err), "coact: the fused density count needs the overwriting form");
        return SWARM_EINVAL;
    }
    using kernel_t = void (*)(const v4i*, int, int, int, int32_t*, uint32_t, int, int, int, const int32_t*, uint32_t*,
                              const int64_t*, int32_t*, v4f*, int, int);
    static const kernel_t kernels[5][4] = {
        {coact_syrk_kernel<0>, coact_syrk_kernel<1>, coact_syrk_kernel<2>, coact_syrk_kernel<0, true>},
        {coact_syrk_kernel<0, false, STREAM>, coact_syrk_kernel<1>, coact_syrk_kernel<2>, coact_syrk_kernel<0, true, STREAM>},
        {coact_syrk_kernel<0, false, STAGGER>, coact_syrk_kernel<1, false, STAGGER>, coact_syrk_kernel<2, false, STAGGER>,
         coact_syrk_kernel<0, true, STAGGER>},
        {coact_syrk_kernel<0, false, STAGGER | STREAM>, coact_syrk_kernel<1, false, STAGGER>, coact_syrk_kernel<2, false, STAGGER>,
         coact_syrk_kernel<0, true, STAGGER | STREAM>},
        {coact_syrk_kernel<0, false, FINISH>, coact_syrk_kernel<1, false, FINISH>, coact_syrk_kernel<2, false, FINISH>,
         coact_syrk_kernel<0, true, FINISH>}};
    static const kernel_t part_kernel = coact_syrk_kernel<0, false, PART>;
    constexpr int RHO_LDS_BYTES = SYRK_LDS_BYTES + (TM + TN) * 4;
    if (!ctx->syrk_lds_opt_in) {
        hipError_t e = hipSuccess;
        for (int f = 0; f < 4; ++f)
            for (int m = 0; m < 4 && e == hipSuccess; ++m)
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernels[f][m]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        m == 3 ? RHO_LDS_BYTES : SYRK_LDS_BYTES);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(part_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, SYRK_LDS_BYTES);
        if (e != hipSuccess) {
            snprintf(ctx->err, sizeof(ctx->err), "coact: cannot opt in to %d bytes of LDS: %s", RHO_LDS_BYTES, hipGetErrorString(e));
            return SWARM_EHIP;
        }
        ctx->syrk_lds_opt_in = true;
    }
    // A little more than the 1024 tiles that the device holds at once: all of those contract together, then all write, and the rest
    // runs nearly alone.  One after the other, the first ones' writing and the rest's start overlap the others' contraction: 16384
    // rows of 8 x 2048 (1088 tiles) 126 -> 114 us without the trace, of 1 x 6000 (1176) 142 -> 130 with it, of 8 x 2304 (1368)
    // 170 -> 167.  Nothing below (1012 tiles 101.2 -> 101.7), and past 1.4 rounds it is in the way (1680 tiles 213 -> 226), as it is where
    // there is little to contract or to write (342 x 64^2 decayed, 512 rows 19.0 -> 19.9, 2048 rows 43.2 -> 44.4, 4096 rows 66.7 -> 65.8;
    // 345 x 100^2, 128 rows 21.9 and 21.9).
    const int64_t elements = (int64_t)H * N * N;
    const bool stagger = total > 1024 && total <= 1408 && (nruns >= 32 || elements >= (int64_t)1 << 21);
    const bool stream = streams(elements, N, (int64_t)H * nruns * Npad * 16, total, nruns, stagger);
    const int form = (stagger ? STAGGER : PLAIN) | (stream ? STREAM : PLAIN);       // rows of `kernels`
    // Few tiles over many trace rows leave most of the device idle: the rows are cut into pieces.
    int pieces = 1, piece_runs = nruns;
    if (split_rows(total, nruns, &pieces, &piece_runs)) {
        bool there;
        st = swarm_try_grow(ctx, &ctx->part, &ctx->part_bytes, (size_t)total * pieces * (TM * TN * sizeof(float)), &there);
        if (st != SWARM_OK) return st;
        if (!there) pieces = 1;
    }
    if (pieces > 1) {
        const int units = (int)total * pieces, units_xcd = (units + 7) / 8;
        v4f* part = static_cast<v4f*>(ctx->part);
        hipLaunchKernelGGL(part_kernel, dim3((unsigned)(units_xcd * 8)), dim3(64 * SYRK_WAVES), SYRK_LDS_BYTES, ctx->stream,
                           reinterpret_cast<const v4i*>(ctx->trace), N, Npad, nruns, C, decay_q16, (int)tiles_per_head, units, units_xcd, tile_order,
                           ctx->dev_flags, nullptr, nullptr, part, pieces, piece_runs);
        hipLaunchKernelGGL(kernels[4][fused ? 3 : mode], dim3((unsigned)(total * SYRK_WAVES)), dim3(64), 32 * TROW + (TM + TN) * 4, ctx->stream,
                           reinterpret_cast<const v4i*>(ctx->trace), N, Npad, nruns, C, decay_q16, (int)tiles_per_head, (int)total, 0, tile_order,
                           ctx->dev_flags, cstar, rho, part, pieces, piece_runs);
        ctx->count_way = SWARM_WAY_DENSE_PIECES;
        return swarm_check_launch(ctx, "coact_syrk_kernel (pieces)");
    }
    dim3 grid((unsigned)(per_xcd * 8)), block(64 * SYRK_WAVES);
    const int tph = (int)tiles_per_head, tot = (int)total;
    hipLaunchKernelGGL(kernels[form][fused ? 3 : mode], grid, block, fused ? RHO_LDS_BYTES : SYRK_LDS_BYTES,
                       ctx->stream, reinterpret_cast<const v4i*>(ctx->trace), N, Npad, nruns, C, decay_q16, tph, tot, per_xcd,
                       tile_order, ctx->dev_flags, cstar, rho, nullptr, 1, nruns);
    ctx->count_way = stagger ? (stream && mode == 0 ? SWARM_WAY_DENSE_STAGGERED_STREAMED : SWARM_WAY_DENSE_STAGGERED)
                             : stream && mode == 0 ? SWARM_WAY_DENSE_STREAMED : SWARM_WAY_DENSE;
    return swarm_check_launch(ctx, "coact_syrk_kernel");
}

swarm_status launch_coact_popcount(swarm_ctx* ctx, int H, int N, int Npad, int nruns, int32_t* C, uint32_t decay_q16) {
    const unsigned nt = (unsigned)(Npad / PT);
    if (nt > 65535u || H > 65535) {
        snprintf(ctx->err, sizeof(ctx->err), "coact: N=%d, H=%d too large for the popcount route", N, H);
        return SWARM_EINVAL;
    }
    const dim3 grid(nt, nt, (unsigned)H), block(256);
    const v4i* bits = reinterpret_cast<const v4i*>(ctx->trace);
    if (decay_q16 == 0u) hipLaunchKernelGGL(coact_popcount_kernel<0>, grid, block, 0, ctx->stream, bits, N, Npad, nruns, C, decay_q16, ctx->dev_flags);
    else if (decay_q16 == 65536u) hipLaunchKernelGGL(coact_popcount_kernel<1>, grid, block, 0, ctx->stream, bits, N, Npad, nruns, C, decay_q16, ctx->dev_flags);
    else hipLaunchKernelGGL(coact_popcount_kernel<2>, grid, block, 0, ctx->stream, bits, N, Npad, nruns, C, decay_q16, ctx->dev_flags);
    ctx->count_way = SWARM_WAY_POPCOUNT;
    return swarm_check_launch(ctx, "coact_popcount_kernel");
}
