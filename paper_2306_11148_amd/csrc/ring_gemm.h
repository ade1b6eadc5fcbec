// Blocked matrix-core contraction over conditioned "record tiles", shared by
// the split-BF16 and scaled-FP8 paths.
//
// Conditioned operands: for every row i of A and every column j of B, the k
// extent is cut into slabs (the sigma loop broken into blocks, section
// "Dimension Lifting to Machine Coordinates" of the paper) and slab s of that
// row becomes one 64-byte record. Records are stored in tiles of 16 rows x 1
// slab: record (r, s) lives at byte ((r / 16) * S + s) * 1024 + (r mod 16) * 64,
// so 16 records are one contiguous KiB of whole cache lines. Row counts are
// padded to a multiple of 16 with zero records. A path may keep NREC record
// arrays per operand (e.g. a high and a low term).
//
// Contraction (Fig. 2 blocking): a workgroup owns a BM x BN block of C and
// walks the S slabs; per slab the NREC*(BM+BN) records go straight from HBM
// into LDS (buffer_load ... lds, no register staging) through a ring of
// NSTAGE buffers, and the slab's block products are summed in registers (the
// "addition loop" over blocks). The fragments of slab s are read from LDS
// while the matrix-core steps of slab s - 1 issue and slab s + NSTAGE - 1 is
// on its way.
//
// LDS holds one 64-byte row per record. gfx950's LDS serves a 16-byte read for
// 16 lanes per cycle out of a 256-byte window (64 banks), i.e. four
// consecutive rows at once: chunk c of row r is stored at chunk position
// c ^ ((r / 4) mod 4), so the 16 rows of a read cycle hit 16 distinct bank
// groups. The direct loads stay linear (lane L writes bytes 16L .. 16L+15 of
// its wave's KiB window = 16 rows), so each lane fetches the logical chunk
// that belongs at its physical position.
#pragma once

#include <algorithm>
#include <type_traits>

#include "moa_internal.h"
#include "tile_common.h"

namespace moa {
namespace ring {

constexpr int REC_BYTES = 64;             // bytes per record
constexpr int GROUP = 16;                 // rows per record tile
constexpr int NSTAGE = 3;                 // default LDS ring depth (slabs in LDS at once)

__host__ __device__ inline int64_t padded_rows(int64_t rows) { return (rows + GROUP - 1) / GROUP * GROUP; }

// byte offset of record (r, s) in a record array with S slabs per row
__host__ __device__ inline int64_t rec_byte(int64_t r, int64_t s, int64_t S) {
    return ((r / GROUP) * S + s) * (GROUP * REC_BYTES) + (r % GROUP) * REC_BYTES;
}

// bytes of one record array for `rows` rows and S slabs
__host__ __device__ inline int64_t array_bytes(int64_t rows, int64_t S) { return padded_rows(rows) * S * REC_BYTES; }

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) float global_f32;
typedef __attribute__((address_space(1))) const int32_t global_i32;

// gfx9 s_waitcnt immediate: at most n vector-memory operations of this wave
// outstanding (expcnt and lgkmcnt not waited on).
constexpr int waitcnt_vm(int n) { return (n & 0xF) | (((n >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8); }

// Workgroup barrier without the release fence of __syncthreads(): that fence
// would also wait for the direct loads still in flight for later slabs. Each
// wave first waits (s_waitcnt) for its own loads of the slab it is about to
// read and for its LDS reads of the slot about to be refilled. The "memory"
// clobber keeps the compiler from moving LDS accesses across the barrier.
__device__ __forceinline__ void ring_barrier() { asm volatile("s_barrier" ::: "memory"); }

template <int BM, int BN, int WM, int WN, int NREC, int NST = NSTAGE> struct Cfg {
    static constexpr int WAVES_M = BM / WM, WAVES_N = BN / WN, NW = WAVES_M * WAVES_N;
    static constexpr int THREADS = NW * 64;
    static constexpr int FM = WM / 32, FN = WN / 32;
    static constexpr int ROWS = NREC * (BM + BN);         // records per slab
    static constexpr int STAGE = ROWS * REC_BYTES;        // bytes per LDS buffer
    static constexpr int LDS = NST * STAGE;
    static constexpr int LPW = ROWS / 16 / NW;            // KiB direct loads per wave per slab
    static_assert(ROWS % (16 * NW) == 0, "whole loads per wave");
    static_assert(NST >= 3 && (NST - 2) * LPW <= 63, "a slot being refilled, one being read, one landing; vmcnt");
    // load q of a slab is the same record array for every wave
    static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "whole loads per wave and array");
};

// Vector offset of a load that must touch no memory: beyond any resource
// range (records per resource stay below 2^31 bytes).
constexpr int kDeadVoffset = (int)0x80000000u;

// Where LDS row `row` of a slab comes from (rows: [A array 0 (BM)] ..
// [A array NREC-1] [B array 0 (BN)] ..): operand A or B, record array, the
// row's index inside the block's part of that array, the block's first row
// tile of the array and how many 16-row tiles of it exist from there (the
// block may overhang the padded end). Shared by the kernels and the host
// check of their loads (check_loads).
struct RowWindow {
    bool a;
    int arr, row_in, tiles;
    int64_t first_tile;
};
__host__ __device__ inline RowWindow row_window(int BM, int BN, int NREC, int row, int64_t i0, int64_t j0, int64_t m,
                                                int64_t p) {
    RowWindow w;
    w.a = row < NREC * BM;
    w.arr = NREC == 1 ? 0 : w.a ? row / BM : (row - NREC * BM) / BN;
    w.row_in = w.a ? row - w.arr * BM : row - NREC * BM - w.arr * BN;
    const int64_t org = w.a ? i0 : j0;
    const int64_t left = padded_rows(w.a ? m : p) - org;
    const int64_t span = w.a ? BM : BN;
    w.first_tile = org / GROUP;
    w.tiles = (int)((left < span ? left : span) / GROUP);
    return w;
}
// The conditioned operands of one product.
struct Operands {
    const uint8_t *a0, *a1;               // record arrays of A (a1 only when NREC == 2)
    const uint8_t *b0, *b1;               // record arrays of B
    float *C;
    const int32_t *row_exp;               // scaled modes: C[i][j] = 2^-(row_exp[i] + col_exp[j]) acc
    const int32_t *col_exp;
    int64_t m, p, S;
    int accumulate;
};

// Byte offset of logical chunk `chunk` of row `row` (of any 32-row group: 32
// rows further on the chunks lie alike).
__device__ __forceinline__ int chunk_at(int row, int chunk) {
    return row * REC_BYTES + ((chunk ^ ((row >> 2) & 3)) << 4);
}

// One BM x BN block of C at (i0, j0). Mode supplies
//   template <int FM, int FN> struct Frags         fragments of one slab
//   static int chunk(half, x)                      the two 16-byte chunks of a record that a lane reads
//   template <int BM, int BN, int FM, int FN>
//   static void read(a, b, at, Frags &)            LDS -> registers: chunk x of row r of the wave's part of A is
//                                                  at a + at[x] + r * REC_BYTES, of its part of B at b + ...
//   template <int FM, int FN> static void mma(const Frags &, acc)
//   static constexpr int TERMS                     matrix-core steps per pair of fragments
//   static constexpr bool SCALED                   apply row/col exponents
// and the LDS rows of a slab are [A array 0 (BM)] .. [A array NREC-1]
// [B array 0 (BN)] .. [B array NREC-1].
// `lds` is the workgroup's ring; on entry no wave may still be reading it, on
// exit every wave has finished.
// The k walk covers slabs s_begin .. s_end-1 (all slabs by default). With
// `partial` set, the epilogue stores the raw block sum there (row-major m x p,
// no descale, no accumulate): one chunk of a split-k product.
template <int BM, int BN, int WM, int WN, int NREC, class Mode, int NSTAGE = ring::NSTAGE>
__device__ __forceinline__ void tile(const Operands &op, int64_t i0, int64_t j0, uint8_t *lds, int s_begin = 0,
                                     int s_end = -1, float *partial = nullptr) {
#ifdef __HIP_DEVICE_COMPILE__           // the host pass would check the 16-byte direct loads against its own target
    using G = Cfg<BM, BN, WM, WN, NREC, NSTAGE>;
    constexpr int WAVES_N = G::WAVES_N, NW = G::NW, FM = G::FM, FN = G::FN;
    constexpr int STAGE = G::STAGE, LPW = G::LPW;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int S = (int)op.S;                 // the planner keeps S below 2^17
    const int s0 = s_begin;
    const int L = (s_end < 0 ? S : s_end) - s_begin;   // slabs this block walks

    // LDS rows of a slab: [A array 0 (BM)] .. [A array NREC-1] [B array 0 (BN)] ..
    // Load q of wave w: rows 16 (NW q + w) .. +15, so which array a load reads
    // is known at compile time, and its buffer resource (over the block's row
    // tiles of that array) is one of 2 NREC, uniform over the workgroup.
    static_assert(NREC == 1 || NREC == 2, "one or two record arrays per operand");
    const int64_t tile_row = S * GROUP * REC_BYTES;       // bytes per row tile (16 rows, all slabs)
    const int64_t m = op.m, p = op.p;
    RowWindow win[LPW];
    const uint8_t *src[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
        win[q] = row_window(BM, BN, NREC, NW * q * 16, i0, j0, m, p);
        const uint8_t *base = win[q].a ? (win[q].arr == 0 ? op.a0 : op.a1) : (win[q].arr == 0 ? op.b0 : op.b1);
        src[q] = base + win[q].first_tile * tile_row;
    }
    // lane L lands at row 16Q + L/4, physical chunk L%4, and fetches logical
    // chunk (L%4) ^ ((row/4) mod 4) = (L%4) ^ (L/16). Rows of the last
    // partial tile past m (or p) are zero records written by the conditioning.
    // A load whose whole 16-row tile lies past the padded end of its array
    // (the block overhangs the operand) gets the vector offset 2^31, beyond
    // the resource's range (below 2^31 bytes), so it touches no memory whether
    // or not the range check counts the scalar offset (below 2^31 too, so the
    // sum does not wrap); its LDS rows feed only outputs past m or p, which
    // are never stored.
    const int voff = (lane >> 2) * REC_BYTES + (((lane & 3) ^ (lane >> 4)) << 4);
    // The next slab into buf. Slabs past the last have empty ranges: their loads
    // touch no memory but keep the count of loads in flight.
    int next_slab = 0;                   // counts from s_begin
    auto issue_next = [&](uint8_t *buf) {
        const bool past = next_slab >= L;
        const int slab_at = (s0 + next_slab) * GROUP * REC_BYTES;
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            const int tile_in = win[q].row_in / GROUP + wave;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                __builtin_amdgcn_make_buffer_rsrc((void *)src[q], (short)0, past ? 0 : (int)(win[q].tiles * tile_row),
                                                  0x00020000),
                (lds_void_t *)(buf + (NW * q + wave) * 16 * REC_BYTES), 16,
                tile_in < win[q].tiles ? voff : kDeadVoffset, (int)(tile_in * tile_row) + slab_at, 0, 0);
        }
        ++next_slab;
    };

    const int frow = lane & 31, fhalf = lane >> 5;
    const int at[2] = {chunk_at(frow, Mode::chunk(fhalf, 0)), chunk_at(frow, Mode::chunk(fhalf, 1))};
    typename Mode::template Frags<FM, FN> f0, f1;
    auto read = [&](const uint8_t *buf, typename Mode::template Frags<FM, FN> &f) {
        Mode::template read<BM, BN, FM, FN>(buf + wm * WM * REC_BYTES, buf + (NREC * BM + wn * WN) * REC_BYTES, at, f);
    };

    f32x16_t acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = f32x16_t{};

    // The next slab landed in every wave; every wave has read the one before it.
    // The scheduling barriers keep a step's work between its barriers: left to
    // itself the compiler moved matrix-core steps (which touch no memory) past
    // the next barrier, so that the wait for the loads came right after their
    // issue with nothing in between. With the steps kept apart, one more slab in
    // flight, no branch in the loop and the loads spread over the step like the
    // reads, the FP8 product 8192 x 4096 x 8192 went from 849 to 762 us (two
    // terms) and the split-BF16 product of order 8192, whose steps had stayed in
    // place, from 2430 to 2350 (2416 with all of a step's loads at its start).
    auto arrive = [] {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm((NSTAGE - 2) * LPW) & ~(0xF << 8));
        ring_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // One step, slab s landed: refill the slot of slab s - 1 (dma), read slab s
    // (nxt), multiply slab s - 1, interleaved. The two slots are disjoint LDS,
    // passed as restrict pointers so that the reads need not wait for the
    // loads, which are meant to stay in flight.
    auto step = [&](uint8_t *__restrict__ dma, const uint8_t *__restrict__ nxt,
                    const typename Mode::template Frags<FM, FN> &cur, typename Mode::template Frags<FM, FN> &next) {
        constexpr int MMAS = Mode::TERMS * FM * FN, READS = 2 * NREC * (FM + FN);
        issue_next(dma);
        read(nxt, next);
        Mode::template mma<FM, FN>(cur, acc);
#pragma unroll
        for (int i = 0; i < MMAS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                  // matrix core
            __builtin_amdgcn_sched_group_barrier(0x100, (READS + MMAS - 1) / MMAS, 0);
            __builtin_amdgcn_sched_group_barrier(0x20, (LPW + MMAS - 1) / MMAS, 0);
        }
    };
    auto fill = [&](uint8_t *__restrict__ dma, const uint8_t *__restrict__ nxt,
                    typename Mode::template Frags<FM, FN> &next) {
        issue_next(dma);
        read(nxt, next);
    };

    if (L > 0) {
        for (int q = 0; q < NSTAGE - 1; ++q) issue_next(lds + q * STAGE);
        int rd = 0, wr = NSTAGE - 1;                         // slots of slabs s and s - 1
        auto next_slot = [&] {
            wr = rd;
            rd = rd + 1 == NSTAGE ? 0 : rd + 1;
        };
        // The loop runs whole pairs, from a slab in f0 to one in f0; the last slab
        // ends in f1, so an odd number of slabs starts there.
        arrive();
        if (L & 1) {
            fill(lds + wr * STAGE, lds + rd * STAGE, f1);
            next_slot();
            if (L > 1) {
                arrive();
                step(lds + wr * STAGE, lds + rd * STAGE, f1, f0);
                next_slot();
            }
        } else {
            fill(lds + wr * STAGE, lds + rd * STAGE, f0);
            next_slot();
        }
        if (L > 1) {
            for (int pairs = L / 2 - 1; pairs > 0; --pairs) {
                arrive();
                step(lds + wr * STAGE, lds + rd * STAGE, f0, f1);
                next_slot();
                arrive();
                step(lds + wr * STAGE, lds + rd * STAGE, f1, f0);
                next_slot();
            }
            arrive();
            step(lds + wr * STAGE, lds + rd * STAGE, f0, f1);
        }
        Mode::template mma<FM, FN>(f1, acc);                 // the last slab
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));           // no load may land in LDS later
    }

    // Epilogue: register r of lane l holds C[8(r/4) + 4(l/32) + r%4][l%32] of
    // each 32x32 block; 32 lanes write one 128-byte run of a row of C, and a row's
    // runs follow each other (a block at a time, 8000 x 100 x 8000 took 97 us in
    // split-BF16 and 75 in FP8, one term; row by row 81 and 61). All loads
    // (exponents; the accumulate form's values of C, 8 rows at a time) come
    // before the stores that need them: a load between two stores waits for
    // both (with the row's exponent loaded before each store that FP8 product
    // took 114 us). Buffer resources end at row m, and columns past p get an
    // offset beyond every range, so no access needs a test of its own; one
    // resource per 8 rows of C keeps the offsets below 2^31 up to p = 2^26. The
    // resources are worked out where they are used: kept in arrays, or the
    // accumulate form's loads moved further ahead, the code grows and small
    // products pay for fetching it (64^3 in FP32 17.4 us against 15.7).
    float *dst = partial ? partial : op.C;
    const bool descale = Mode::SCALED && !partial;
    const int64_t iw = i0 + wm * WM, jw = j0 + wn * WN;      // the wave's part of C
    auto rsrc_of = [](const void *base, int64_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, bytes > 0 ? (int)bytes : 0, 0x00020000);
    };
    auto epilogue = [&](auto acc_form) {
        constexpr bool ACC = decltype(acc_form)::value;
        const int pb = (int)(p * 4);
        const int vrow = (lane >> 5) * 4 * pb;
        int fj[FN];
        if constexpr (Mode::SCALED) {
            const __amdgpu_buffer_rsrc_t cols = rsrc_of(op.col_exp + jw, descale ? (p - jw < WN ? p - jw : WN) * 4 : 0);
#pragma unroll
            for (int b = 0; b < FN; ++b)
                fj[b] = (int)__builtin_amdgcn_raw_buffer_load_b32(cols, (b * 32 + (lane & 31)) * 4, 0, 0);
        }
#pragma unroll
        for (int a = 0; a < FM; ++a) {
            const int64_t ia = iw + a * 32;
            i32x4_t ei[4];                                   // rows 8 g + 4 (lane / 32) .. + 3
            if constexpr (Mode::SCALED) {
                // whole quads: the exponents' array is padded to 256 bytes
                const int64_t quads = m - ia < 32 ? (m - ia + 3) / 4 : 8;
                const __amdgpu_buffer_rsrc_t rows = rsrc_of(op.row_exp + ia, descale ? quads * 16 : 0);
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    ei[g] = __builtin_bit_cast(i32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                            rows, (8 * g + 4 * (lane >> 5)) * 4, 0, 0));
            }
            int vj[FN];
#pragma unroll
            for (int b = 0; b < FN; ++b)
                vj[b] = jw + b * 32 + (lane & 31) < p ? (b * 32 + (lane & 31)) * 4 + vrow : kDeadVoffset;
#pragma unroll
            for (int g = 0; g < 4; ++g) {                    // rows ia + 8 g .. + 7, from column jw on
                const int64_t i = ia + 8 * g, live = m - i < 8 ? m - i : 8;
                const __amdgpu_buffer_rsrc_t c_rows = rsrc_of(dst + i * p + jw, live > 0 ? live * pb - jw * 4 : 0);
                float old[FN][4];
                if constexpr (ACC) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int b = 0; b < FN; ++b)
                            old[b][r] = __builtin_bit_cast(
                                float, __builtin_amdgcn_raw_buffer_load_b32(c_rows, vj[b] + r * pb, 0, 0));
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int b = 0; b < FN; ++b) {
                        float v = acc[a][b][4 * g + r];
                        if constexpr (Mode::SCALED) v = ldexpf(v, -(ei[g][r] + fj[b]));
                        if constexpr (ACC) v += old[b][r];
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), c_rows, vj[b] + r * pb,
                                                              0, 0);
                    }
            }
        }
    };
    // p beyond 2^26: 64-bit addresses. C is addressed as global memory: a generic
    // (flat) access could alias LDS.
    auto wide_epilogue = [&] {
        global_f32 *C = (global_f32 *)dst;
        const global_i32 *row_exp = (const global_i32 *)op.row_exp;
        const global_i32 *col_exp = (const global_i32 *)op.col_exp;
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                const int64_t j = jw + b * 32 + (lane & 31);
                if (j >= p) continue;
                const int fj = descale ? col_exp[j] : 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t i = iw + a * 32 + mfma32_row(r, lane);
                    if (i < m) {
                        float v = acc[a][b][r];
                        if (descale) v = ldexpf(v, -(row_exp[i] + fj));
                        if (op.accumulate && !partial) v += C[i * p + j];
                        C[i * p + j] = v;
                    }
                }
            }
    };
    if (p >= (int64_t(1) << 26)) wide_epilogue();
    else if (op.accumulate && !partial) epilogue(std::true_type{});
    else epilogue(std::false_type{});
#endif
}

// Tile-id -> block mapping of a single-product launch (XCD-aware bands).
__device__ __forceinline__ void block_of(int tiles_m, int tiles_n, int *tm, int *tn) {
    tile_coords(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, 8, tm, tn);
    // the integer divisions above run on the vector ALU; pin the (uniform)
    // results to scalar registers so everything derived from them stays scalar
    *tm = __builtin_amdgcn_readfirstlane(*tm);
    *tn = __builtin_amdgcn_readfirstlane(*tn);
}

// Workgroups per CU the register allocation must allow: two for four-wave
// blocks with a ring of more than 64 KiB that still leaves room for a second
// one in LDS (left to the compiler otherwise, which reaches three for the
// 48 KiB rings by itself).
template <int BM, int BN, int WM, int WN, int NREC, int NST>
constexpr int min_blocks() {
    using G = Cfg<BM, BN, WM, WN, NREC, NST>;
    return G::NW == 4 && G::LDS > 64 * 1024 && 2 * G::LDS <= 160 * 1024 ? 2 : 1;
}

template <int BM, int BN, int WM, int WN, int NREC, class Mode, int NST = NSTAGE>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, (min_blocks<BM, BN, WM, WN, NREC, NST>())) void single_kernel(Operands op, int tiles_m,
                                                                            int tiles_n) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg<BM, BN, WM, WN, NREC, NST>::LDS];
    int tm, tn;
    block_of(tiles_m, tiles_n, &tm, &tn);
    tile<BM, BN, WM, WN, NREC, Mode, NST>(op, (int64_t)tm * BM, (int64_t)tn * BN, lds);
}

// Split-k (the sigma loop cut into `chunks` contiguous runs of chunk_slabs
// slabs, Fig. 2's "addition loop" done across workgroups): workgroup w takes
// chunk w / tiles of tile w mod tiles (after the XCD remap, so the blocks of
// one chunk share an L2) and stores its raw block sum in partials + chunk m p.
template <int BM, int BN, int WM, int WN, int NREC, class Mode, int NST = NSTAGE>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void splitk_kernel(Operands op, int tiles_m, int tiles_n,
                                                                            int chunk_slabs, float *partials) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg<BM, BN, WM, WN, NREC, NST>::LDS];
    const int tiles = tiles_m * tiles_n;
    const int id = __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, (int)gridDim.x));
    const int chunk = id / tiles;
    int tm, tn;
    tile_coords(id - chunk * tiles, tiles_m, tiles_n, 8, &tm, &tn);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    const int s_begin = chunk * chunk_slabs;
    const int s_end = min((int)op.S, s_begin + chunk_slabs);
    tile<BM, BN, WM, WN, NREC, Mode, NST>(op, (int64_t)tm * BM, (int64_t)tn * BN, lds, s_begin, s_end,
                                          partials + (int64_t)chunk * op.m * op.p);
}

// W consecutive elements of C from their chunk partials (mp apart), in chunk
// order: C = ((P_0 + P_1) + ...) + P_c-1, then the descale (scaled modes) and
// the accumulate form, as the epilogue of an unsplit product does. Eight chunks'
// loads are in flight together: the sum is a chain, the loads need not be.
template <int W>
__device__ __forceinline__ void splitk_sum(const float *__restrict__ partials, int chunks, int64_t mp, int64_t x,
                                           float *__restrict__ C, int exponent, const int32_t *col_exp,
                                           int accumulate) {
    typedef float vec __attribute__((ext_vector_type(W == 1 ? 2 : W)));
    float v[W];
    auto load = [&](const float *src, float (&out)[W]) {
        if constexpr (W == 1) {
            out[0] = *src;
        } else {
            const vec y = *reinterpret_cast<const vec *>(src);
#pragma unroll
            for (int e = 0; e < W; ++e) out[e] = y[e];
        }
    };
    load(partials + x, v);
#pragma unroll 8
    for (int q = 1; q < chunks; ++q) {
        float y[W];
        load(partials + (int64_t)q * mp + x, y);
#pragma unroll
        for (int e = 0; e < W; ++e) v[e] += y[e];
    }
    if (col_exp) {
#pragma unroll
        for (int e = 0; e < W; ++e) v[e] = ldexpf(v[e], -(exponent + col_exp[e]));
    }
    if (accumulate) {
        float old[W];
        load(C + x, old);
#pragma unroll
        for (int e = 0; e < W; ++e) v[e] += old[e];
    }
    if constexpr (W == 1) {
        C[x] = v[0];
    } else {
        vec y;
#pragma unroll
        for (int e = 0; e < W; ++e) y[e] = v[e];
        *reinterpret_cast<vec *>(C + x) = y;
    }
}

// The whole m x p array, W elements per thread (W divides p).
template <int W>
static __global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ partials, int chunks,
                                                                   int64_t m, int64_t p, float *__restrict__ C,
                                                                   const int32_t *__restrict__ row_exp,
                                                                   const int32_t *__restrict__ col_exp,
                                                                   int accumulate) {
    const int64_t mp = m * p;
    for (int64_t x = ((int64_t)blockIdx.x * 256 + threadIdx.x) * W; x < mp; x += (int64_t)gridDim.x * 256 * W) {
        const int64_t i = row_exp ? x / p : 0;
        splitk_sum<W>(partials, chunks, mp, x, C, row_exp ? row_exp[i] : 0, row_exp ? col_exp + (x - i * p) : nullptr,
                      accumulate);
    }
}

inline hipError_t launch_splitk_reduce(const float *partials, int chunks, int64_t m, int64_t p, float *C,
                                       const int32_t *row_exp, const int32_t *col_exp, int accumulate,
                                       hipStream_t st) {
    const bool wide = p % 4 == 0 && (uintptr_t)C % 16 == 0 && (uintptr_t)partials % 16 == 0;
    const dim3 grid((unsigned)std::min<int64_t>((m * p / (wide ? 4 : 1) + 255) / 256, 65536));
    if (wide)
        hipLaunchKernelGGL(splitk_reduce_kernel<4>, grid, dim3(256), 0, st, partials, chunks, m, p, C, row_exp, col_exp,
                           accumulate);
    else
        hipLaunchKernelGGL(splitk_reduce_kernel<1>, grid, dim3(256), 0, st, partials, chunks, m, p, C, row_exp, col_exp,
                           accumulate);
    return hipGetLastError();
}

// Host side of a split-k launch: chunk kernel, then the reduction.
template <int BM, int BN, int WM, int WN, int NREC, class Mode, int NST>
hipError_t launch_splitk(const Operands &op, int chunks, float *partials, hipStream_t st) {
    const int tiles_m = (int)((op.m + BM - 1) / BM), tiles_n = (int)((op.p + BN - 1) / BN);
    const int chunk_slabs = (int)((op.S + chunks - 1) / chunks);
    chunks = (int)((op.S + chunk_slabs - 1) / chunk_slabs);   // every chunk non-empty
    hipLaunchKernelGGL((splitk_kernel<BM, BN, WM, WN, NREC, Mode, NST>), dim3(tiles_m * tiles_n * chunks),
                       dim3(Cfg<BM, BN, WM, WN, NREC, NST>::THREADS), 0, st, op, tiles_m, tiles_n, chunk_slabs,
                       partials);
    return launch_splitk_reduce(partials, chunks, op.m, op.p, op.C, op.row_exp, op.col_exp, op.accumulate, st);
}

// Host check of the direct loads of single-product launches over an m x p
// product with S slabs and blocks of BM x BN (waves WM x WN, NREC record
// arrays per operand), through the same window functions as the kernel. For
// every block, wave and load: a live load's last window (slab S-1, where the
// offsets peak) lies inside its array's padded rows and inside its
// resource's range, with both offsets below 2^31; a dead load's tile lies
// wholly past the operand's padded rows (so its LDS rows feed only outputs
// that are not stored), and its vector offset 2^31 exceeds every resource
// range (num_records below 2^31). Returns the number of violations and the number of
// loads checked per slab in *loads.
inline int64_t check_loads(int BM, int BN, int WM, int WN, int NREC, int64_t m, int64_t p, int64_t S,
                           int64_t *loads) {
    const int NW = (BM / WM) * (BN / WN);
    const int ROWS = NREC * (BM + BN);
    const int LPW = ROWS / 16 / NW;
    const int64_t tile_row = S * GROUP * REC_BYTES;
    const int64_t lim31 = (int64_t(1) << 31) - 1;
    int64_t bad = 0, count = 0;
    if (BM % (16 * NW) != 0 || BN % (16 * NW) != 0 || S <= 0) return 1;
    for (int64_t i0 = 0; i0 < m; i0 += BM)
        for (int64_t j0 = 0; j0 < p; j0 += BN)
            for (int wave = 0; wave < NW; ++wave)
                for (int q = 0; q < LPW; ++q) {
                    ++count;
                    const RowWindow w = row_window(BM, BN, NREC, (NW * q + wave) * 16, i0, j0, m, p);
                    const int tile_in = w.row_in / GROUP;
                    // every wave's load q reads the array of wave 0's, from the same first tile
                    const RowWindow w0 = row_window(BM, BN, NREC, NW * q * 16, i0, j0, m, p);
                    if (w0.a != w.a || w0.arr != w.arr || w0.first_tile != w.first_tile || w0.tiles != w.tiles ||
                        w0.row_in + 16 * wave != w.row_in)
                        ++bad;
                    const int64_t padded_tiles = padded_rows(w.a ? m : p) / GROUP;
                    const int64_t num_records = (int64_t)w.tiles * tile_row;
                    if (w.tiles < 1 || num_records > lim31) ++bad;
                    const int64_t soff = tile_in * tile_row + (S - 1) * GROUP * REC_BYTES;
                    if (soff > lim31) ++bad;
                    if (tile_in < w.tiles) {                  // live
                        const int64_t end = soff + GROUP * REC_BYTES;   // voffset < 1 KiB, 16 bytes each
                        if (w.first_tile + tile_in >= padded_tiles || end > num_records) ++bad;
                    } else if (w.first_tile + tile_in < padded_tiles) {
                        ++bad;                                // dead but inside the operand
                    }
                }
    if (loads) *loads = count;
    return bad;
}

}  // namespace ring
}  // namespace moa
