// Split-BF16 contraction straight from FP32 operands: no conditioning pass and
// no records in memory. A workgroup owns a BM x BN block of C and walks the k
// slabs of 16; per slab the FP32 values of its rows of A and columns of B go
// from memory into an LDS ring (buffer_load ... lds), and every wave splits the
// values of the fragments it multiplies into hi/lo BF16 in registers.
//
// Every element of C receives the operation sequence of the record ring
// (ring_gemm.h with the split-BF16 mode): the same hi/lo values, zero past n,
// and per slab lo.hi, hi.lo, hi.hi on the same matrix-core step, slabs
// ascending. Results are therefore bitwise those of the conditioned path,
// whatever the block.
//
// An operand is laid down by its contiguous extent, so every layout runs the
// same loop:
//   k-contiguous (row-major A, column-major B): one 64-byte row (16 k) per row
//     of the block, 16-byte chunk c of row r at chunk c ^ ((r / 4) mod 4);
//   k-strided (row-major B, column-major A): the slab's 16 rows of the block's
//     extent, rows 8 .. 15 turned by 128 bytes, so that the two halves of a
//     wave (k and k + 8 of the same columns) read disjoint banks.
//
// What bounds a step of a 128 x 128 block (four waves of 64 x 64): per wave 12
// matrix-core steps of 32 cycles (384), 96 vector instructions for the split
// (the SIMD issues one of either kind every 4 cycles while both run: 430), 16
// KiB into LDS and 32 KiB out of it. A wave that splits a slab and then
// multiplies it takes the sum, so the step is a pipeline: slab s is read from
// LDS, slab s - 1 split and slab s - 2 multiplied in one stretch of
// independent instructions. 2048^3 with one block per CU: 65 us (0.50 us per
// step), 75 us when each slab is split just before it is multiplied, and 80 us
// with the conditioning pass and the record ring. bf16 dot products for the
// residuals (two vector instructions per value instead of three) measured
// slower (they run on the matrix cores' pipeline), and so did 256 x 128 blocks
// of eight waves (4096^3: 435-444 against 434 us).
#pragma once

#include "moa_internal.h"
#include "ring_gemm.h"
#include "tile_common.h"

namespace moa {
namespace raw {

constexpr int SLAB = 16;

// One product's operands. ld: elements from row to row of a k-contiguous operand
// (n for a whole product, more for a window of its k walk).
struct Operands {
    const float *A, *B;
    float *C;
    int64_t m, n, p, ld;
    int accumulate;
};

// One operand's share of a slab: W rows (or columns) of the block; KC: k is
// its contiguous extent.
template <int W, bool KC> struct Operand {
    static constexpr int BYTES = W * 64;
    static constexpr int LOADS = W / 16;                     // KiB loads
    static constexpr int CPR = W / 4;                        // 16-byte chunks of a k-strided row
    static_assert(W == 64 || W == 128 || W == 256, "whole loads, rows of at most one load");

    // Vector offset of lane `lane` in load g; live: rows of the block inside
    // the operand (KC), ld: bytes from row to row (KC) or from k to k.
    static __host__ __device__ __forceinline__ int voffset(int g, int lane, int64_t live, int64_t ld) {
        if constexpr (KC) {
            const int r = 16 * g + (lane >> 2);
            const int c = (lane & 3) ^ ((lane >> 4) & 3);
            return r < live ? (int)(r * ld + 16 * c) : ring::kDeadVoffset;
        } else {
            const int k = g * (64 / CPR) + lane / CPR;
            const int c = (lane % CPR + CPR - (8 * (k >> 3)) % CPR) % CPR;
            return (int)(k * ld + 16 * c);
        }
    }
    // The 8 values k = 8 half .. 8 half + 7 of row r.
    static __device__ __forceinline__ void read8(const uint8_t *buf, int r, int half, float (&x)[8]) {
        if constexpr (KC) {
            const int sw = (r >> 2) & 3;
            const float4 v0 = *reinterpret_cast<const float4 *>(buf + r * 64 + (((2 * half) ^ sw) << 4));
            const float4 v1 = *reinterpret_cast<const float4 *>(buf + r * 64 + (((2 * half + 1) ^ sw) << 4));
            x[0] = v0.x; x[1] = v0.y; x[2] = v0.z; x[3] = v0.w;
            x[4] = v1.x; x[5] = v1.y; x[6] = v1.z; x[7] = v1.w;
        } else {
            const uint8_t *b = buf + 8 * half * W * 4 + ((((r >> 2) + 8 * half) % CPR) << 4) + ((r & 3) << 2);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = *reinterpret_cast<const float *>(b + e * W * 4);
        }
    }
};

template <int BM, int BN, int WM, int WN, int NST> struct Cfg {
    static constexpr int WAVES_N = BN / WN;
    static constexpr int FM = WM / 32, FN = WN / 32;
    static constexpr int STAGE = (BM + BN) * 64, LDS = NST * STAGE;
    static constexpr int LPA = BM / 64, LPB = BN / 64, LPW = LPA + LPB;      // KiB loads per wave and slab
    static_assert((BM / WM) * (BN / WN) == 4, "four waves");
    static_assert(NST >= 3 && (NST - 2) * LPW <= 63, "a slot being refilled, one being read, one landing");
};

// The BM x BN block of C at (i0, j0). `lds`: the workgroup's ring; on entry no
// wave may still be reading it, on exit this wave has no load in flight.
template <int BM, int BN, int WM, int WN, int NST, bool A_KC, bool B_KC>
__device__ __forceinline__ void block(const Operands &d, int64_t i0, int64_t j0, uint8_t *lds) {
#ifdef __HIP_DEVICE_COMPILE__           // the host pass would check the 16-byte direct loads against its own target
    using G = Cfg<BM, BN, WM, WN, NST>;
    using OA = Operand<BM, A_KC>;
    using OB = Operand<BN, B_KC>;
    constexpr int FM = G::FM, FN = G::FN, LPA = G::LPA, LPB = G::LPB, LPW = G::LPW, STAGE = G::STAGE;
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));         // lane constants are worked out per block, not held across a persistent loop
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / G::WAVES_N, wn = wave % G::WAVES_N;
    const int64_t m = d.m, n = d.n, p = d.p;
    const int S = (int)((n + SLAB - 1) / SLAB);

    // Both resources start at the slab and end where the operand's live data
    // ends (rows past m or p and k past n come as zeros, or as values of the
    // next row, masked in the last slab), so the lanes' offsets are the same
    // for every slab. Slabs past the last have empty ranges: their loads touch
    // no memory but keep the count of loads in flight.
    const int64_t a_live = m - i0 < BM ? m - i0 : BM, b_live = p - j0 < BN ? p - j0 : BN;
    const char *a_src = reinterpret_cast<const char *>(d.A + (A_KC ? i0 * d.ld : i0));
    const char *b_src = reinterpret_cast<const char *>(d.B + (B_KC ? j0 * d.ld : j0));
    int64_t a_left = (A_KC ? (a_live - 1) * d.ld + n : n * m - i0) * 4;
    int64_t b_left = (B_KC ? (b_live - 1) * d.ld + n : n * p - j0) * 4;
    const int64_t a_step = (A_KC ? 1 : m) * SLAB * 4, b_step = (B_KC ? 1 : p) * SLAB * 4;
    int voff[LPW];
#pragma unroll
    for (int q = 0; q < LPA; ++q) voff[q] = OA::voffset(wave * LPA + q, lane, a_live, (A_KC ? d.ld : m) * 4);
#pragma unroll
    for (int q = 0; q < LPB; ++q) voff[LPA + q] = OB::voffset(wave * LPB + q, lane, b_live, (B_KC ? d.ld : p) * 4);
    int to_issue = S;
    auto clip = [](int64_t x) {                              // 0 .. 2^31 - 1, in 32-bit scalar steps
        const int hi = (int)(x >> 32);
        const uint32_t lo = min((uint32_t)x, 0x7FFFFFFFu);
        return hi < 0 ? 0 : hi > 0 ? 0x7FFFFFFF : (int)lo;
    };
    // The next slab into buf.
    auto issue_next = [&](uint8_t *buf) {
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void *)a_src, (short)0,
                                                                            to_issue > 0 ? clip(a_left) : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)b_src, (short)0,
                                                                            to_issue > 0 ? clip(b_left) : 0, 0x00020000);
#pragma unroll
        for (int q = 0; q < LPA; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (ring::lds_void_t *)(buf + (wave * LPA + q) * 1024), 16,
                                                     voff[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < LPB; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rb, (ring::lds_void_t *)(buf + OA::BYTES + (wave * LPB + q) * 1024), 16, voff[LPA + q], 0, 0, 0);
        a_src += a_step;
        b_src += b_step;
        a_left -= a_step;
        b_left -= b_step;
        --to_issue;
    };

    const int row = lane & 31, half = lane >> 5;
    const int a_row = wm * WM + row, b_row = wn * WN + row;
    struct Raw { float a[FM][8], b[FN][8]; };                        // one slab's values
    struct Split { bf16x8_t ah[FM], al[FM], bh[FN], bl[FN]; };       // and its hi/lo fragments
    Raw raw[2];
    Split cv[2];
    f32x16_t acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = f32x16_t{};
    auto split8 = [&](const float (&x)[8], bf16x8_t &hi, bf16x8_t &lo) {
        uint4 h, l;
        split_pair(x[0], x[1], &h.x, &l.x);
        split_pair(x[2], x[3], &h.y, &l.y);
        split_pair(x[4], x[5], &h.z, &l.z);
        split_pair(x[6], x[7], &h.w, &l.w);
        hi = __builtin_bit_cast(bf16x8_t, h);
        lo = __builtin_bit_cast(bf16x8_t, l);
    };
    auto read = [&](const uint8_t *buf, Raw &x) {
#pragma unroll
        for (int a = 0; a < FM; ++a) OA::read8(buf, a_row + a * 32, half, x.a[a]);
#pragma unroll
        for (int b = 0; b < FN; ++b) OB::read8(buf + OA::BYTES, b_row + b * 32, half, x.b[b]);
    };
    auto split = [&](const Raw &x, Split &f) {
#pragma unroll
        for (int a = 0; a < FM; ++a) split8(x.a[a], f.ah[a], f.al[a]);
#pragma unroll
        for (int b = 0; b < FN; ++b) split8(x.b[b], f.bh[b], f.bl[b]);
    };
    // Matrix-core step x of a slab's 3 FM FN, term-major: consecutive ones are
    // independent.
    constexpr int MMAS = 3 * FM * FN;
    auto multiply_one = [&](const Split &f, int x) {
        const int term = x / (FM * FN), a = x / FN % FM, b = x % FN;
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(term == 0 ? f.al[a] : f.ah[a], term == 1 ? f.bl[b] : f.bh[b],
                                                            acc[a][b], 0, 0, 0);
    };
    auto multiply = [&](const Split &f) {
#pragma unroll
        for (int x = 0; x < MMAS; ++x) multiply_one(f, x);
    };
    // One step of the pipeline, slab s landed: refill the slot of slab s - 1
    // (dma), read slab s (nxt) into registers, split slab s - 1, multiply slab
    // s - 2; C = s mod 2. The three are independent and are interleaved: a
    // matrix-core step takes 32 cycles, in which the wave issues its share of
    // the vector and LDS instructions. The two slots are disjoint LDS, passed as
    // restrict pointers so that the reads need not wait for the loads, which
    // are meant to stay in flight.
    auto step = [&](uint8_t *__restrict__ dma, const uint8_t *__restrict__ nxt, int C) {
        constexpr int VALU = (24 * (FM + FN) + 4 + MMAS - 1) / MMAS;          // per matrix-core step
        constexpr int LDS = 2 * (A_KC ? FM : 2 * FM) + 2 * (B_KC ? FN : 2 * FN);
        issue_next(dma);
        read(nxt, raw[C]);
        split(raw[C ^ 1], cv[C ^ 1]);
        multiply(cv[C]);
#pragma unroll
        for (int i = 0; i < MMAS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                  // matrix core
            __builtin_amdgcn_sched_group_barrier(0x100, (LDS + MMAS - 1) / MMAS, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, VALU, 0);               // vector
        }
    };
    auto fill0 = [&](uint8_t *__restrict__ dma, const uint8_t *__restrict__ nxt) {
        issue_next(dma);
        read(nxt, raw[0]);
    };
    auto fill1 = [&](uint8_t *__restrict__ dma, const uint8_t *__restrict__ nxt) {
        issue_next(dma);
        read(nxt, raw[1]);
        split(raw[0], cv[0]);
    };
    // the last slab (in raw[1]): k past n counts as zero
    auto finish = [&] {
        multiply(cv[0]);
        const int live = (int)(n - (int64_t)(S - 1) * SLAB) - 8 * half;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
            for (int a = 0; a < FM; ++a) raw[1].a[a][e] = e < live ? raw[1].a[a][e] : 0.0f;
#pragma unroll
            for (int b = 0; b < FN; ++b) raw[1].b[b][e] = e < live ? raw[1].b[b][e] : 0.0f;
        }
        split(raw[1], cv[1]);
        multiply(cv[1]);
    };
    // the next slab landed in every wave; every wave has read the one before it
    auto arrive = [] {
        __builtin_amdgcn_sched_barrier(0);                   // a step's work stays between its barriers
        __builtin_amdgcn_s_waitcnt(ring::waitcnt_vm((NST - 2) * LPW) & ~(0xF << 8));
        ring::ring_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    if (S > 0) {
        for (int q = 0; q < NST - 1; ++q) issue_next(lds + q * STAGE);
        int rd = 0, wr = NST - 1;                            // slots of slabs s and s - 1
        auto next_slot = [&] {
            wr = rd;
            rd = rd + 1 == NST ? 0 : rd + 1;
        };
        // An odd number of slabs starts with one of zeros, so that the loop runs
        // whole pairs (its products add +0 to accumulators that are +0).
        if (S & 1) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
#pragma unroll
                for (int a = 0; a < FM; ++a) raw[0].a[a][e] = 0.0f;
#pragma unroll
                for (int b = 0; b < FN; ++b) raw[0].b[b][e] = 0.0f;
            }
        } else {
            arrive();
            fill0(lds + wr * STAGE, lds + rd * STAGE);
            next_slot();
        }
        arrive();
        fill1(lds + wr * STAGE, lds + rd * STAGE);
        next_slot();
        for (int pairs = (S + 1) / 2 - 1; pairs > 0; --pairs) {
            arrive();
            step(lds + wr * STAGE, lds + rd * STAGE, 0);
            next_slot();
            arrive();
            step(lds + wr * STAGE, lds + rd * STAGE, 1);
            next_slot();
        }
        finish();
        __builtin_amdgcn_s_waitcnt(ring::waitcnt_vm(0));     // no load may land in LDS later
    }

    // Epilogue: one resource per 8 rows of C, which ends at the last row inside
    // m; columns past p get an offset beyond every range. The accumulate form
    // reads a 32 x 32 block's values before any store.
    auto store = [&](auto acc_form) {
        constexpr bool ACC = decltype(acc_form)::value;
        const int pb = (int)(p * 4);
        const int vrow = (lane >> 5) * 4 * pb;
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            const int64_t j = j0 + wn * WN + b * 32 + row;
            const uint32_t vj = j < p ? (uint32_t)(j * 4) + vrow : (uint32_t)ring::kDeadVoffset;
#pragma unroll
            for (int a = 0; a < FM; ++a) {
                const int64_t ia = i0 + wm * WM + a * 32;
                float old[16];
                auto rsrc = [&](int g) {                     // rows ia + 8 g .. + 7
                    const int64_t i = ia + 8 * g, rows = m - i < 8 ? m - i : 8;
                    return __builtin_amdgcn_make_buffer_rsrc((void *)(d.C + i * p), (short)0,
                                                             rows > 0 ? (int)rows * pb : 0, 0x00020000);
                };
                if constexpr (ACC) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        old[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                               rsrc(r >> 2), (int)(vj + (r & 3) * pb), 0, 0));
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float v = acc[a][b][r];
                    if constexpr (ACC) v += old[r];
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rsrc(r >> 2),
                                                          (int)(vj + (r & 3) * pb), 0, 0);
                }
            }
        }
    };
    if (d.accumulate) store(std::true_type{});
    else store(std::false_type{});
#endif
}

// A single product: one block per workgroup.
template <int BM, int BN, int WM, int WN, int NST, bool A_KC, bool B_KC>
__global__ __launch_bounds__(256, 2) void single_kernel(Operands d, int tiles_m, int tiles_n) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg<BM, BN, WM, WN, NST>::LDS];
    int tm, tn;
    ring::block_of(tiles_m, tiles_n, &tm, &tn);
    block<BM, BN, WM, WN, NST, A_KC, B_KC>(d, (int64_t)tm * BM, (int64_t)tn * BN, lds);
}

// Split-k (the sigma loop cut into runs of chunk_slabs slabs): workgroup w takes
// chunk w / tiles of block w mod tiles (after the XCD remap, so the blocks of
// one chunk share an L2) and writes its block sum to partials + chunk m p.
template <int BM, int BN, int WM, int WN, int NST, bool A_KC, bool B_KC>
__global__ __launch_bounds__(256, 2) void splitk_kernel(Operands d, int tiles_m, int tiles_n, int chunk_slabs,
                                                        float *partials) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg<BM, BN, WM, WN, NST>::LDS];
    const int tiles = tiles_m * tiles_n;
    const int id = __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, (int)gridDim.x));
    const int chunk = id / tiles;
    int tm, tn;
    tile_coords(id - chunk * tiles, tiles_m, tiles_n, 8, &tm, &tn);
    const int64_t k0 = (int64_t)chunk * chunk_slabs * SLAB;
    d.A += A_KC ? k0 : k0 * d.m;
    d.B += B_KC ? k0 : k0 * d.p;
    d.C = partials + (int64_t)chunk * d.m * d.p;
    d.n = min((int64_t)chunk_slabs * SLAB, d.n - k0);
    d.accumulate = 0;
    block<BM, BN, WM, WN, NST, A_KC, B_KC>(d, (int64_t)__builtin_amdgcn_readfirstlane(tm) * BM,
                                           (int64_t)__builtin_amdgcn_readfirstlane(tn) * BN, lds);
}

// Host check of the loads of one operand of a launch (or of one chunk of its k
// walk): `extent` rows or columns in blocks of W, n of k, ld elements from row to
// row, `size` elements from the operand's first to its end. For every block and
// the first and last slab: the buffer range ends inside the operand, no lane's
// 16 bytes pass the 32-bit offsets, and what the block needs (rows inside the
// operand, k below n) is inside the range. Returns the violations; adds the loads
// per slab to *loads.
template <int W, bool KC>
int64_t check_operand(int64_t extent, int64_t n, int64_t ld, int64_t size, int64_t *loads) {
    using O = Operand<W, KC>;
    const int64_t lim31 = 0x7FFFFFFF, S = (n + SLAB - 1) / SLAB;
    int64_t bad = 0;
    for (int64_t at = 0; at < extent; at += W) {
        // as block() lays them out: rows inside the operand, first element, bytes
        // to the live end and per slab, bytes from row to row or from k to k
        const int64_t live = std::min<int64_t>(extent - at, W), first = KC ? at * ld : at;
        const int64_t end = (KC ? (live - 1) * ld + n : n * extent - at) * 4;
        const int64_t step = (KC ? 1 : extent) * SLAB * 4, pitch = (KC ? ld : extent) * 4;
        *loads += O::LOADS;
        if (first * 4 + end > size * 4) ++bad;
        for (int64_t s = 0; s < S; s += std::max<int64_t>(S - 1, 1)) {
            const int64_t left = end - s * step, range = std::min(left, lim31);
            if (left <= 0) ++bad;
            for (int g = 0; g < O::LOADS; ++g)
                for (int lane = 0; lane < 64; ++lane) {
                    // the row (KC) or k of the lane's 16 bytes, and their chunk of it
                    const int r = KC ? 16 * g + (lane >> 2) : g * (64 / O::CPR) + lane / O::CPR;
                    const uint32_t v = (uint32_t)O::voffset(g, lane, live, pitch);
                    if (KC && r >= live) {
                        if (v <= (uint32_t)lim31) ++bad;    // must pass every range
                        continue;
                    }
                    const int64_t c = ((int64_t)v - r * pitch) / 16;
                    if (v + 15 > (uint32_t)lim31 || c < 0 || c >= (KC ? 4 : O::CPR)) ++bad;
                    for (int e = 0; e < 4; ++e) {
                        const int64_t k = s * SLAB + (KC ? 4 * c + e : r), at_row = KC ? r : 4 * c + e;
                        if (k < n && at_row < live && (int64_t)v + 4 * e + 4 > range) ++bad;
                    }
                }
        }
    }
    return bad;
}

}  // namespace raw
}  // namespace moa
