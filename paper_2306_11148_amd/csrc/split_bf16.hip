// Split-BF16 matrix-core path: C = hi(A).hi(B) + hi(A).lo(B) + lo(A).hi(B)
// with FP32 accumulation, where x = hi + lo + O(2^-16 |x|), hi = RNE_bf16(x),
// lo = RNE_bf16(x - hi). This evaluates Eq. 3 (section "MoA Matrix
// Multiplication") to about FP32 accuracy on the BF16 matrix cores.
//
// Two stages.
//
// 1. Conditioning (HBM-bound): A and B are rewritten as record tiles (layout
//    in ring_gemm.h). The k extent is cut into slabs of 16 (the sigma loop
//    broken into blocks, section "Dimension Lifting to Machine Coordinates");
//    for every row i of A and every column j of B, slab s becomes one
//    contiguous 64-byte record
//        [hi of x[16s .. 16s+15] (16 bf16)][lo of the same (16 bf16)]
//    zero-padded past n. B is transposed on the way (column j of B becomes
//    record row j), so both operands are k-contiguous.
//
// 2. Contraction (matrix-core bound): the record-tile ring of ring_gemm.h
//    (blocked form of Fig. 2) with three BF16 matrix-core steps per slab and
//    block pair, FP32 accumulation.
//
// Products of few blocks and grouped products skip stage 1: raw_gemm.h streams
// the FP32 operands and splits them on the way, with the same bits.
#include <algorithm>
#include <cstring>
#include <vector>

#include "moa_internal.h"
#include "raw_gemm.h"
#include "ring_gemm.h"
#include "tile_common.h"

namespace moa {
namespace {

using ring::GROUP;
using ring::padded_rows;
using ring::REC_BYTES;

constexpr int SLAB = 16;                  // k per record: [hi 16 bf16][lo 16 bf16] = 64 bytes
static_assert(REC_BYTES == 2 * SLAB * 2, "one record holds hi and lo of one slab");

// ---------------------------------------------------------------- stage 1 --

// Rows of X (rows x K, row-major) -> records: chunk q = 8 k values of one
// record (2 chunks per record).
__device__ __forceinline__ void pack_rows_chunk(const float *__restrict__ X, int64_t rows, int64_t K,
                                                int64_t S, uint8_t *__restrict__ P, int64_t q) {
    // q -> (row tile g, slab s, row rr in the tile, chunk c): consecutive
    // threads fill one KiB tile contiguously
    const int c = (int)(q & 1);
    const int64_t rr = (q >> 1) % GROUP;
    const int64_t gs = (q >> 1) / GROUP;
    const int64_t s = gs % S, g = gs / S;
    const int64_t r = g * GROUP + rr;
    const int64_t k = s * SLAB + c * 8;
    f32x4_t x[2] = {};
    if (r < rows) {
        x[0] = row4(X + r * K, k, K);
        x[1] = row4(X + r * K, k + 4, K);
    }
    uint4 hi, lo;
    split_pair(x[0][0], x[0][1], &hi.x, &lo.x);
    split_pair(x[0][2], x[0][3], &hi.y, &lo.y);
    split_pair(x[1][0], x[1][1], &hi.z, &lo.z);
    split_pair(x[1][2], x[1][3], &hi.w, &lo.w);
    uint8_t *rec = P + ring::rec_byte(r, s, S);
    *reinterpret_cast<uint4 *>(rec + c * 16) = hi;          // hi: bytes 0 .. 31
    *reinterpret_cast<uint4 *>(rec + 32 + c * 16) = lo;     // lo: bytes 32 .. 63
}

__global__ __launch_bounds__(256) void pack_rows_kernel(const float *__restrict__ X, int64_t rows,
                                                        int64_t K, int64_t S, uint8_t *__restrict__ P) {
    const int64_t chunks = padded_rows(rows) * S * 2;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < chunks; q += (int64_t)gridDim.x * 256)
        pack_rows_chunk(X, rows, K, S, P, q);
}

// Columns of X (K x cols, row-major) -> records (transposed), 64 columns x
// 64 k (4 slabs) per block through LDS: reads of X rows are contiguous
// float4s and each thread writes two half records. Columns past
// `cols` get zero records. All 256 threads must take part.
struct ColBlockRegs { f32x4_t v[4]; };

__device__ __forceinline__ void pack_cols_load(const float *__restrict__ X, int64_t K, int64_t cols,
                                               int64_t bx, int64_t by, ColBlockRegs &r) {
    const int t = threadIdx.x;
    const int jq = (t & 15) * 4;                 // four columns 4 (t%16) .. +3
    const int64_t j = bx * 64 + jq;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t k = by * 4 * SLAB + (t >> 4) + 16 * i;
        f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k < K) v = row4(X + k * cols, j, cols);
        r.v[i] = v;
    }
}

// Stores a loaded block to LDS, then (after a barrier) writes its records.
// The 512 half records of the block (4 slabs x 64 columns x {k 0-7, k 8-15})
// are taken two per thread; within a wave consecutive lanes take the two
// halves of consecutive records, so that each 16-byte store instruction fills
// half of every 64-byte record of two row tiles (as the row packer does),
// rather than a quarter of 64 scattered records.
__device__ __forceinline__ void pack_cols_emit(const ColBlockRegs &r, int64_t cols, int64_t S,
                                               uint8_t *__restrict__ P, int64_t bx, int64_t by,
                                               float (*tile)[64 + 4]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4_t *>(&tile[(t >> 4) + 16 * i][(t & 15) * 4]) = r.v[i];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int u = t + 256 * h;
        const int c = u & 1, jj = (u >> 1) & 63, part = u >> 7;
        const int64_t j = bx * 64 + jj, s = by * 4 + part;
        if (j < padded_rows(cols) && s < S) {
            const int kb = part * SLAB + c * 8;
            uint4 hi, lo;
            split_pair(tile[kb + 0][jj], tile[kb + 1][jj], &hi.x, &lo.x);
            split_pair(tile[kb + 2][jj], tile[kb + 3][jj], &hi.y, &lo.y);
            split_pair(tile[kb + 4][jj], tile[kb + 5][jj], &hi.z, &lo.z);
            split_pair(tile[kb + 6][jj], tile[kb + 7][jj], &hi.w, &lo.w);
            uint8_t *rec = P + ring::rec_byte(j, s, S);
            *reinterpret_cast<uint4 *>(rec + c * 16) = hi;          // hi: bytes 0 .. 31
            *reinterpret_cast<uint4 *>(rec + 32 + c * 16) = lo;     // lo: bytes 32 .. 63
        }
    }
    __syncthreads();                             // tile free for the next block
}

// Each workgroup walks up to COL_BLOCKS consecutive 64-k blocks of one
// 64-column strip, loading block b+1 while it writes block b.
constexpr int COL_BLOCKS = 4;

__global__ __launch_bounds__(256) void pack_cols_kernel(const float *__restrict__ X, int64_t K,
                                                        int64_t cols, int64_t S, uint8_t *__restrict__ P) {
    __shared__ __attribute__((aligned(16))) float tile[4 * SLAB][64 + 4];
    const int64_t by_count = (S + 3) / 4;
    const int64_t bx = blockIdx.x;
    for (int64_t by0 = (int64_t)blockIdx.y * COL_BLOCKS; by0 < by_count; by0 += (int64_t)gridDim.y * COL_BLOCKS) {
        const int64_t by_end = min(by0 + COL_BLOCKS, by_count);
        ColBlockRegs cur, next;
        pack_cols_load(X, K, cols, bx, by0, cur);
        for (int64_t by = by0; by < by_end; ++by) {
            if (by + 1 < by_end) pack_cols_load(X, K, cols, bx, by + 1, next);
            pack_cols_emit(cur, cols, S, P, bx, by, tile);
            cur = next;
        }
    }
}

// ---------------------------------------------------------------- stage 2 --

// Fragments of 32 records (rows) x 8 k: lane l reads row base + l%32; its hi
// values are logical chunk l/32 of the record, its lo values chunk 2 + l/32.
struct SplitMode {
    static constexpr bool SCALED = false;
    template <int FM, int FN> struct Frags { bf16x8_t ah[FM], al[FM], bh[FN], bl[FN]; };

    static constexpr int TERMS = 3;
    static __device__ __forceinline__ int chunk(int half, int x) { return 2 * x + half; }
    static __device__ __forceinline__ bf16x8_t frag(const uint8_t *rows, int at) {
        return *reinterpret_cast<const bf16x8_t *>(rows + at);
    }

    template <int BM, int BN, int FM, int FN>
    static __device__ __forceinline__ void read(const uint8_t *a_part, const uint8_t *b_part, const int (&at)[2],
                                                Frags<FM, FN> &f) {
#pragma unroll
        for (int a = 0; a < FM; ++a) {
            f.ah[a] = frag(a_part + a * 32 * ring::REC_BYTES, at[0]);
            f.al[a] = frag(a_part + a * 32 * ring::REC_BYTES, at[1]);
        }
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            f.bh[b] = frag(b_part + b * 32 * ring::REC_BYTES, at[0]);
            f.bl[b] = frag(b_part + b * 32 * ring::REC_BYTES, at[1]);
        }
    }

    // term-major order: consecutive matrix-core steps are independent; every
    // element sees lo.hi, hi.lo, hi.hi of each slab, slabs in ascending order
    template <int FM, int FN>
    static __device__ __forceinline__ void mma(const Frags<FM, FN> &f, f32x16_t (&acc)[FM][FN]) {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.al[a], f.bh[b], acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[a], f.bl[b], acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.ah[a], f.bh[b], acc[a][b], 0, 0, 0);
    }
};

ring::Operands split_operands(const uint8_t *Ap, const uint8_t *Bp, float *C, int64_t m, int64_t p,
                              int64_t S, int accumulate) {
    ring::Operands op;
    op.a0 = Ap; op.a1 = nullptr;
    op.b0 = Bp; op.b1 = nullptr;
    op.C = C;
    op.row_exp = op.col_exp = nullptr;
    op.m = m; op.p = p; op.S = S;
    op.accumulate = accumulate;
    return op;
}

// ------------------------------------------------------- grouped (persistent)
// Independent products share one launch. Members are listed longest k walk
// first; their tiles form one work list (member g owns tile ids
// [first[g], first[g+1])), and persistent workgroups claim tile ids from an
// atomic counter until the list is exhausted. Grouped members skip the
// conditioning pass: every tile is a block of raw_gemm.h, so grouped and single
// results are bitwise equal, whichever kernel and block shape run.
struct GroupMember {
    SplitItem item;
    int32_t tiles_n;
    int64_t first_tile;                 // first contraction work-list id of this item
};

// Work-list claims, XCD by XCD. The tile list is cut into eight segments of
// about equal work, one per XCD (workgroups go to the XCDs round-robin by id),
// each a run of whole members, so that the tiles sharing a member's rows and
// columns run under one L2. A workgroup claims from its own XCD's segment
// (counter 4 x, bounds[x] .. bounds[x + 1]) and, once that is drained, from
// the next XCDs' in turn; `seg` counts the segments it found drained. Called
// by one thread; -1: nothing left anywhere.
__device__ __forceinline__ int64_t claim_tile(unsigned long long *ctr, const int64_t *bounds, int &seg) {
    const int xcd = blockIdx.x & 7;
    while (seg < 8) {
        const int x = (xcd + seg) & 7;
        const int64_t t = bounds[x] + (int64_t)atomicAdd(ctr + 4 * x, 1ull);
        if (t < bounds[x + 1]) return t;
        ++seg;
    }
    return -1;
}

template <int BM, int BN, int WM, int WN, int NST>
__device__ __forceinline__ void grouped_tile(const GroupMember &g, int64_t local, uint8_t *lds) {
    const int64_t tm = local / g.tiles_n, tn = local - tm * g.tiles_n;
    const SplitItem &d = g.item;
    const raw::Operands op{d.A, d.B, d.C, d.m, d.n, d.p, d.ld, d.accumulate};
    raw::block<BM, BN, WM, WN, NST, true, false>(op, __builtin_amdgcn_readfirstlane((int)tm) * (int64_t)BM,
                                                 __builtin_amdgcn_readfirstlane((int)tn) * (int64_t)BN, lds);
}

template <int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__(256, 2) void split_grouped_kernel(const GroupMember *__restrict__ g,
                                                               const int32_t *__restrict__ tile_owner,
                                                               const int64_t *__restrict__ bounds,
                                                               unsigned long long *__restrict__ counter) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[raw::Cfg<BM, BN, WM, WN, NST>::LDS];
    // the claimed tile id lives in the ring's last slot, whose first load is
    // issued behind the tile's first barrier
    int64_t *s_tile = reinterpret_cast<int64_t *>(lds + (NST - 1) * raw::Cfg<BM, BN, WM, WN, NST>::STAGE);
    int seg = 0;
    for (;;) {
        __syncthreads();                // nobody still reads the ring
        if (threadIdx.x == 0) *s_tile = claim_tile(counter, bounds, seg);
        __syncthreads();
        const int64_t claimed = *s_tile;
        const int64_t tile = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)claimed) |
                                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(claimed >> 32)) << 32);
        if (tile < 0) break;
        const int k = __builtin_amdgcn_readfirstlane(tile_owner[tile]);
        grouped_tile<BM, BN, WM, WN, NST>(g[k], tile - g[k].first_tile, lds);
    }
}

// Sums of the split members' chunk partials: block b works on the last member
// whose first_block is at most b, 1024 elements per block.
constexpr int SUM_BLOCK = 1024;
__global__ __launch_bounds__(256) void split_sums_kernel(const SplitSum *__restrict__ sums, int count, int64_t total) {
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= total) return;
    int k = 0;
    while (k + 1 < count && sums[k + 1].first_block <= block) ++k;
    const SplitSum d = sums[__builtin_amdgcn_readfirstlane(k)];
    const int64_t x0 = (block - d.first_block) * SUM_BLOCK;
    if (d.mp % 4 == 0 && (uintptr_t)d.C % 16 == 0) {
        const int64_t x = x0 + threadIdx.x * 4;
        if (x < d.mp) ring::splitk_sum<4>(d.partials, d.chunks, d.mp, x, d.C, 0, nullptr, d.accumulate);
    } else {
#pragma unroll
        for (int e = 0; e < SUM_BLOCK / 256; ++e) {
            const int64_t x = x0 + e * 256 + threadIdx.x;
            if (x < d.mp) ring::splitk_sum<1>(d.partials, d.chunks, d.mp, x, d.C, 0, nullptr, d.accumulate);
        }
    }
}

// Standalone conditioning kernel: hi/lo planes of a row-major FP32 array.
__global__ __launch_bounds__(256) void split_only_kernel(const float *__restrict__ X, int64_t count,
                                                         uint16_t *__restrict__ hi,
                                                         uint16_t *__restrict__ lo) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * 2;
    for (int64_t t = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 2; t < count; t += stride) {
        const float x0 = X[t];
        const float x1 = (t + 1 < count) ? X[t + 1] : 0.0f;
        uint32_t h, l;
        split_pair(x0, x1, &h, &l);
        hi[t] = (uint16_t)(h & 0xFFFF);
        lo[t] = (uint16_t)(l & 0xFFFF);
        if (t + 1 < count) {
            hi[t + 1] = (uint16_t)(h >> 16);
            lo[t + 1] = (uint16_t)(l >> 16);
        }
    }
}

struct SplitShape { int bm, bn, wm, wn, stages; };
// (deeper rings were measured no faster for this path at N = 8192). The
// rectangular blocks run four waves of 128 x 64 or 64 x 128, two workgroups
// per CU.
constexpr SplitShape kSplit[] = {{128, 128, 64, 64, 3}, {256, 256, 128, 64, 3}, {256, 128, 128, 64, 3},
                                 {128, 256, 64, 128, 3}};

template <int BM, int BN, int WM, int WN, int NST>
hipError_t launch_shape(const moa_gemm_desc &d, const uint8_t *Ap, const uint8_t *Bp, int64_t S,
                        hipStream_t st) {
    const ring::Operands op = split_operands(Ap, Bp, static_cast<float *>(d.C), d.m, d.p, S, d.accumulate);
    const int tiles_m = (int)((d.m + BM - 1) / BM);
    const int tiles_n = (int)((d.p + BN - 1) / BN);
    hipLaunchKernelGGL((ring::single_kernel<BM, BN, WM, WN, 1, SplitMode, NST>), dim3(tiles_m * tiles_n),
                       dim3(ring::Cfg<BM, BN, WM, WN, 1, NST>::THREADS), 0, st, op, tiles_m, tiles_n);
    return hipGetLastError();
}

// Blocks of the kernel without conditioning, and what one 16-k step of them
// takes on a CU that holds b of them: fixed + b * each, in ns (fitted to
// 512^3 .. 3072^3 and 1531 x 2029 x 1237; one to nine blocks per CU).
struct RawBlock { int bm, bn; double fixed, each; };
constexpr RawBlock kRaw[] = {{64, 64, 130, 150}, {64, 128, 130, 240}, {128, 64, 130, 240}, {128, 128, 100, 380}};

template <int BM, int BN, int WM, int WN, int NST>
hipError_t launch_raw(const moa_gemm_desc &d, hipStream_t st) {
    const raw::Operands op{static_cast<const float *>(d.A), static_cast<const float *>(d.B), static_cast<float *>(d.C),
                           d.m, d.n, d.p, d.n, d.accumulate};
    const int tiles_m = (int)((d.m + BM - 1) / BM), tiles_n = (int)((d.p + BN - 1) / BN);
    const dim3 grid((unsigned)(tiles_m * tiles_n)), bl(256);
    const bool a_kc = !(d.flags & MOA_FLAG_A_COL), b_kc = (d.flags & MOA_FLAG_B_COL) != 0;
    if (a_kc && b_kc)
        hipLaunchKernelGGL((raw::single_kernel<BM, BN, WM, WN, NST, true, true>), grid, bl, 0, st, op, tiles_m, tiles_n);
    else if (a_kc)
        hipLaunchKernelGGL((raw::single_kernel<BM, BN, WM, WN, NST, true, false>), grid, bl, 0, st, op, tiles_m, tiles_n);
    else if (b_kc)
        hipLaunchKernelGGL((raw::single_kernel<BM, BN, WM, WN, NST, false, true>), grid, bl, 0, st, op, tiles_m, tiles_n);
    else
        hipLaunchKernelGGL((raw::single_kernel<BM, BN, WM, WN, NST, false, false>), grid, bl, 0, st, op, tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace

// Split-k without conditioning: 128 x 128 blocks, chunks summed in order.
hipError_t launch_raw_splitk(const moa_gemm_desc &d, int chunks, float *partials, hipStream_t st) {
    const raw::Operands op{static_cast<const float *>(d.A), static_cast<const float *>(d.B), static_cast<float *>(d.C),
                           d.m, d.n, d.p, d.n, 0};
    const int tiles_m = (int)((d.m + 127) / 128), tiles_n = (int)((d.p + 127) / 128);
    const int S = (int)((d.n + SLAB - 1) / SLAB), per = (S + chunks - 1) / chunks;
    const dim3 grid((unsigned)(tiles_m * tiles_n * chunks)), bl(256);
    const bool a_kc = !(d.flags & MOA_FLAG_A_COL), b_kc = (d.flags & MOA_FLAG_B_COL) != 0;
    if (a_kc && b_kc)
        hipLaunchKernelGGL((raw::splitk_kernel<128, 128, 64, 64, 3, true, true>), grid, bl, 0, st, op, tiles_m, tiles_n,
                           per, partials);
    else if (a_kc)
        hipLaunchKernelGGL((raw::splitk_kernel<128, 128, 64, 64, 3, true, false>), grid, bl, 0, st, op, tiles_m, tiles_n,
                           per, partials);
    else if (b_kc)
        hipLaunchKernelGGL((raw::splitk_kernel<128, 128, 64, 64, 3, false, true>), grid, bl, 0, st, op, tiles_m, tiles_n,
                           per, partials);
    else
        hipLaunchKernelGGL((raw::splitk_kernel<128, 128, 64, 64, 3, false, false>), grid, bl, 0, st, op, tiles_m, tiles_n,
                           per, partials);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return ring::launch_splitk_reduce(partials, chunks, d.m, d.p, static_cast<float *>(d.C), nullptr, nullptr,
                                      d.accumulate, st);
}

// The block a product takes without conditioning, -1 for the conditioned path:
// the one whose busiest CU is done first, unless the record ring, whose step is
// shorter, makes up for its conditioning (two launches, each operand read and
// written once at 4.6 TB/s); beyond three 128 x 128 blocks per CU the ring's
// larger blocks always do (us, without / with conditioning: 192 x 320 x 160 8 /
// 26, 1024^3 21 / 38, 2048^3 64 / 68, 3072 x 1024 x 3072 79 / 82, 2560^3 124 /
// 112, 2048 x 8192 x 2048 239 / 223, 3072^3 227 / 192, 4096^3 434 / 343). Operands
// whose offsets inside a block exceed 32 bits stay on the conditioned path.
int split_raw_block(const moa_gemm_desc &d) {
    if (((d.m + 127) / 128) * ((d.p + 127) / 128) > 3 * kNumCUs) return -1;
    int best = -1;
    double best_ns = 0;
    for (int v = 0; v < (int)(sizeof(kRaw) / sizeof(kRaw[0])); ++v) {
        const RawBlock r = kRaw[v];
        const int64_t lim = 0x7FFFFFFF / 4;
        const int64_t a = (d.flags & MOA_FLAG_A_COL) ? (raw::SLAB + 1) * d.m : (int64_t)(r.bm + 1) * d.n;
        const int64_t b = (d.flags & MOA_FLAG_B_COL) ? (int64_t)(r.bn + 1) * d.n : (raw::SLAB + 1) * d.p;
        if (a >= lim || b >= lim || 9 * d.p >= lim) continue;
        const int64_t blocks = ((d.m + r.bm - 1) / r.bm) * ((d.p + r.bn - 1) / r.bn);
        const double ns = r.fixed + (double)((blocks + kNumCUs - 1) / kNumCUs) * r.each;
        if (best < 0 || ns < best_ns) {
            best = v;
            best_ns = ns;
        }
    }
    // the ring's 128 x 128 blocks: fitted like kRaw
    const double slabs = (double)((d.n + SLAB - 1) / SLAB);
    const double rounds = (double)((((d.m + 127) / 128) * ((d.p + 127) / 128) + kNumCUs - 1) / kNumCUs);
    const double records = 20000 + 8.0 * (double)d.n * (double)(d.m + d.p) / 4600 + slabs * (80 + 235 * rounds);
    return slabs * best_ns <= records ? best : -1;
}

// Split-k products: likewise, at most three 128 x 128 blocks per CU (512 x 32768
// x 512 in 32 chunks: 73 us without, 119 with conditioning).
bool split_raw_splitk(const moa_gemm_desc &d) {
    const int64_t lim = 0x7FFFFFFF / 4;
    const int64_t a = (d.flags & MOA_FLAG_A_COL) ? (raw::SLAB + 1) * d.m : (int64_t)129 * d.n;
    const int64_t b = (d.flags & MOA_FLAG_B_COL) ? (int64_t)129 * d.n : (raw::SLAB + 1) * d.p;
    return ((d.m + 127) / 128) * ((d.p + 127) / 128) <= 3 * kNumCUs && a < lim && b < lim && 9 * d.p < lim;
}

int64_t split_raw_check(const moa_gemm_desc &d, int block, int chunks, int64_t *loads) {
    const int64_t S = (d.n + SLAB - 1) / SLAB, window = (S + chunks - 1) / chunks * SLAB;
    const bool a_kc = !(d.flags & MOA_FLAG_A_COL), b_kc = (d.flags & MOA_FLAG_B_COL) != 0;
    int64_t bad = 0, seen = 0;
    auto check = [&](int width, bool kc, int64_t extent, int64_t k0, int64_t n) {
        const int64_t size = kc ? extent * d.n - k0 : extent * (d.n - k0);
        if (width == 64)
            bad += kc ? raw::check_operand<64, true>(extent, n, d.n, size, &seen)
                      : raw::check_operand<64, false>(extent, n, d.n, size, &seen);
        else
            bad += kc ? raw::check_operand<128, true>(extent, n, d.n, size, &seen)
                      : raw::check_operand<128, false>(extent, n, d.n, size, &seen);
    };
    for (int64_t c = 0; c < chunks; c += std::max(chunks - 1, 1)) {      // the first chunk and the last
        const int64_t k0 = c * window, n = std::min(window, d.n - k0);
        check(kRaw[block].bm, a_kc, d.m, k0, n);
        check(kRaw[block].bn, b_kc, d.p, k0, n);
    }
    if (loads) *loads = seen;
    return bad;
}

void split_raw_shape(int block, int *rows, int *cols) {
    *rows = kRaw[block].bm;
    *cols = kRaw[block].bn;
}

int split_bf16_variant_count() { return (int)(sizeof(kSplit) / sizeof(kSplit[0])); }

// Default block: 256 x 256 (one workgroup per CU) once it gives every CU a
// block, else 128 x 128. When its blocks fill more than one round of the CUs
// but leave the last round less than 40% full, the rectangular blocks (two
// per CU, half the area) shorten that tail: measured N = 6144 and 7168
// (2.25 and 3.06 rounds) 7-9% faster, while 256 x 256 stays ahead at whole
// or well-filled rounds (N = 4096, 5120, 8192, 12288).
int split_bf16_default_variant(int64_t m, int64_t p) {
    const int64_t big = ((m + 255) / 256) * ((p + 255) / 256);
    if (big < kNumCUs) return 0;
    const int64_t tail = big % kNumCUs;
    if (big > kNumCUs && tail != 0 && 10 * tail < 4 * kNumCUs) return p >= m ? 3 : 2;
    return 1;
}

int64_t split_bf16_workspace_bytes(int64_t m, int64_t n, int64_t p) {
    const int64_t S = (n + SLAB - 1) / SLAB;
    return ring::array_bytes(m, S) + ring::array_bytes(p, S);
}

void split_bf16_shape(int v, Plan *p) {
    const SplitShape s = kSplit[v];
    p->variant = v;
    p->tile_m = s.bm;
    p->tile_n = s.bn;
    p->tile_k = SLAB;
    p->wave_m = s.wm;
    p->wave_n = s.wn;
    p->lane_m = p->lane_n = 0;
    p->threads = (s.bm / s.wm) * (s.bn / s.wn) * 64;
    p->lds_bytes = s.stages * (s.bm + s.bn) * REC_BYTES;
}

namespace {
// Records of the `rows` rows of a row-major rows x K array.
void rows_records(const float *X, int64_t rows, int64_t K, int64_t S, uint8_t *P, hipStream_t st) {
    int64_t blocks = (padded_rows(rows) * S * 2 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, X, rows, K, S, P);
}
// Records of the `cols` columns of a row-major K x cols array.
void cols_records(const float *X, int64_t K, int64_t cols, int64_t S, uint8_t *P, hipStream_t st) {
    const int64_t by = ((S + 3) / 4 + COL_BLOCKS - 1) / COL_BLOCKS;
    hipLaunchKernelGGL(pack_cols_kernel, dim3((unsigned)((cols + 63) / 64), (unsigned)(by < 65535 ? by : 65535)),
                       dim3(256), 0, st, X, K, cols, S, P);
}
}  // namespace

// Records of A's rows and B's columns. A column-major A (element (i, k) at
// i + k m) is a row-major n x m array whose columns are A's rows; a
// column-major B is a row-major p x n array whose rows are B's columns.
hipError_t launch_split_pack(const moa_gemm_desc &d, void *ws, hipStream_t st) {
    const int64_t S = (d.n + SLAB - 1) / SLAB;
    uint8_t *Ap = static_cast<uint8_t *>(ws);
    uint8_t *Bp = Ap + ring::array_bytes(d.m, S);
    const float *A = static_cast<const float *>(d.A);
    const float *B = static_cast<const float *>(d.B);
    if (S == 0) return hipSuccess;
    if (d.flags & MOA_FLAG_A_COL) cols_records(A, d.n, d.m, S, Ap, st);
    else rows_records(A, d.m, d.n, S, Ap, st);
    if (d.flags & MOA_FLAG_B_COL) rows_records(B, d.p, d.n, S, Bp, st);
    else cols_records(B, d.n, d.p, S, Bp, st);
    return hipGetLastError();
}

hipError_t launch_split_bf16(const moa_gemm_desc &d, const Plan &plan, void *ws, hipStream_t st) {
    if (plan.raw_block >= 0) {
        TraceScope ts(MOA_K_SPLIT_BF16, st);
        if (plan.split_k > 1)
            return launch_raw_splitk(d, plan.split_k,
                                     reinterpret_cast<float *>(static_cast<char *>(ws) + plan.partial_offset), st);
        switch (plan.raw_block) {
        case 0: return launch_raw<64, 64, 32, 32, 4>(d, st);
        case 1: return launch_raw<64, 128, 32, 64, 3>(d, st);
        case 2: return launch_raw<128, 64, 64, 32, 3>(d, st);
        default: return launch_raw<128, 128, 64, 64, 3>(d, st);
        }
    }
    hipError_t e;
    {
        TraceScope ts(MOA_K_SPLIT_PACK, st);
        e = launch_split_pack(d, ws, st);
    }
    if (e != hipSuccess) return e;
    TraceScope ts(MOA_K_SPLIT_BF16, st);
    const int64_t S = (d.n + SLAB - 1) / SLAB;
    const uint8_t *Ap = static_cast<const uint8_t *>(ws);
    const uint8_t *Bp = Ap + ring::array_bytes(d.m, S);
    if (plan.split_k > 1) {
        const ring::Operands op = split_operands(Ap, Bp, static_cast<float *>(d.C), d.m, d.p, S, d.accumulate);
        float *partials = reinterpret_cast<float *>(static_cast<char *>(ws) + plan.partial_offset);
        return ring::launch_splitk<128, 128, 64, 64, 1, SplitMode, 3>(op, plan.split_k, partials, st);
    }
    switch (plan.variant) {
    case 0: return launch_shape<128, 128, 64, 64, 3>(d, Ap, Bp, S, st);
    case 2: return launch_shape<256, 128, 128, 64, 3>(d, Ap, Bp, S, st);
    case 3: return launch_shape<128, 256, 64, 128, 3>(d, Ap, Bp, S, st);
    default: return launch_shape<256, 256, 128, 64, 3>(d, Ap, Bp, S, st);
    }
}

namespace {
__global__ void zero_counters_kernel(unsigned long long *x) {
    if (threadIdx.x < 8) x[4 * threadIdx.x] = 0ull;
}
constexpr int GB_M = 128;              // largest grouped block rows

// Persistent kernels of a grouped launch: block, workgroups per CU, weight of a
// slab step of a block in groups of short k walks, and for longer ones the time
// of a launch (us): fixed + step x (slab steps per CU) + walk x (slabs of the
// longest walk) + wg x (workgroups per CU: they claim their tiles one after
// another). Fitted to 90 groups of 4 to 396 products of 32 .. 2048 (n to 4096),
// uniform and mixed.
struct GroupedKernel { int bm, bn, occ; double weight, fixed, step, walk, wg; };
constexpr GroupedKernel kGroupedK[] = {
    {128, 128, 2, 1.0, 18.5, 0.423, 0.303, 6.98},   // 0: five stages
    {64, 64, 4, 0.0, 17.8, 0.210, 0.128, 8.11},     // 1 (longer walks only)
    {128, 128, 2, 1.0, 18.5, 0.423, 0.303, 6.98},   // 2: three stages
    {64, 128, 3, 0.8, 18.3, 0.284, 0.200, 7.37},    // 3
    {128, 64, 4, 0.8, 17.8, 0.357, 0.244, 7.19},    // 4
};
constexpr int kGroupedVariants = (int)(sizeof(kGroupedK) / sizeof(kGroupedK[0]));
int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }

int64_t item_tiles(const SplitItem &d, int bm, int bn) { return ((d.m + bm - 1) / bm) * ((d.p + bn - 1) / bn); }
int64_t item_slabs(const SplitItem &d) { return (d.n + SLAB - 1) / SLAB; }

// The table: items, then the nine segment bounds of the XCD claims (int64, 256
// bytes), the sums of the split members, and the tile -> item table (int32),
// sized for 64 x 64 blocks (at least as many tiles as every block of the list):
// the part a launch uses is one prefix.
struct TableAt { int64_t bounds, sums, owner, bytes; };
TableAt table_at(const SplitGroup &g) {
    TableAt t;
    t.bounds = align256((int64_t)(g.items.size() * sizeof(GroupMember)));
    t.sums = t.bounds + 256;
    t.owner = t.sums + align256((int64_t)(g.sums.size() * sizeof(SplitSum)));
    int64_t tiles = 0;
    for (const SplitItem &d : g.items) tiles += item_tiles(d, 64, 64);
    t.bytes = t.owner + align256(4 * tiles);
    return t;
}
}  // namespace

// The raw ring addresses a tile's rows of A with 32-bit offsets (128 rows of
// n FP32) and a slab of B likewise (16 rows of p FP32).
bool split_grouped_fits(const moa_gemm_desc &d) {
    return ((int64_t)GB_M + 1) * d.n * 4 < 0x7FFFFFFF && ((int64_t)SLAB + 1) * d.p * 4 < 0x7FFFFFFF;
}

void split_group_add(SplitGroup &g, const moa_gemm_desc &d, int split_k, float *partials) {
    SplitItem it{static_cast<const float *>(d.A), static_cast<const float *>(d.B), static_cast<float *>(d.C),
                 d.m, d.n, d.p, d.n, d.accumulate};
    if (split_k <= 1) {
        g.items.push_back(it);
        return;
    }
    const int64_t S = (d.n + SLAB - 1) / SLAB, window = (S + split_k - 1) / split_k * SLAB;
    for (int c = 0; c < split_k; ++c) {
        const int64_t k0 = c * window;
        it.A = static_cast<const float *>(d.A) + k0;
        it.B = static_cast<const float *>(d.B) + k0 * d.p;
        it.C = partials ? partials + (int64_t)c * d.m * d.p : nullptr;
        it.n = std::min(window, d.n - k0);
        it.accumulate = 0;
        g.items.push_back(it);
    }
    g.sums.push_back({partials, static_cast<float *>(d.C), d.m * d.p, split_k, d.accumulate, 0});
}

int64_t split_grouped_table_bytes(const SplitGroup &g) { return table_at(g).bytes; }

int64_t split_grouped_workspace_bytes(const SplitGroup &g) { return 256 + split_grouped_table_bytes(g); }

int split_grouped_variant_count() { return kGroupedVariants; }

// Static rule. Short k walks (below 32 slabs): the block among 128 x 128, 64 x
// 128 and 128 x 64 with the fewest slab steps over the items, weighted by what a
// tile takes: half a block costs 0.8 of a whole one or more, C and the change of
// tiles included (43 products of 137 x 67 x 1192: 47.5 us with 128 x 128 blocks, 59
// with 64 x 128, which have 1.5 times the tiles; 62 of 43 x 14 x 967, the same
// tiles, 40.3 and 39.5). Longer ones: the block with the shortest estimated launch, 64 x
// 64 among them -- a group that leaves CUs idle is as slow as its longest walk
// (4 products, the longest walk 197 slabs: 97 us with 128 x 128 blocks, 68 with 64 x
// 64), a large one pays for every step (64 products of 64 .. 2048: 232 us with 128 x 128
// blocks, 271 with 64 x 128, 348 with 64 x 64). Over the fitted groups the choice
// takes 2% longer than the best block on average and 16% at most. Ties to the
// earlier variant in the list; variant 0 is left to the autotuner.
int split_grouped_default_variant(const SplitGroup &g) {
    // slab steps and tiles of every block, in shifts: the rule runs on each call
    double steps[kGroupedVariants] = {}, tiles[kGroupedVariants] = {};
    int64_t longest = 0;
    for (const SplitItem &d : g.items) {
        const int64_t slabs = item_slabs(d);
        const int64_t m64 = (d.m + 63) / 64, m128 = (d.m + 127) / 128, p64 = (d.p + 63) / 64, p128 = (d.p + 127) / 128;
        const int64_t t[kGroupedVariants] = {m128 * p128, m64 * p64, m128 * p128, m64 * p128, m128 * p64};
        longest = std::max(longest, slabs);
        for (int v = 0; v < kGroupedVariants; ++v) {
            tiles[v] += (double)t[v];
            steps[v] += (double)t[v] * (double)slabs;
        }
    }
    int best = 2;
    double best_cost = 0;
    for (int v : {2, 3, 4, 1}) {
        if (v == 1 && longest < 32) continue;
        const GroupedKernel k = kGroupedK[v];
        const double cost = longest < 32 ? steps[v] * k.weight
                                         : k.fixed + k.step * steps[v] / kNumCUs + k.walk * (double)longest +
                                               k.wg * std::min(tiles[v] / kNumCUs, (double)k.occ);
        if (v == 2 || cost < best_cost) {
            best = v;
            best_cost = cost;
        }
    }
    return best;
}

// Lays out the items in `host_staging` for grouped kernel `variant`. Items are
// dealt, heaviest first (tiles x slab steps), to the lightest of eight XCD
// segments; inside a segment they run longest k walk first, so each segment's
// tail holds its cheapest tiles. On the device the claim counters are at the
// workspace's start and the table 256 bytes behind it.
GroupedWork split_grouped_layout(const SplitGroup &g, void *host_staging, int variant) {
    const GroupedKernel gk = kGroupedK[variant];
    const int count = (int)g.items.size();
    std::vector<int64_t> member_tiles(count);
    std::vector<double> cost(count);
    std::vector<int> heavy(count);
    for (int k = 0; k < count; ++k) {
        heavy[k] = k;
        member_tiles[k] = item_tiles(g.items[k], gk.bm, gk.bn);
        cost[k] = (double)member_tiles[k] * (double)item_slabs(g.items[k]);
    }
    std::stable_sort(heavy.begin(), heavy.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    std::vector<int> seg_of(count);
    double load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int k : heavy) {
        int x = 0;
        for (int y = 1; y < 8; ++y)
            if (load[y] < load[x]) x = y;
        seg_of[k] = x;
        load[x] += cost[k];
    }
    std::vector<int> order(count);
    for (int k = 0; k < count; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        if (seg_of[a] != seg_of[b]) return seg_of[a] < seg_of[b];
        return g.items[a].n > g.items[b].n;
    });
    const TableAt at = table_at(g);
    char *base = static_cast<char *>(host_staging);
    GroupMember *h = reinterpret_cast<GroupMember *>(base);
    int32_t *tile_owner = reinterpret_cast<int32_t *>(base + at.owner);
    int64_t tiles = 0;
    int64_t bounds[9];
    int next_seg = 0;
    for (int q = 0; q < count; ++q) {
        const SplitItem &d = g.items[order[q]];
        while (next_seg <= seg_of[order[q]]) bounds[next_seg++] = tiles;
        GroupMember m{};
        m.item = d;
        m.first_tile = tiles;
        m.tiles_n = (int32_t)((d.p + gk.bn - 1) / gk.bn);
        const int64_t mt = member_tiles[order[q]];
        for (int64_t t = 0; t < mt; ++t) tile_owner[tiles + t] = q;
        tiles += mt;
        h[q] = m;
    }
    while (next_seg <= 8) bounds[next_seg++] = tiles;
    std::memcpy(base + at.bounds, bounds, sizeof(bounds));
    SplitSum *sums = reinterpret_cast<SplitSum *>(base + at.sums);
    int64_t blocks = 0;
    for (size_t k = 0; k < g.sums.size(); ++k) {
        sums[k] = g.sums[k];
        sums[k].first_block = blocks;
        blocks += (g.sums[k].mp + SUM_BLOCK - 1) / SUM_BLOCK;
    }
    return {tiles, blocks, variant, at.owner + 4 * tiles};
}

namespace {
// The persistent contraction of a grouped launch whose table and cleared claim
// counters are in place, and the sums of its split members.
hipError_t launch_persistent(void *ws, const SplitGroup &g, const GroupedWork &work, hipStream_t st) {
    const TableAt at = table_at(g);
    char *base = static_cast<char *>(ws);
    unsigned long long *counter = reinterpret_cast<unsigned long long *>(base);
    const GroupMember *dev_members = reinterpret_cast<const GroupMember *>(base + 256);
    const int64_t *bounds = reinterpret_cast<const int64_t *>(base + 256 + at.bounds);
    const int32_t *tile_owner = reinterpret_cast<const int32_t *>(base + 256 + at.owner);
    const int v = work.variant;
    const int64_t grid = std::min<int64_t>(work.tiles, (int64_t)kGroupedK[v].occ * kNumCUs);   // resident blocks
    TraceScope ts(MOA_K_SPLIT_GROUPED, st);
    if (grid > 0) {
        const dim3 gr((unsigned)grid), bl(256);
        switch (v) {
        case 1:
            hipLaunchKernelGGL((split_grouped_kernel<64, 64, 32, 32, 4>), gr, bl, 0, st, dev_members, tile_owner,
                               bounds, counter);
            break;
        case 2:
            hipLaunchKernelGGL((split_grouped_kernel<128, 128, 64, 64, 3>), gr, bl, 0, st, dev_members, tile_owner,
                               bounds, counter);
            break;
        case 3:
            hipLaunchKernelGGL((split_grouped_kernel<64, 128, 32, 64, 3>), gr, bl, 0, st, dev_members, tile_owner,
                               bounds, counter);
            break;
        case 4:
            hipLaunchKernelGGL((split_grouped_kernel<128, 64, 64, 32, 3>), gr, bl, 0, st, dev_members, tile_owner,
                               bounds, counter);
            break;
        default:
            hipLaunchKernelGGL((split_grouped_kernel<128, 128, 64, 64, 5>), gr, bl, 0, st, dev_members, tile_owner,
                               bounds, counter);
            break;
        }
    }
    if (work.sum_blocks > 0)
        hipLaunchKernelGGL(split_sums_kernel, item_grid(work.sum_blocks), dim3(256), 0, st,
                           reinterpret_cast<const SplitSum *>(base + 256 + at.sums), (int)g.sums.size(),
                           work.sum_blocks);
    return hipGetLastError();
}

// Uploads the used prefix of a member table (n16 16-byte words) straight from
// pinned host memory mapped into the device's address space, and clears the
// claim counters: one small kernel in place of a copy-engine transfer, whose
// hand-offs to and from the compute queue cost more than the copy.
__global__ __launch_bounds__(256) void stage_table_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                          int64_t n16, unsigned long long *__restrict__ counters) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
    if (blockIdx.x == 0 && threadIdx.x < 8) counters[4 * threadIdx.x] = 0ull;
}
}  // namespace

// The device part of a grouped launch whose table is already on the device:
// clear the claim counters, run the persistent contraction. Contains no
// allocation, copy or memset, so it can be captured in a graph and replayed.
hipError_t split_grouped_enqueue(void *ws, const SplitGroup &g, const GroupedWork &work, hipStream_t st) {
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, st, static_cast<unsigned long long *>(ws));
    return launch_persistent(ws, g, work, st);
}

hipError_t launch_split_grouped(const SplitGroup &g, int variant, void *ws, void *host_staging,
                                const void *host_staging_dev, hipStream_t st) {
    if (g.items.empty()) return hipSuccess;
    const GroupedWork work = split_grouped_layout(g, host_staging, variant);
    char *base = static_cast<char *>(ws);
    if (!host_staging_dev) {
        hipError_t e = hipMemcpyAsync(base + 256, host_staging, (size_t)work.table_used, hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return e;
        return split_grouped_enqueue(ws, g, work, st);
    }
    const int64_t n16 = (work.table_used + 15) / 16;
    const int64_t blocks = std::min<int64_t>((n16 + 255) / 256, 64);
    hipLaunchKernelGGL(stage_table_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint4 *>(host_staging_dev), reinterpret_cast<uint4 *>(base + 256), n16,
                       reinterpret_cast<unsigned long long *>(base));
    return launch_persistent(ws, g, work, st);
}

hipError_t launch_split_only(const float *X, int64_t count, uint16_t *hi, uint16_t *lo,
                             hipStream_t st) {
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count / 2 + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(split_only_kernel, dim3((unsigned)blocks), dim3(256), 0, st, X, count, hi, lo);
    return hipGetLastError();
}

}  // namespace moa
