// Power-of-two scaled FP8 path. Eq. 3 is invariant under C = D_r^-1 ((D_r A)
// (B D_c)) D_c^-1 for diagonal D_r = diag(2^e_i), D_c = diag(2^f_j): the
// scales factor out of the k-sum, so they are applied exactly before rounding
// the operands to OCP E4M3 and removed exactly (ldexp) in the epilogue.
//
//   e_i = largest integer with amax_k |A[i,k]| * 2^e_i <= 448 (0 if the row
//         is zero); f_j likewise for column j of B.
//   qA[i,k] = RNE_e4m3(A[i,k] 2^e_i),  qB[k,j] = RNE_e4m3(B[k,j] 2^f_j)
//   C[i,j] = 2^-(e_i+f_j) sum_k qA[i,k] qB[k,j]          (one term)
// With the residual term r = x 2^e - q (exact in FP32) kept as
// l = RNE_e4m3(2^4 r):
//   C[i,j] = 2^-(e_i+f_j) (sum qA qB + 2^-4 (sum qA lB + sum lA qB))
// The factor 2^-4 is the E8M0 block scale of the residual operand of the
// scaled matrix-core step, so all three sums share one FP32 accumulator.
//
// Conditioning (HBM-bound), straight into record tiles (layout in ring_gemm.h):
// record (r, s) holds the 64 codes of k = 64s .. 64s+63 of row r of A, or of
// column r of B. Rows of up to 8192 values are conditioned in one pass, a wave
// per row that holds the row in registers: amax, exponent, codes (longer rows:
// exponents first, then codes). Columns take two: column amax (atomic max on
// the bit patterns of |x|, which order like unsigned ints), then the codes,
// transposed on the way. The two-term path keeps the residual codes in a second
// record array per operand. The
// contraction is the record-tile ring of ring_gemm.h with
// v_mfma_scale_f32_32x32x64_f8f6f4 steps.
#include <algorithm>
#include <vector>

#include "moa_internal.h"
#include "ring_gemm.h"
#include "tile_common.h"

namespace moa {
namespace {

using ring::GROUP;
using ring::padded_rows;
using ring::REC_BYTES;

constexpr int SLAB8 = 64;                // k per record: 64 E4M3 codes
static_assert(REC_BYTES == SLAB8, "one record holds one slab of codes");
// E8M0 block scales of the scaled matrix-core step: 2^(x - 127).
constexpr int kScaleOne = 0x7f;          // 2^0 (0 would mean 2^-127)
constexpr int kScaleLo = 0x7f - 4;       // 2^-4: residual codes carry a factor 2^4


__device__ __forceinline__ int pow2_exponent(float amax) {
    if (!(amax > 0.0f)) return 0;
    int E;
    const float f = frexpf(amax, &E);   // amax = f 2^E, f in [0.5, 1)
    // 448 = 0.875 * 2^9: f 2^(E+e) <= 0.875 2^9 decides e exactly.
    return (f <= 0.875f) ? 9 - E : 8 - E;
}

// Four values -> four E4M3 codes (round to nearest even), byte t = value t.
__device__ __forceinline__ uint32_t e4m3x4(float a, float b, float c, float d) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
    return (uint32_t)w;
}

__device__ __forceinline__ float e4m3_value(uint32_t word, int byte) {
    switch (byte) {
    case 0: return __builtin_amdgcn_cvt_f32_fp8((int)word, 0);
    case 1: return __builtin_amdgcn_cvt_f32_fp8((int)word, 1);
    case 2: return __builtin_amdgcn_cvt_f32_fp8((int)word, 2);
    default: return __builtin_amdgcn_cvt_f32_fp8((int)word, 3);
    }
}

// hi and (2^4 x residual) codes of four scaled values.
__device__ __forceinline__ void quant4(const float v[4], bool two_term, uint32_t *hi, uint32_t *lo) {
    const uint32_t h = e4m3x4(v[0], v[1], v[2], v[3]);
    *hi = h;
    if (two_term) {
        float r[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) r[t] = ldexpf(v[t] - e4m3_value(h, t), 4);
        *lo = e4m3x4(r[0], r[1], r[2], r[3]);
    }
}

__global__ void fill_u32_kernel(uint32_t *x, int64_t count) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) x[t] = 0u;
}

__device__ __forceinline__ float amax4(const f32x4_t v) {
    return fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
}
__device__ __forceinline__ float wave_max(float mx) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    return mx;
}
// e_i of every row of A, one workgroup per row (at most ROW_BLOCKS: a launch
// holds fewer than 2^32 threads).
constexpr int64_t ROW_BLOCKS = 1 << 20;
__global__ __launch_bounds__(256) void row_exp_kernel(const float *__restrict__ A, int64_t m, int64_t n,
                                                      int32_t *__restrict__ e) {
    __shared__ float part[4];
    for (int64_t i = blockIdx.x; i < m; i += gridDim.x) {
        const float *row = A + i * n;
        float mx = 0.0f;
#pragma unroll 8
        for (int64_t k = (int64_t)threadIdx.x * 4; k < n; k += 1024) mx = fmaxf(mx, amax4(row4(row, k, n)));
        mx = wave_max(mx);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mx;
        __syncthreads();
        if (threadIdx.x == 0) e[i] = pow2_exponent(fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3])));
        __syncthreads();                           // part free for the next row
    }
}

// Column amax of B: a workgroup takes 256 columns (four per lane) over a band
// of COL_BAND rows, a quarter of the band per wave, all its loads in flight at
// once, and adds one atomic per column. HBM-bound for large operands (4096 x
// 8192: 34 us); a small one takes the latency of one round of loads (1000 x
// 1000: 4.1 us; with 64 rows per wave 14.9, with one column per lane 9.5).
constexpr int COL_BAND = 64;
__device__ __forceinline__ void col_amax_block(const float *__restrict__ B, int64_t n, int64_t p, int64_t bx,
                                               int64_t by, uint32_t *__restrict__ amax, float (*part)[256]) {
    constexpr int R = COL_BAND / 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t j = bx * 256 + lane * 4;
    const int64_t k0 = by * COL_BAND + wave * R;
    f32x4_t x[R], mx = {0.0f, 0.0f, 0.0f, 0.0f};
    if (k0 + R <= n && j + 4 <= p) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = load4(B + (k0 + r) * p + j);
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            x[r] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if (k0 + r < n) x[r] = row4(B + (k0 + r) * p, j, p);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t) mx[t] = fmaxf(mx[t], fabsf(x[r][t]));
    __syncthreads();                               // earlier readers of `part` are done
    *reinterpret_cast<f32x4_t *>(&part[wave][lane * 4]) = mx;
    __syncthreads();
    const int c = threadIdx.x;
    const float m = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
    if (bx * 256 + c < p) atomicMax(&amax[bx * 256 + c], __float_as_uint(m));
}

__global__ __launch_bounds__(256) void col_amax_kernel(const float *__restrict__ B, int64_t n,
                                                       int64_t p, uint32_t *__restrict__ amax) {
    __shared__ __attribute__((aligned(16))) float part[4][256];
    for (int64_t by = blockIdx.y; by * COL_BAND < n; by += gridDim.y) col_amax_block(B, n, p, blockIdx.x, by, amax, part);
}

// --------------------------------------------------- record conditioning --

// One wave: row i of A (rows past m up to the padded end: zeros) held in
// registers, J x 256 values; exponent, then the codes as one dword per four
// values, 16 lanes filling a record. n <= 256 J. One read of the operand and one
// launch in place of two each; all of a lane's loads are in flight together, at
// any 4-byte alignment (3001 x 2777 rows: exponents and codes were 15 + 13.5 us
// with scalar loads for the odd length, the product of two such operands, one
// term, 99 us and now 41).
template <bool TWO, int J>
__device__ __forceinline__ void condition_row(const float *__restrict__ A, int64_t i, int64_t m, int64_t n, int64_t S,
                                              int lane, int32_t *__restrict__ e, uint8_t *__restrict__ qa,
                                              uint8_t *__restrict__ la) {
    f32x4_t x[J];
    float mx = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        x[j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (i < m && 256 * j < n) x[j] = row4(A + i * n, 256 * j + 4 * lane, n);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) mx = fmaxf(mx, amax4(x[j]));
    const int ei = pow2_exponent(wave_max(mx));
    if (lane == 0 && i < m) e[i] = ei;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int64_t s = 4 * j + (lane >> 4);
        if (s >= S) continue;
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = ldexpf(x[j][t], ei);
        uint32_t hi, lo = 0u;
        quant4(v, TWO, &hi, &lo);
        const int64_t at = ring::rec_byte(i, s, S) + 4 * (lane & 15);
        *reinterpret_cast<uint32_t *>(qa + at) = hi;
        if (TWO) *reinterpret_cast<uint32_t *>(la + at) = lo;
    }
}

// The rows of one operand and where they go. `blocks`: workgroups of four rows.
struct RowsJob {
    const float *X;
    int64_t rows, blocks;
    int32_t *e;
    uint8_t *q, *l;
};

// Four rows of n values per workgroup of an item_grid: the rows of one job, then
// those of a second one (no blocks: none). Clears `count` words at `clear` on the
// way (the column amax of an operand taken by columns).
template <bool TWO, int J>
__global__ __launch_bounds__(256) void rows_fp8_kernel(RowsJob first, RowsJob second, int64_t n, int64_t S,
                                                       uint32_t *__restrict__ clear, int64_t count) {
    const int64_t item = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    for (int64_t t = item * 256 + threadIdx.x; t < count; t += (int64_t)gridDim.x * gridDim.y * 256) clear[t] = 0u;
    const bool of_first = item < first.blocks;
    const RowsJob d = of_first ? first : second;
    const int64_t i = (item - (of_first ? 0 : first.blocks)) * 4 + (threadIdx.x >> 6);
    if (i < padded_rows(d.rows)) condition_row<TWO, J>(d.X, i, d.rows, n, S, threadIdx.x & 63, d.e, d.q, d.l);
}

// Rows of A -> records, exponents given. Chunk q = 16 codes of one record (4
// per record); consecutive chunks fill one KiB record tile contiguously.
template <bool TWO>
__device__ __forceinline__ void pack_rows_fp8_chunk(const float *__restrict__ A, int64_t m, int64_t n,
                                                    int64_t S, const int32_t *__restrict__ e,
                                                    uint8_t *__restrict__ qa, uint8_t *__restrict__ la,
                                                    int64_t q) {
    const int c = (int)(q & 3);
    const int64_t rr = (q >> 2) % GROUP;
    const int64_t gs = (q >> 2) / GROUP;
    const int64_t s = gs % S, g = gs / S;
    const int64_t r = g * GROUP + rr;
    const int64_t k = s * SLAB8 + c * 16;
    uint32_t hi[4], lo[4] = {0u, 0u, 0u, 0u};
    const int er = r < m ? e[r] : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        f32x4_t x = {0.0f, 0.0f, 0.0f, 0.0f};
        if (r < m) x = row4(A + r * n, k + 4 * u, n);
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = ldexpf(x[t], er);
        quant4(v, TWO, &hi[u], &lo[u]);
    }
    const int64_t at = ring::rec_byte(r, s, S) + c * 16;
    *reinterpret_cast<uint4 *>(qa + at) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    if (TWO) *reinterpret_cast<uint4 *>(la + at) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

template <bool TWO>
__global__ __launch_bounds__(256) void pack_rows_fp8_kernel(const float *__restrict__ A, int64_t m,
                                                            int64_t n, int64_t S,
                                                            const int32_t *__restrict__ e,
                                                            uint8_t *__restrict__ qa,
                                                            uint8_t *__restrict__ la) {
    const int64_t chunks = padded_rows(m) * S * 4;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < chunks; q += (int64_t)gridDim.x * 256)
        pack_rows_fp8_chunk<TWO>(A, m, n, S, e, qa, la, q);
}

// Columns of B -> records (transposed), 64 columns x one slab (64 k) per
// workgroup step. Thread t reads rows 4(t/16) .. +3 of columns 4(t%16) .. +3
// (each row of the block is 256 contiguous bytes), quantises them, turns the
// 4 x 4 codes around in registers and stores one dword per column into an LDS
// tile (row stride 17 dwords: the 64 lanes of a store hit 64 distinct banks).
// Then thread t writes bytes 16(t%4) .. +15 of the record of column t/4, so a
// wave stores one whole KiB record tile. Column exponents come from the column
// amax; workgroups with blockIdx.y == 0 also store them. Columns past p get
// zero records.
constexpr int TSTRIDE = 17;

__device__ __forceinline__ uint32_t byte_column(const uint32_t w[4], int c) {
    const int sh = 8 * c;
    return ((w[0] >> sh) & 0xFFu) | (((w[1] >> sh) & 0xFFu) << 8) | (((w[2] >> sh) & 0xFFu) << 16) |
           (((w[3] >> sh) & 0xFFu) << 24);
}

// Column exponents of the 64 columns of block bx (threads 0 .. 63).
__device__ __forceinline__ void write_col_exps(const uint32_t *__restrict__ amax, int64_t p, int64_t bx,
                                               int32_t *__restrict__ f_out) {
    const int64_t j = bx * 64 + threadIdx.x;
    if (threadIdx.x < 64 && j < p) f_out[j] = pow2_exponent(__uint_as_float(amax[j]));
}

// Block (bx, s): columns 64 bx .. 64 bx + 63, slab s < S. All 256 threads
// take part; the LDS tiles are free again when it returns.
template <bool TWO>
__device__ __forceinline__ void pack_cols_fp8_block(const float *__restrict__ B, int64_t n, int64_t p,
                                                    int64_t S, const uint32_t *__restrict__ amax,
                                                    uint8_t *__restrict__ qb, uint8_t *__restrict__ lb,
                                                    int64_t bx, int64_t s, uint32_t *tq, uint32_t *tl) {
    const int t = threadIdx.x;
    const int cg = t & 15, kq = t >> 4;
    const int64_t j0 = bx * 64;
    const int64_t j = j0 + 4 * cg;                 // this thread's first column
    int fcol[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) fcol[u] = (j + u < p) ? pow2_exponent(__uint_as_float(amax[j + u])) : 0;
    uint32_t wq[4], wl[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t k = s * SLAB8 + 4 * kq + i;
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k < n) {
            const float *row = B + k * p + j;
            const f32x4_t x = row4(row, 0, p - j);
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = x[u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = ldexpf(v[u], fcol[u]);
        quant4(v, TWO, &wq[i], &wl[i]);
    }
    __syncthreads();                               // earlier readers of the tiles are done
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        tq[(4 * cg + u) * TSTRIDE + kq] = byte_column(wq, u);
        if (TWO) tl[(4 * cg + u) * TSTRIDE + kq] = byte_column(wl, u);
    }
    __syncthreads();
    const int jj = t >> 2, c = t & 3;              // writer: column j0 + jj, chunk c
    if (j0 + jj < padded_rows(p)) {
        const uint32_t *r = tq + jj * TSTRIDE + 4 * c;
        const int64_t at = ring::rec_byte(j0 + jj, s, S) + 16 * c;
        *reinterpret_cast<uint4 *>(qb + at) = make_uint4(r[0], r[1], r[2], r[3]);
        if (TWO) {
            const uint32_t *q = tl + jj * TSTRIDE + 4 * c;
            *reinterpret_cast<uint4 *>(lb + at) = make_uint4(q[0], q[1], q[2], q[3]);
        }
    }
}

template <bool TWO>
__global__ __launch_bounds__(256) void pack_cols_fp8_kernel(const float *__restrict__ B, int64_t n,
                                                            int64_t p, int64_t S,
                                                            const uint32_t *__restrict__ amax,
                                                            int32_t *__restrict__ f_out,
                                                            uint8_t *__restrict__ qb,
                                                            uint8_t *__restrict__ lb) {
    __shared__ uint32_t tq[64 * TSTRIDE];
    __shared__ uint32_t tl[TWO ? 64 * TSTRIDE : 1];
    if (blockIdx.y == 0) write_col_exps(amax, p, blockIdx.x, f_out);
    for (int64_t s = blockIdx.y; s < S; s += gridDim.y)
        pack_cols_fp8_block<TWO>(B, n, p, S, amax, qb, lb, blockIdx.x, s, tq, tl);
}

// ------------------------------------------- row-major codes (exposed API) --

// qA (row-major, like A): 4 consecutive elements per thread.
__global__ __launch_bounds__(256) void quant_rows_kernel(const float *__restrict__ A, int64_t m,
                                                         int64_t n, const int32_t *__restrict__ e,
                                                         int two_term, uint8_t *__restrict__ q,
                                                         uint8_t *__restrict__ l) {
    const int64_t i = blockIdx.x;
    const int64_t k = ((int64_t)blockIdx.y * 256 + threadIdx.x) * 4;
    if (k >= n) return;
    const int ei = e[i];
    float v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = (k + t < n) ? ldexpf(A[i * n + k + t], ei) : 0.0f;
    uint32_t hi, lo = 0;
    quant4(v, two_term != 0, &hi, &lo);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (k + t < n) {
            q[i * n + k + t] = (uint8_t)(hi >> (8 * t));
            if (two_term) l[i * n + k + t] = (uint8_t)(lo >> (8 * t));
        }
}

// qB (row-major, like B): 4 consecutive columns x 4 rows per thread.
__global__ __launch_bounds__(256) void quant_cols_kernel(const float *__restrict__ B, int64_t n,
                                                         int64_t p, const uint32_t *__restrict__ amax,
                                                         int two_term, int32_t *__restrict__ f_out,
                                                         uint8_t *__restrict__ q,
                                                         uint8_t *__restrict__ l) {
    const int64_t k0 = (int64_t)blockIdx.y * 64, jb = (int64_t)blockIdx.x * 64;
    const int tx = threadIdx.x & 15;      // 4 columns each
    const int ty = threadIdx.x >> 4;      // 16 rows, 4 passes
    const int64_t j = jb + tx * 4;
    int f[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        f[t] = (j + t < p) ? pow2_exponent(__uint_as_float(amax[j + t])) : 0;
        if (blockIdx.y == 0 && ty == 0 && j + t < p) f_out[j + t] = f[t];
    }
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int64_t k = k0 + ty + 16 * pass;
        if (k >= n) continue;
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = (j + t < p) ? ldexpf(B[k * p + j + t], f[t]) : 0.0f;
        uint32_t hi, lo = 0;
        quant4(v, two_term != 0, &hi, &lo);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (j + t < p) {
                q[k * p + j + t] = (uint8_t)(hi >> (8 * t));
                if (two_term) l[k * p + j + t] = (uint8_t)(lo >> (8 * t));
            }
    }
}

// ---------------------------------------------------------- contraction --

// Fragments of 32 records x 32 codes: lane l reads row base + l%32, logical
// chunks 2(l/32) and 2(l/32) + 1 (k = 32(l/32) .. +31 of the slab); A and B
// use the same k assignment, which is all the step's dot product needs.
template <bool TWO> struct Fp8Mode {
    static constexpr bool SCALED = true;
    template <int FM, int FN> struct Frags {
        i32x8_t ah[FM], bh[FN], al[TWO ? FM : 1], bl[TWO ? FN : 1];
    };

    static constexpr int TERMS = TWO ? 3 : 1;
    static __device__ __forceinline__ int chunk(int half, int x) { return 2 * half + x; }
    static __device__ __forceinline__ i32x8_t frag(const uint8_t *rows, const int (&at)[2]) {
        const i32x4_t x = *reinterpret_cast<const i32x4_t *>(rows + at[0]);
        const i32x4_t y = *reinterpret_cast<const i32x4_t *>(rows + at[1]);
        return __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
    }

    // LDS rows: [A hi (BM)][A lo (BM)][B hi (BN)][B lo (BN)] (lo: two-term only)
    template <int BM, int BN, int FM, int FN>
    static __device__ __forceinline__ void read(const uint8_t *a_part, const uint8_t *b_part, const int (&at)[2],
                                                Frags<FM, FN> &f) {
#pragma unroll
        for (int a = 0; a < FM; ++a) {
            if constexpr (TWO) f.al[a] = frag(a_part + (BM + a * 32) * ring::REC_BYTES, at);
            f.ah[a] = frag(a_part + a * 32 * ring::REC_BYTES, at);
        }
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            f.bh[b] = frag(b_part + b * 32 * ring::REC_BYTES, at);
            if constexpr (TWO) f.bl[b] = frag(b_part + (BN + b * 32) * ring::REC_BYTES, at);
        }
    }

    // every element sees, per slab in ascending order: 2^-4 lA.qB, 2^-4 qA.lB
    // (two-term only), then qA.qB
    template <int FM, int FN>
    static __device__ __forceinline__ void mma(const Frags<FM, FN> &f, f32x16_t (&acc)[FM][FN]) {
        if constexpr (TWO) {
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        f.al[a], f.bh[b], acc[a][b], 0, 0, 0, kScaleLo, 0, kScaleOne);
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        f.ah[a], f.bl[b], acc[a][b], 0, 0, 0, kScaleOne, 0, kScaleLo);
        }
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    f.ah[a], f.bh[b], acc[a][b], 0, 0, 0, kScaleOne, 0, kScaleOne);
    }
};

// ------------------------------------------------ grouped (persistent) --
// Independent FP8 products of one term count share one launch sequence:
// clear (claim counter + every member's column amax), rows (every member's rows,
// exponents and records, and its column amax), columns (every member's column
// blocks), contraction (persistent workgroups claim tiles of all members from
// one counter). The row and column steps each walk one work list over all
// members, so large and small members share the machine evenly. Every element
// sees the operation sequence of the single-product path, so results are
// bitwise those of moa_gemm.
struct Fp8Member {
    ring::Operands op;                  // the contraction's view (read by ring::tile in place)
    const float *A, *B;
    uint8_t *qa, *la, *qb, *lb;         // record arrays (la, lb: two-term only)
    int32_t *e, *f;                     // row / column exponents
    uint32_t *amaxB;                    // column amax (bit patterns)
    int64_t m, n, p, S;
    int64_t first_tile;                 // first contraction work-list id
    int64_t row_first;                  // first row work-list id
    int64_t col_first;                  // first column work-list id
    float *partials;                    // split k walk: chunk q's sums at partials + q m p
    int64_t sum_first;                  // first block of the summing kernel
    int32_t tiles_n, tiles;             // blocks of a row of C, and of C
    int32_t chunks, chunk_slabs;        // contraction items: `tiles` per chunk of the k walk
    int32_t row_items;                  // row items: row_items (4 rows each), then
    int32_t col_amax_x;                 //   col_amax_x * ceil(n / COL_BAND) column bands
    int32_t col_x;                      // column items: col_x * max(S, 1) 64-column blocks
};

template <int64_t Fp8Member::*F>
__device__ __forceinline__ int find_member(const Fp8Member *__restrict__ g, int count, int64_t item) {
    int lo = 0, hi = count - 1;         // last member whose list starts at or before item
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (g[mid].*F <= item) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// A row of any length by one wave: in registers up to 4096 values (the kernel
// keeps four workgroups a CU), else in two passes over memory.
template <bool TWO>
__device__ __forceinline__ void condition_any_row(const Fp8Member &d, int64_t i, int lane) {
    if (d.n <= 1024) return condition_row<TWO, 4>(d.A, i, d.m, d.n, d.S, lane, d.e, d.qa, d.la);
    if (d.n <= 4096) return condition_row<TWO, 16>(d.A, i, d.m, d.n, d.S, lane, d.e, d.qa, d.la);
    const float *row = d.A + i * d.n;
    float mx = 0.0f;
    if (i < d.m)
#pragma unroll 8
        for (int64_t k = 4 * lane; k < d.n; k += 256) mx = fmaxf(mx, amax4(row4(row, k, d.n)));
    const int ei = pow2_exponent(wave_max(mx));
    if (lane == 0 && i < d.m) d.e[i] = ei;
    for (int64_t k = 4 * lane; k < d.S * SLAB8; k += 256) {
        f32x4_t x = {0.0f, 0.0f, 0.0f, 0.0f};
        if (i < d.m) x = row4(row, k, d.n);
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = ldexpf(x[t], ei);
        uint32_t hi, lo = 0u;
        quant4(v, TWO, &hi, &lo);
        const int64_t at = ring::rec_byte(i, k / SLAB8, d.S) + k % SLAB8;
        *reinterpret_cast<uint32_t *>(d.qa + at) = hi;
        if (TWO) *reinterpret_cast<uint32_t *>(d.la + at) = lo;
    }
}

// One item per workgroup: in a loop over items the compiler spills the row.
template <bool TWO>
__global__ __launch_bounds__(256) void grouped_rows_kernel(const Fp8Member *__restrict__ g, int count, int64_t total) {
    __shared__ __attribute__((aligned(16))) float part[4][256];
    const int64_t item = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (item >= total) return;
    const int k = __builtin_amdgcn_readfirstlane(find_member<&Fp8Member::row_first>(g, count, item));
    const Fp8Member &d = g[k];
    const int64_t local = item - d.row_first;
    if (local < d.row_items) {
        const int64_t i = local * 4 + (threadIdx.x >> 6);
        if (i < padded_rows(d.m)) condition_any_row<TWO>(d, i, threadIdx.x & 63);
    } else {
        const int64_t b = local - d.row_items;
        col_amax_block(d.B, d.n, d.p, b % d.col_amax_x, b / d.col_amax_x, d.amaxB, part);
    }
}

template <bool TWO>
__global__ __launch_bounds__(256) void grouped_cols_kernel(const Fp8Member *__restrict__ g, int count, int64_t total) {
    __shared__ uint32_t tq[64 * TSTRIDE];
    __shared__ uint32_t tl[TWO ? 64 * TSTRIDE : 1];
    for (int64_t item = blockIdx.x; item < total; item += gridDim.x) {
        const int k = __builtin_amdgcn_readfirstlane(find_member<&Fp8Member::col_first>(g, count, item));
        const Fp8Member &d = g[k];
        const int64_t b = item - d.col_first;
        const int64_t bx = b % d.col_x, s = b / d.col_x;
        if (s == 0) write_col_exps(d.amaxB, d.p, bx, d.f);
        if (s < d.S) pack_cols_fp8_block<TWO>(d.B, d.n, d.p, d.S, d.amaxB, d.qb, d.lb, bx, s, tq, tl);
    }
}

struct Fp8Shape { int bm, bn, wm, wn, stages; };
constexpr Fp8Shape kOne[] = {{128, 128, 64, 64, 3}, {256, 256, 128, 64, 3}, {256, 256, 128, 64, 4},
                             {256, 256, 128, 64, 5}};
// Deeper rings pay off here: a slab carries 64 k, so a step is short next
// to the latency of its loads.
// The rectangular two-term blocks (8 waves of 64 x 64, 144 KB ring) read a
// third less LDS per matrix-core step than 128 x 128 with 64 x 32 waves.
// (8192 x 4096 x 8192: 714 us, 128 x 256, and 732, 256 x 128, against 840-858; four
// waves of 128 x 64, one per SIMD, were slower, 834 when eight took 777).
constexpr Fp8Shape kTwo[] = {{128, 128, 64, 64, 3}, {128, 128, 64, 32, 3}, {128, 128, 64, 32, 5},
                             {128, 128, 64, 32, 4}, {128, 256, 64, 64, 3}, {256, 128, 64, 64, 3}};
constexpr int kOneCount = sizeof(kOne) / sizeof(kOne[0]);
constexpr int kTwoCount = sizeof(kTwo) / sizeof(kTwo[0]);

template <int BM, int BN, int WM, int WN, bool TWO, int NST = ring::NSTAGE>
hipError_t launch_shape(const ring::Operands &op, hipStream_t st) {
    constexpr int NREC = TWO ? 2 : 1;
    const int tiles_m = (int)((op.m + BM - 1) / BM);
    const int tiles_n = (int)((op.p + BN - 1) / BN);
    hipLaunchKernelGGL((ring::single_kernel<BM, BN, WM, WN, NREC, Fp8Mode<TWO>, NST>), dim3(tiles_m * tiles_n),
                       dim3(ring::Cfg<BM, BN, WM, WN, NREC, NST>::THREADS), 0, st, op, tiles_m, tiles_n);
    return hipGetLastError();
}

template <bool TWO, int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, TWO ? 1 : 2) void fp8_grouped_kernel(
    const Fp8Member *__restrict__ g, int count, int64_t total_tiles, unsigned long long *__restrict__ counter) {
    constexpr int NREC = TWO ? 2 : 1;
    using G = ring::Cfg<BM, BN, WM, WN, NREC, NST>;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[G::LDS];
    // the claimed tile id lives in the ring's last slot, whose first load is
    // issued behind the tile's first barrier (in an array of its own it makes
    // the compiler wait for the loads in flight before every read of the ring)
    int64_t *s_tile = reinterpret_cast<int64_t *>(lds + (NST - 1) * G::STAGE);
    for (;;) {
        // the last tile's loads and stores of C are done (or the compiler waits
        // for them behind the next tile's first loads, and so for those too)
        __builtin_amdgcn_s_waitcnt(ring::waitcnt_vm(0));
        __syncthreads();                // nobody still reads the ring
        if (threadIdx.x == 0) *s_tile = (int64_t)atomicAdd(counter, 1ull);
        __syncthreads();
        const int64_t claimed = *s_tile;
        const int64_t tile = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)claimed) |
                                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(claimed >> 32)) << 32);
        if (tile >= total_tiles) break;
        const int k = __builtin_amdgcn_readfirstlane(find_member<&Fp8Member::first_tile>(g, count, tile));
        const Fp8Member &d = g[k];
        const int local = (int)(tile - d.first_tile);        // chunks x tiles: below 2^31
        const int chunk = local / d.tiles, at = local - chunk * d.tiles;
        const int tm = at / d.tiles_n, tn = at - tm * d.tiles_n;
        const int s_begin = __builtin_amdgcn_readfirstlane(chunk * d.chunk_slabs);
        const int s_end = __builtin_amdgcn_readfirstlane(min((int)d.S, s_begin + d.chunk_slabs));
        float *partial = d.chunks > 1 ? d.partials + (int64_t)__builtin_amdgcn_readfirstlane(chunk) * d.m * d.p : nullptr;
        ring::tile<BM, BN, WM, WN, NREC, Fp8Mode<TWO>, NST>(d.op, __builtin_amdgcn_readfirstlane(tm) * (int64_t)BM,
                                                            __builtin_amdgcn_readfirstlane(tn) * (int64_t)BN, lds,
                                                            s_begin, s_end, partial);
    }
}

// C of the members with a split k walk from their chunks' partials, in chunk
// order and descaled as ring::splitk_reduce_kernel does, 1024 elements per block.
constexpr int SUM_BLOCK = 1024;
__global__ __launch_bounds__(256) void fp8_sums_kernel(const Fp8Member *__restrict__ g, int count, int64_t total) {
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= total) return;
    // sum_first counts the blocks of the members before: the last member that
    // starts at or before this block owns it (an unsplit one takes no blocks)
    const int k = __builtin_amdgcn_readfirstlane(find_member<&Fp8Member::sum_first>(g, count, block));
    const Fp8Member &d = g[k];
    const int64_t mp = d.m * d.p, x0 = (block - d.sum_first) * SUM_BLOCK;
    if (d.p % 4 == 0 && (uintptr_t)d.op.C % 16 == 0) {
        const int64_t x = x0 + threadIdx.x * 4;
        if (x < mp) {
            const int64_t i = x / d.p;
            ring::splitk_sum<4>(d.partials, d.chunks, mp, x, d.op.C, d.e[i], d.f + (x - i * d.p), d.op.accumulate);
        }
    } else {
#pragma unroll
        for (int e = 0; e < SUM_BLOCK / 256; ++e) {
            const int64_t x = x0 + e * 256 + threadIdx.x;
            if (x >= mp) continue;
            const int64_t i = x / d.p;
            ring::splitk_sum<1>(d.partials, d.chunks, mp, x, d.op.C, d.e[i], d.f + (x - i * d.p), d.op.accumulate);
        }
    }
}

// Block shapes of the persistent launch: two terms 128 x 128 with 8 waves and
// a 4-deep ring (128 KiB LDS, one workgroup per CU); one term 128 x 128 with
// 4 waves and a 3-deep ring (48 KiB; its registers allow two per CU -- asking
// the compiler for three makes it spill).
constexpr int G_BM = 128, G_BN = 128;
constexpr int G_PER_CU_TWO = 1, G_PER_CU_ONE = 2;

int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }

struct Fp8Workspace {
    uint32_t *amaxA, *amaxB;
    int32_t *e, *f;
    uint8_t *qA, *lA, *qB, *lB;
};

Fp8Workspace carve(void *ws, int64_t m, int64_t n, int64_t p, bool two) {
    const int64_t S = (n + SLAB8 - 1) / SLAB8;
    char *c = static_cast<char *>(ws);
    Fp8Workspace w;
    w.amaxB = reinterpret_cast<uint32_t *>(c); c += align256(4 * p);
    w.amaxA = reinterpret_cast<uint32_t *>(c); c += align256(4 * m);
    w.e = reinterpret_cast<int32_t *>(c); c += align256(4 * m);
    w.f = reinterpret_cast<int32_t *>(c); c += align256(4 * p);
    w.qA = reinterpret_cast<uint8_t *>(c); c += align256(ring::array_bytes(m, S));
    w.qB = reinterpret_cast<uint8_t *>(c); c += align256(ring::array_bytes(p, S));
    w.lA = two ? reinterpret_cast<uint8_t *>(c) : nullptr; c += two ? align256(ring::array_bytes(m, S)) : 0;
    w.lB = two ? reinterpret_cast<uint8_t *>(c) : nullptr;
    return w;
}

// Amax of the columns of X (K x cols) into `amax`, which holds zeros.
void col_amax(const float *X, int64_t K, int64_t cols, uint32_t *amax, hipStream_t st) {
    if (K <= 0 || cols <= 0) return;
    const dim3 grid((unsigned)((cols + 255) / 256), (unsigned)std::min<int64_t>((K + COL_BAND - 1) / COL_BAND, 32768));
    hipLaunchKernelGGL(col_amax_kernel, grid, dim3(256), 0, st, X, K, cols, amax);
}

// Exponents of A's rows and amax of B's columns.
void scales(const float *A, int64_t m, int64_t n, const float *B, int64_t p, int32_t *e, uint32_t *amaxB,
            hipStream_t st) {
    if (p > 0) hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((p + 255) / 256)), dim3(256), 0, st, amaxB, p);
    if (m > 0)
        hipLaunchKernelGGL(row_exp_kernel, dim3((unsigned)std::min(m, ROW_BLOCKS)), dim3(256), 0, st, A, m, n, e);
    col_amax(B, n, p, amaxB, st);
}

RowsJob rows_job(const float *X, int64_t rows, int32_t *e, uint8_t *q, uint8_t *l) {
    return {X, rows, padded_rows(rows) / 4, e, q, l};
}

// Exponents and records of operands whose wanted vectors are the rows (of K
// values) of an array: A's rows, a column-major B's columns, or both in one
// launch. Clears `count` words at `clear` on the way. The smallest J that holds
// a row: registers (28, 42, 74 and 138) set the waves per SIMD. Beyond 8192
// values a row would take over 256 registers, one wave per SIMD: two passes
// there, a workgroup per row.
template <bool TWO>
void row_records(const RowsJob &a, const RowsJob &b, int64_t K, int64_t S, uint32_t *clear, int64_t count,
                 hipStream_t st) {
    const dim3 grid = item_grid(a.blocks + b.blocks), bl(256);
    if (K <= 1024) {
        hipLaunchKernelGGL((rows_fp8_kernel<TWO, 4>), grid, bl, 0, st, a, b, K, S, clear, count);
    } else if (K <= 2048) {
        hipLaunchKernelGGL((rows_fp8_kernel<TWO, 8>), grid, bl, 0, st, a, b, K, S, clear, count);
    } else if (K <= 4096) {
        hipLaunchKernelGGL((rows_fp8_kernel<TWO, 16>), grid, bl, 0, st, a, b, K, S, clear, count);
    } else if (K <= 8192) {
        hipLaunchKernelGGL((rows_fp8_kernel<TWO, 32>), grid, bl, 0, st, a, b, K, S, clear, count);
    } else {
        if (count > 0)
            hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((count + 255) / 256)), bl, 0, st, clear, count);
        for (const RowsJob *d : {&a, &b}) {
            if (d->blocks == 0) continue;
            hipLaunchKernelGGL(row_exp_kernel, dim3((unsigned)std::min(d->rows, ROW_BLOCKS)), bl, 0, st, d->X, d->rows, K,
                               d->e);
            const int64_t blocks = std::min<int64_t>((padded_rows(d->rows) * S * 4 + 255) / 256, 65536);
            hipLaunchKernelGGL(pack_rows_fp8_kernel<TWO>, dim3((unsigned)blocks), bl, 0, st, d->X, d->rows, K, S, d->e,
                               d->q, d->l);
        }
    }
}

// The same where they are the columns of X (K x cols); `amax` holds zeros.
template <bool TWO>
void col_records(const float *X, int64_t cols, int64_t K, int64_t S, uint32_t *amax, int32_t *exps, uint8_t *q,
                 uint8_t *l, hipStream_t st) {
    col_amax(X, K, cols, amax, st);
    // also when S == 0: the epilogue reads the exponents
    const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)(S < 1 ? 1 : S > 65535 ? 65535 : S));
    hipLaunchKernelGGL(pack_cols_fp8_kernel<TWO>, grid, dim3(256), 0, st, X, K, cols, S, amax, exps, q, l);
}

// A column-major A (element (i, k) at i + k m) is a row-major n x m array
// whose columns are A's rows; a column-major B is a row-major p x n array
// whose rows are B's columns. An operand taken by rows goes first and clears
// the other's column amax; two taken by columns share one clear (their amax
// arrays are neighbours in the workspace).
template <bool TWO>
hipError_t pack_records(const moa_gemm_desc &d, const Fp8Workspace &w, hipStream_t st) {
    const float *A = static_cast<const float *>(d.A);
    const float *B = static_cast<const float *>(d.B);
    const int64_t S = (d.n + SLAB8 - 1) / SLAB8;
    const bool a_rows = !(d.flags & MOA_FLAG_A_COL), b_rows = (d.flags & MOA_FLAG_B_COL) != 0;
    if (!a_rows && !b_rows) {
        const int64_t words = align256(4 * d.p) / 4 + d.m;
        hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, w.amaxB, words);
    }
    const RowsJob a = rows_job(A, d.m, w.e, w.qA, w.lA), b = rows_job(B, d.p, w.f, w.qB, w.lB), none{};
    if (a_rows && b_rows) row_records<TWO>(a, b, d.n, S, nullptr, 0, st);
    else if (a_rows) row_records<TWO>(a, none, d.n, S, w.amaxB, d.p, st);
    else if (b_rows) row_records<TWO>(b, none, d.n, S, w.amaxA, d.m, st);
    if (!a_rows) col_records<TWO>(A, d.m, d.n, S, w.amaxA, w.e, w.qA, w.lA, st);
    if (!b_rows) col_records<TWO>(B, d.p, d.n, S, w.amaxB, w.f, w.qB, w.lB, st);
    return hipGetLastError();
}

}  // namespace

int fp8_variant_count(bool two) { return two ? kTwoCount : kOneCount; }

void fp8_shape(bool two, int v, Plan *p) {
    const Fp8Shape s = two ? kTwo[v] : kOne[v];
    p->variant = v;
    p->tile_m = s.bm;
    p->tile_n = s.bn;
    p->tile_k = SLAB8;
    p->wave_m = s.wm;
    p->wave_n = s.wn;
    p->lane_m = p->lane_n = 0;
    p->threads = (s.bm / s.wm) * (s.bn / s.wn) * 64;
    p->lds_bytes = s.stages * (two ? 2 : 1) * (s.bm + s.bn) * REC_BYTES;
}

int64_t fp8_workspace_bytes(int64_t m, int64_t n, int64_t p, bool two) {
    const int64_t S = (n + SLAB8 - 1) / SLAB8;
    const int64_t rec = align256(ring::array_bytes(m, S)) + align256(ring::array_bytes(p, S));
    return align256(4 * p) * 2 + align256(4 * m) * 2 + (two ? 2 : 1) * rec;
}

hipError_t launch_fp8(const moa_gemm_desc &d, const Plan &plan, void *ws, hipStream_t st) {
    const bool two = fp8_two_term(d);
    const Fp8Workspace w = carve(ws, d.m, d.n, d.p, two);
    hipError_t err;
    {
        TraceScope ts(MOA_K_FP8_QUANT, st);
        err = two ? pack_records<true>(d, w, st) : pack_records<false>(d, w, st);
    }
    if (err != hipSuccess) return err;
    TraceScope ts(two ? MOA_K_FP8_2TERM : MOA_K_FP8, st);
    ring::Operands op;
    op.a0 = w.qA; op.a1 = w.lA;
    op.b0 = w.qB; op.b1 = w.lB;
    op.C = static_cast<float *>(d.C);
    op.row_exp = w.e;
    op.col_exp = w.f;
    op.m = d.m; op.p = d.p;
    op.S = (d.n + SLAB8 - 1) / SLAB8;
    op.accumulate = d.accumulate;
    if (plan.split_k > 1) {
        float *partials = reinterpret_cast<float *>(static_cast<char *>(ws) + plan.partial_offset);
        if (two) return ring::launch_splitk<128, 128, 64, 64, 2, Fp8Mode<true>, 3>(op, plan.split_k, partials, st);
        return ring::launch_splitk<128, 128, 64, 64, 1, Fp8Mode<false>, 3>(op, plan.split_k, partials, st);
    }
    if (two) {
        switch (plan.variant) {
        case 0: return launch_shape<128, 128, 64, 64, true>(op, st);
        case 1: return launch_shape<128, 128, 64, 32, true>(op, st);
        case 2: return launch_shape<128, 128, 64, 32, true, 5>(op, st);
        case 4: return launch_shape<128, 256, 64, 64, true, 3>(op, st);
        case 5: return launch_shape<256, 128, 64, 64, true, 3>(op, st);
        default: return launch_shape<128, 128, 64, 32, true, 4>(op, st);
        }
    }
    switch (plan.variant) {
    case 0: return launch_shape<128, 128, 64, 64, false>(op, st);
    case 1: return launch_shape<256, 256, 128, 64, false>(op, st);
    case 2: return launch_shape<256, 256, 128, 64, false, 4>(op, st);
    default: return launch_shape<256, 256, 128, 64, false, 5>(op, st);
    }
}

int64_t fp8_grouped_desc_bytes(int count) { return (int64_t)count * (int64_t)sizeof(Fp8Member); }

namespace {
int64_t partial_bytes(const Fp8Product &x) {
    return x.split_k > 1 ? align256((int64_t)x.split_k * x.d->m * x.d->p * 4) : 0;
}
int64_t header_bytes(const Fp8Product *members, int count) {
    int64_t cols = 0;
    for (int k = 0; k < count; ++k) cols += members[k].d->p;
    return align256(8 + 4 * cols);     // claim counter, then every member's column amax
}
}  // namespace

int64_t fp8_member_bytes(const Fp8Product &x, bool two) {
    const moa_gemm_desc &d = *x.d;
    const int64_t S = (d.n + SLAB8 - 1) / SLAB8;
    const int64_t rec = align256(ring::array_bytes(d.m, S)) + align256(ring::array_bytes(d.p, S));
    return align256(4 * d.m) + align256(4 * d.p) + (two ? 2 : 1) * rec + partial_bytes(x);
}

int64_t fp8_grouped_workspace_bytes(const Fp8Product *members, int count, bool two) {
    int64_t b = header_bytes(members, count) + align256(fp8_grouped_desc_bytes(count));
    for (int k = 0; k < count; ++k) b += fp8_member_bytes(members[k], two);
    return b;
}

// Workspace: [counter u64 | amax of every member][member table][per member:
// e, f, record arrays, partials]. Members are listed longest k walk (of a
// chunk) first.
Fp8GroupWork fp8_grouped_layout(const Fp8Product *members, int count, bool two, void *ws,
                                void *host_staging) {
    std::vector<int> order(count);
    for (int k = 0; k < count; ++k) order[k] = k;
    auto walk = [&](int k) { return members[k].d->n / std::max(members[k].split_k, 1); };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return walk(a) > walk(b); });
    char *base = static_cast<char *>(ws);
    uint32_t *amax = reinterpret_cast<uint32_t *>(base + 8);
    char *cur = base + header_bytes(members, count) + align256(fp8_grouped_desc_bytes(count));
    Fp8Member *h = static_cast<Fp8Member *>(host_staging);
    Fp8GroupWork w{0, 0, 0, 0, 2, header_bytes(members, count)};
    for (int q = 0; q < count; ++q) {
        const Fp8Product &x = members[order[q]];
        const moa_gemm_desc &d = *x.d;
        Fp8Member g;
        g.A = static_cast<const float *>(d.A);
        g.B = static_cast<const float *>(d.B);
        g.m = d.m; g.n = d.n; g.p = d.p;
        g.S = (d.n + SLAB8 - 1) / SLAB8;
        g.amaxB = amax;
        amax += d.p;
        w.clear_words += d.p;
        g.e = reinterpret_cast<int32_t *>(cur); cur += align256(4 * d.m);
        g.f = reinterpret_cast<int32_t *>(cur); cur += align256(4 * d.p);
        g.qa = reinterpret_cast<uint8_t *>(cur); cur += align256(ring::array_bytes(d.m, g.S));
        g.qb = reinterpret_cast<uint8_t *>(cur); cur += align256(ring::array_bytes(d.p, g.S));
        g.la = g.lb = nullptr;
        if (two) {
            g.la = reinterpret_cast<uint8_t *>(cur); cur += align256(ring::array_bytes(d.m, g.S));
            g.lb = reinterpret_cast<uint8_t *>(cur); cur += align256(ring::array_bytes(d.p, g.S));
        }
        g.op.a0 = g.qa; g.op.a1 = g.la;
        g.op.b0 = g.qb; g.op.b1 = g.lb;
        g.op.C = static_cast<float *>(d.C);
        g.op.row_exp = g.e;
        g.op.col_exp = g.f;
        g.op.m = d.m; g.op.p = d.p; g.op.S = g.S;
        g.op.accumulate = d.accumulate;
        g.tiles_n = (int32_t)((d.p + G_BN - 1) / G_BN);
        g.tiles = (int32_t)((d.m + G_BM - 1) / G_BM) * g.tiles_n;
        g.chunks = 1;
        g.chunk_slabs = (int32_t)g.S;
        g.partials = nullptr;
        g.sum_first = w.sum_items;
        if (x.split_k > 1 && g.S > 1) {                    // as ring::launch_splitk cuts them
            g.chunk_slabs = (int32_t)((g.S + x.split_k - 1) / x.split_k);
            g.chunks = (int32_t)((g.S + g.chunk_slabs - 1) / g.chunk_slabs);
        }
        if (g.chunks > 1) {
            g.partials = reinterpret_cast<float *>(cur);
            cur += partial_bytes(x);
            w.sum_items += (d.m * d.p + SUM_BLOCK - 1) / SUM_BLOCK;
        }
        g.first_tile = w.tiles;
        w.tiles += (int64_t)g.chunks * g.tiles;
        g.row_items = (int32_t)(padded_rows(d.m) / 4);
        g.col_amax_x = (int32_t)((d.p + 255) / 256);
        g.row_first = w.row_items;
        w.row_items += g.row_items + (int64_t)g.col_amax_x * ((d.n + COL_BAND - 1) / COL_BAND);
        g.col_x = (int32_t)((d.p + 63) / 64);
        g.col_first = w.col_items;
        w.col_items += (int64_t)g.col_x * (g.S > 0 ? g.S : 1);
        h[q] = g;
    }
    return w;
}

hipError_t fp8_grouped_enqueue(void *ws, int count, bool two, const Fp8GroupWork &w, bool cleared, hipStream_t st) {
    char *base = static_cast<char *>(ws);
    unsigned long long *counter = reinterpret_cast<unsigned long long *>(base);
    const Fp8Member *dev = reinterpret_cast<const Fp8Member *>(base + w.table_offset);
    {
        TraceScope ts(MOA_K_FP8_QUANT, st);
        if (!cleared)
            hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((w.clear_words + 255) / 256)), dim3(256), 0, st,
                               reinterpret_cast<uint32_t *>(base), w.clear_words);
        if (w.row_items > 0) {
            const dim3 grid = item_grid(w.row_items);
            if (two) hipLaunchKernelGGL(grouped_rows_kernel<true>, grid, dim3(256), 0, st, dev, count, w.row_items);
            else hipLaunchKernelGGL(grouped_rows_kernel<false>, grid, dim3(256), 0, st, dev, count, w.row_items);
        }
        if (w.col_items > 0) {
            const dim3 grid((unsigned)std::min<int64_t>(w.col_items, 8 * kNumCUs));
            if (two) hipLaunchKernelGGL(grouped_cols_kernel<true>, grid, dim3(256), 0, st, dev, count, w.col_items);
            else hipLaunchKernelGGL(grouped_cols_kernel<false>, grid, dim3(256), 0, st, dev, count, w.col_items);
        }
    }
    TraceScope ts(MOA_K_FP8_GROUPED, st);
    if (w.tiles > 0) {
        if (two) {
            constexpr int WM = 64, WN = 32, NST = 4;
            hipLaunchKernelGGL((fp8_grouped_kernel<true, G_BM, G_BN, WM, WN, NST>),
                               dim3((unsigned)std::min<int64_t>(w.tiles, G_PER_CU_TWO * kNumCUs)),
                               dim3(ring::Cfg<G_BM, G_BN, WM, WN, 2, NST>::THREADS), 0, st, dev, count, w.tiles,
                               counter);
        } else {
            constexpr int WM = 64, WN = 64, NST = 3;
            hipLaunchKernelGGL((fp8_grouped_kernel<false, G_BM, G_BN, WM, WN, NST>),
                               dim3((unsigned)std::min<int64_t>(w.tiles, G_PER_CU_ONE * kNumCUs)),
                               dim3(ring::Cfg<G_BM, G_BN, WM, WN, 1, NST>::THREADS), 0, st, dev, count, w.tiles,
                               counter);
        }
    }
    if (w.sum_items > 0)
        hipLaunchKernelGGL(fp8_sums_kernel, item_grid(w.sum_items), dim3(256), 0, st, dev, count, w.sum_items);
    return hipGetLastError();
}

namespace {
// The member table straight from pinned host memory mapped into the device's
// address space (n16 16-byte words), and the clear of the claim counter and the
// column amax: one kernel in place of a copy-engine transfer and its hand-offs
// to and from the compute queue.
__global__ __launch_bounds__(256) void table_from_host_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                              int64_t n16, uint32_t *__restrict__ clear,
                                                              int64_t words) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += stride) clear[i] = 0u;
}
}  // namespace

hipError_t launch_fp8_grouped(const Fp8Product *members, int count, bool two, void *ws,
                              void *host_staging, const void *host_staging_dev, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const Fp8GroupWork w = fp8_grouped_layout(members, count, two, ws, host_staging);
    char *table = static_cast<char *>(ws) + w.table_offset;
    const int64_t bytes = fp8_grouped_desc_bytes(count);
    if (host_staging_dev) {
        const int64_t n16 = (bytes + 15) / 16;
        const int64_t blocks = std::min<int64_t>((std::max(n16, w.clear_words) + 255) / 256, 64);
        hipLaunchKernelGGL(table_from_host_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                           static_cast<const uint4 *>(host_staging_dev), reinterpret_cast<uint4 *>(table), n16,
                           static_cast<uint32_t *>(ws), w.clear_words);
        return fp8_grouped_enqueue(ws, count, two, w, true, st);
    }
    hipError_t e = hipMemcpyAsync(table, host_staging, (size_t)bytes, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return e;
    return fp8_grouped_enqueue(ws, count, two, w, false, st);
}

hipError_t launch_quantise_fp8(const float *A, int64_t m, int64_t n, const float *B, int64_t p,
                               bool two, int32_t *e, uint8_t *qA, uint8_t *lA, int32_t *f,
                               uint8_t *qB, uint8_t *lB, uint32_t *amax, hipStream_t st) {
    uint32_t *amaxB = amax + m;
    scales(A, m, n, B, p, e, amaxB, st);
    if (m > 0 && n > 0)
        hipLaunchKernelGGL(quant_rows_kernel, dim3((unsigned)m, (unsigned)((n + 1023) / 1024)), dim3(256), 0, st, A,
                           m, n, e, (int)two, qA, lA);
    if (p > 0)
        hipLaunchKernelGGL(quant_cols_kernel, dim3((unsigned)((p + 63) / 64), (unsigned)((n + 63) / 64 > 0 ? (n + 63) / 64 : 1)),
                           dim3(256), 0, st, B, n, p, amaxB, (int)two, f, qB, lB);
    return hipGetLastError();
}

}  // namespace moa
