// The ipophp family (conclusion and appendix: one formulation for the
// Hadamard product, the Kronecker product and the matrix product; higher
// dimensional contractions as many parallel 2-d products).
//
//   Hadamard:  C[i,j] := A[i,j] B[i,j]                          (m x n)
//   Kronecker: C[i p + k, j q + l] := A[i,j] B[k,l]             A m x n, B p x q
//   batched:   C[b] := A[b] B[b]                                (grouped launch)
//
// Every element of the first two is one product (plus, in the accumulate
// form, one addition to C), each rounded to the element type: floating-point
// contraction is off in these kernels, so results are bitwise those of the
// definition. Both are bound by HBM traffic: the Kronecker kernel writes C
// row by row (row i p + k of C is A[i, :] (x) B[k, :]), A and B stay in cache.
#include <algorithm>
#include <vector>

#include "moa_internal.h"

namespace moa {
namespace {

template <typename T> struct Vec16;
template <> struct Vec16<float> { using type = float4; static constexpr int N = 4; };
template <> struct Vec16<double> { using type = double2; static constexpr int N = 2; };

template <typename T>
__device__ __forceinline__ T product(T a, T b, const T *c, int accumulate) {
#pragma clang fp contract(off)
    T v = a * b;
    if (accumulate) v = v + *c;
    return v;
}

template <typename T>
__global__ __launch_bounds__(256) void hadamard_kernel(const T *A, const T *B, T *C, int64_t count, int vec,
                                                       int accumulate) {   // C may be A or B (in place)
    using V = typename Vec16<T>::type;
    constexpr int N = Vec16<T>::N;
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t nvec = vec ? count / N : 0;
    for (int64_t t = t0; t < nvec; t += stride) {
        const V a = reinterpret_cast<const V *>(A)[t];
        const V b = reinterpret_cast<const V *>(B)[t];
        V c = accumulate ? reinterpret_cast<V *>(C)[t] : V{};   // C is read only when accumulating
        const T *pa = reinterpret_cast<const T *>(&a);
        const T *pb = reinterpret_cast<const T *>(&b);
        T *pc = reinterpret_cast<T *>(&c);
#pragma unroll
        for (int e = 0; e < N; ++e) pc[e] = product(pa[e], pb[e], pc + e, accumulate);
        reinterpret_cast<V *>(C)[t] = c;
    }
    for (int64_t x = nvec * N + t0; x < count; x += stride) C[x] = product(A[x], B[x], C + x, accumulate);
}

// A workgroup writes 256 N columns of `run` consecutive rows of C; row i p + k
// is A[i, :] (x) B[k, :]. A thread's N columns keep their (j, l) = (c / q, c mod
// q), found once in 32-bit arithmetic (the entry point keeps n q below 2^31),
// and its N values of A stay in registers until i changes; (i, k) advance by
// counting, one 64-bit division per workgroup. What is left per row is reading
// B and the store, so the kernel is bound by writing C. Wide: q and C in whole
// 16-byte vectors and B aligned, so a thread's columns share j, run along l and
// move as one vector; Scalar: its columns are 256 apart, so that the lanes of each
// 4- or 8-byte access are consecutive; Gather: rows of C in whole vectors,
// written so from values of B read one by one. 64^2 (x) 128^2 in FP32 (8192^2):
// 95 us with a 64-bit division and eight scalar reads per row and 16 bytes, 46-48
// us (5.7 TB/s written; a plain fill of that size reaches 6.9) this way.
enum class Row { Scalar, Gather, Wide };
template <typename T, Row R>
__global__ __launch_bounds__(256) void kronecker_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                        T *__restrict__ C, int64_t m, int64_t n, int64_t p,
                                                        int64_t q, int64_t run, int accumulate) {
    using V = typename Vec16<T>::type;
    constexpr int N = Vec16<T>::N;
    constexpr bool VEC = R != Row::Scalar;
    const int64_t rows = m * p;
    const int cols = (int)(n * q), qq = (int)q;
    const int64_t r0 = (int64_t)blockIdx.y * run, r1 = min(r0 + run, rows);
    const int64_t i0 = r0 / p;
    for (int64_t base = (int64_t)blockIdx.x * 256 * N; base < cols; base += (int64_t)gridDim.x * 256 * N) {
        int64_t c[N];
        int jj[N], ll[N];
        bool live[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
            c[e] = VEC ? base + (int64_t)threadIdx.x * N + e : base + e * 256 + threadIdx.x;
            live[e] = c[e] < cols;
            const int cc = live[e] ? (int)c[e] : 0;
            jj[e] = cc / qq;
            ll[e] = cc - jj[e] * qq;
        }
        int64_t i = i0, k = r0 - i0 * p;
        T a[N];
        auto row_of_a = [&] {
#pragma unroll
            for (int e = 0; e < N; ++e) a[e] = A[i * n + jj[e]];
        };
        if (!live[0]) continue;          // the whole vector, or every later column too
        row_of_a();
#pragma unroll 4
        for (int64_t r = r0; r < r1; ++r) {
            T *crow = C + r * (int64_t)cols;
            const T *brow = B + k * q;
            if constexpr (VEC) {
                V bv;
                T *pb = reinterpret_cast<T *>(&bv);
                if constexpr (R == Row::Wide) {
                    bv = *reinterpret_cast<const V *>(brow + ll[0]);
                } else {
#pragma unroll
                    for (int e = 0; e < N; ++e) pb[e] = brow[ll[e]];
                }
                V out = accumulate ? *reinterpret_cast<const V *>(crow + c[0]) : V{};
                T *po = reinterpret_cast<T *>(&out);
#pragma unroll
                for (int e = 0; e < N; ++e) po[e] = product(a[e], pb[e], po + e, accumulate);
                *reinterpret_cast<V *>(crow + c[0]) = out;
            } else {
#pragma unroll
                for (int e = 0; e < N; ++e)
                    if (live[e]) crow[c[e]] = product(a[e], brow[ll[e]], crow + c[e], accumulate);
            }
            if (++k == p) {
                k = 0;
                if (++i < m) row_of_a();
            }
        }
    }
}

}  // namespace

hipError_t launch_hadamard(int64_t count, moa_dtype dt, const void *A, const void *B, void *C, int accumulate,
                           hipStream_t st) {
    int64_t blocks = (count + 1023) / 1024;
    blocks = std::max<int64_t>(1, std::min<int64_t>(blocks, 8 * kNumCUs));
    const bool aligned = ((uintptr_t)A % 16 == 0) && ((uintptr_t)B % 16 == 0) && ((uintptr_t)C % 16 == 0);
    TraceScope ts(MOA_K_HADAMARD, st);
    if (dt == MOA_F64)
        hipLaunchKernelGGL(hadamard_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, st,
                           static_cast<const double *>(A), static_cast<const double *>(B), static_cast<double *>(C),
                           count, (int)aligned, accumulate);
    else
        hipLaunchKernelGGL(hadamard_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st,
                           static_cast<const float *>(A), static_cast<const float *>(B), static_cast<float *>(C),
                           count, (int)aligned, accumulate);
    return hipGetLastError();
}

hipError_t launch_kronecker(int64_t m, int64_t n, int64_t p, int64_t q, moa_dtype dt, const void *A, const void *B,
                            void *C, int accumulate, hipStream_t st) {
    const int64_t cols = n * q, rows = m * p;
    const int N = dt == MOA_F64 ? 2 : 4;
    const bool wide = q % N == 0 && (uintptr_t)C % 16 == 0 && (uintptr_t)B % 16 == 0;
    // Gather for rows of one or two chunks, where columns 256 apart leave most of
    // the last chunk empty (kernel alone, FP32: 64 x 64 (x) 100 x 17 13 us against
    // 14.7, but 64 x 64 (x) 127 x 127 73 against 51)
    const bool gather = cols < 2048 && cols % N == 0 && (uintptr_t)C % 16 == 0;
    // All column chunks of a row; rows in runs for about 16384 workgroups (8192^2
    // FP32: 46 us, 52 with 4096, of fewer and longer runs). Small products: single
    // rows up to 1024 workgroups, then runs of up to four rows, more where a chunk
    // has less than 2 KiB (20 x 10 (x) 20 x 16, 400 rows: 2.9 us in single rows, 3.4
    // in runs of four; 50 x 8 (x) 80 x 20, 4000 rows: 7.3 and 4.4)
    const int64_t gx = std::min<int64_t>((cols + 256 * N - 1) / (256 * N), 64);
    const int64_t chunk_bytes = std::min<int64_t>(cols, 256 * N) * (16 / N);
    const int64_t few = std::min<int64_t>(std::max<int64_t>(4, 8192 / chunk_bytes), rows * gx / 1024);
    const int64_t run = std::max<int64_t>({1, few, rows * gx / 16384, (rows + 65534) / 65535});
    const dim3 grid((unsigned)gx, (unsigned)((rows + run - 1) / run));
    TraceScope ts(MOA_K_KRONECKER, st);
#define MOA_KRONECKER(T, R)                                                                                        \
    hipLaunchKernelGGL((kronecker_kernel<T, R>), grid, dim3(256), 0, st, static_cast<const T *>(A),                \
                       static_cast<const T *>(B), static_cast<T *>(C), m, n, p, q, run, accumulate)
    if (dt == MOA_F64) {
        if (wide) MOA_KRONECKER(double, Row::Wide);
        else if (gather) MOA_KRONECKER(double, Row::Gather);
        else MOA_KRONECKER(double, Row::Scalar);
    } else {
        if (wide) MOA_KRONECKER(float, Row::Wide);
        else if (gather) MOA_KRONECKER(float, Row::Gather);
        else MOA_KRONECKER(float, Row::Scalar);
    }
#undef MOA_KRONECKER
    return hipGetLastError();
}

}  // namespace moa

using namespace moa;

namespace {
bool spans_overlap(const void *x, int64_t xb, const void *y, int64_t yb) {
    if (xb == 0 || yb == 0) return false;
    const uintptr_t x0 = (uintptr_t)x, y0 = (uintptr_t)y;
    return x0 < y0 + (uintptr_t)yb && y0 < x0 + (uintptr_t)xb;
}
}  // namespace

extern "C" {

moa_status moa_hadamard(int64_t m, int64_t n, int32_t dtype, const void *A, const void *B, void *C,
                        int32_t accumulate, void *stream) {
    try {
        if (m < 0 || n < 0) return fail(MOA_ERR_SHAPE, "negative shape");
        if (dtype != MOA_F64 && dtype != MOA_F32) return fail(MOA_ERR_INVALID, "unknown dtype %d", dtype);
        const int64_t es = dtype == MOA_F64 ? 8 : 4;
        int64_t count = 0;
        if (__builtin_mul_overflow(m, n, &count) || count > INT64_MAX / es) return fail(MOA_ERR_SHAPE, "size overflow");
        if (count == 0) return MOA_OK;
        if (!A || !B || !C) return fail(MOA_ERR_INVALID, "null pointer");
        if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % (uintptr_t)es)
            return fail(MOA_ERR_INVALID, "pointers must be aligned to the element size");
        // C may be A or B exactly (elementwise), but not a shifted overlap
        if ((C != A && spans_overlap(C, count * es, A, count * es)) ||
            (C != B && spans_overlap(C, count * es, B, count * es)))
            return fail(MOA_ERR_INVALID, "C partially overlaps A or B");
        const hipError_t e = launch_hadamard(count, (moa_dtype)dtype, A, B, C, accumulate != 0,
                                             static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return hip_fail(e, "hadamard launch");
        return MOA_OK;
    } catch (...) {
        return fail(MOA_ERR_DEVICE, "internal error");
    }
}

moa_status moa_kronecker(int64_t m, int64_t n, int64_t p, int64_t q, int32_t dtype, const void *A, const void *B,
                         void *C, int32_t accumulate, void *stream) {
    try {
        if (m < 0 || n < 0 || p < 0 || q < 0) return fail(MOA_ERR_SHAPE, "negative shape");
        if (dtype != MOA_F64 && dtype != MOA_F32) return fail(MOA_ERR_INVALID, "unknown dtype %d", dtype);
        const int64_t es = dtype == MOA_F64 ? 8 : 4;
        int64_t rows, cols, count, na, nb;
        if (__builtin_mul_overflow(m, p, &rows) || __builtin_mul_overflow(n, q, &cols) ||
            __builtin_mul_overflow(rows, cols, &count) || count > INT64_MAX / es ||
            __builtin_mul_overflow(m, n, &na) || __builtin_mul_overflow(p, q, &nb))
            return fail(MOA_ERR_SHAPE, "size overflow");
        if (cols > INT32_MAX) return fail(MOA_ERR_SHAPE, "n q = %lld exceeds 2^31 - 1", (long long)cols);
        if (count == 0) return MOA_OK;
        if (!A || !B || !C) return fail(MOA_ERR_INVALID, "null pointer");
        if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % (uintptr_t)es)
            return fail(MOA_ERR_INVALID, "pointers must be aligned to the element size");
        if (spans_overlap(C, count * es, A, na * es) || spans_overlap(C, count * es, B, nb * es))
            return fail(MOA_ERR_INVALID, "C overlaps A or B");
        const hipError_t e = launch_kronecker(m, n, p, q, (moa_dtype)dtype, A, B, C, accumulate != 0,
                                              static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return hip_fail(e, "kronecker launch");
        return MOA_OK;
    } catch (...) {
        return fail(MOA_ERR_DEVICE, "internal error");
    }
}

moa_status moa_gemm_batched(const moa_gemm_desc *first, int64_t batch, int64_t stride_a, int64_t stride_b,
                            int64_t stride_c, void *stream) {
    try {
        if (!first) return fail(MOA_ERR_INVALID, "null descriptor");
        if (batch < 0 || stride_a < 0 || stride_b < 0 || stride_c < 0)
            return fail(MOA_ERR_INVALID, "negative batch or stride");
        if (batch == 0) return MOA_OK;
        const int64_t es = first->dtype == MOA_F64 ? 8 : 4;
        std::vector<moa_gemm_desc> descs((size_t)batch, *first);
        for (int64_t b = 0; b < batch; ++b) {
            int64_t oa, ob, oc;
            if (__builtin_mul_overflow(b, stride_a * es, &oa) || __builtin_mul_overflow(b, stride_b * es, &ob) ||
                __builtin_mul_overflow(b, stride_c * es, &oc))
                return fail(MOA_ERR_SHAPE, "batch offset overflow");
            if (first->A) descs[b].A = static_cast<const char *>(first->A) + oa;
            if (first->B) descs[b].B = static_cast<const char *>(first->B) + ob;
            if (first->C) descs[b].C = static_cast<char *>(first->C) + oc;
        }
        return moa_gemm_grouped(descs.data(), batch, stream);
    } catch (...) {
        return fail(MOA_ERR_DEVICE, "internal error");
    }
}

}  // extern "C"
