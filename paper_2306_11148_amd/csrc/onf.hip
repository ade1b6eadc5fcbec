// Plain ONF kernels: Eq. 3 with one fused multiply-add per (i, j, k), k in
// ascending order for every element of C.
//
// The paper's generic program walks row i of C and, for each k, adds the
// scalar A[i,k] times the contiguous row k of B (Fig. 1, section "From Normal
// Form to C Program"). Its dimension lifting (section "Dimension Lifting to
// Machine Coordinates") splits i over processors and j over register groups,
// and the k (sigma) loop into blocks. Two kernels carry out the splits, with
// the same bits:
//  * onf_mm_kernel (below, the one that runs): the matrix-core steps whose
//    element results are fma chains over ascending k;
//  * onf_kernel: scalar fma, register-staged slabs and 64-bit addresses, for
//    products whose rows exceed the matrix-core kernel's 32-bit offsets:
//   i -> (workgroup row block of TM rows, lane row group; R rows per lane,
//         strided by the TR row groups of the workgroup)
//   j -> (workgroup column block of TN columns, lane column group; VJ columns
//         per lane in VJ/VW runs of VW contiguous elements = one 16-byte
//         vector each)
//   k -> (LDS slab of BK, in-slab index)
//    Rows of A and B enter LDS as contiguous 16-byte vectors, double-buffered
//    through registers; a column-major operand (the paper's gamma_col layout)
//    is read along its contiguous extent and transposed on the way into the
//    same row-major slab. Each lane keeps its R x VJ block of C in registers
//    for the whole k loop.
#include "moa_internal.h"
#include "ring_gemm.h"

namespace moa {
namespace {

template <typename T> struct Vec;
template <> struct Vec<float> { using type = float4; static constexpr int W = 4; };
template <> struct Vec<double> { using type = double2; static constexpr int W = 2; };

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename T, int TM, int TN, int BK, int R, int VJ>
__global__ __launch_bounds__(256) void onf_kernel(const T *__restrict__ A,
                                                  const T *__restrict__ B,
                                                  T *__restrict__ C, int64_t m,
                                                  int64_t n, int64_t p,
                                                  int accumulate, int vec_a,
                                                  int vec_b, int vec_c, int a_col,
                                                  int b_col) {
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::W;          // elements per 16-byte vector
    constexpr int TC = TN / VJ;            // lane column groups
    constexpr int TR = TM / R;             // lane row groups
    static_assert(TC * TR == 256, "256 threads");
    static_assert(VJ % VW == 0 && BK % VW == 0, "vector multiples");
    constexpr int G = VJ / VW;             // column runs per lane
    constexpr int PAD_A = VW;              // keeps rows 16-byte aligned, skews banks
    constexpr int LDA = BK + PAD_A;
    constexpr int A_VECS = TM * BK / VW;   // vectors per A slab
    constexpr int B_VECS = BK * TN / VW;
    constexpr int A_PER = (A_VECS + 255) / 256;
    constexpr int B_PER = (B_VECS + 255) / 256;

    __shared__ __attribute__((aligned(16))) T As[2][TM * LDA];
    __shared__ __attribute__((aligned(16))) T Bs[2][BK * TN];

    const int t = threadIdx.x;
    const int tr = t / TC;                 // row group
    const int tc = t % TC;                 // column group
    const int64_t i0 = (int64_t)blockIdx.y * TM;
    const int64_t j0 = (int64_t)blockIdx.x * TN;

    // ---- C block in registers; the accumulate form starts from C --------
    T acc[R][VJ];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int v = 0; v < VJ; ++v) acc[q][v] = T(0);
    if (accumulate) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int64_t i = i0 + tr + (int64_t)TR * q;
            if (i >= m) continue;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < VW; ++e) {
                    const int64_t j = j0 + g * (TC * VW) + tc * VW + e;
                    if (j < p) acc[q][g * VW + e] = C[i * p + j];
                }
        }
    }

    // ---- global -> registers for one k slab ------------------------------
    V ra[A_PER], rb[B_PER];
    // whole blocks (inside m and p, the slab inside n, vector-aligned rows)
    // load without per-vector checks
    const bool inner = i0 + TM <= m && j0 + TN <= p && vec_a && vec_b && !a_col && !b_col;
    auto load_slab = [&](int64_t k0) {
        if (inner && k0 + BK <= n) {
#pragma unroll
            for (int s = 0; s < A_PER; ++s) {
                const int v = t + 256 * s;
                if (A_VECS % 256 == 0 || v < A_VECS)
                    ra[s] = *reinterpret_cast<const V *>(A + (i0 + v / (BK / VW)) * n + k0 + (v % (BK / VW)) * VW);
            }
#pragma unroll
            for (int s = 0; s < B_PER; ++s) {
                const int v = t + 256 * s;
                if (B_VECS % 256 == 0 || v < B_VECS)
                    rb[s] = *reinterpret_cast<const V *>(B + (k0 + v / (TN / VW)) * p + j0 + (v % (TN / VW)) * VW);
            }
            return;
        }
#pragma unroll
        for (int s = 0; s < A_PER; ++s) {
            const int v = t + 256 * s;
            V val;
#pragma unroll
            for (int e = 0; e < VW; ++e) ((T *)&val)[e] = T(0);
            if (v < A_VECS && !a_col) {
                const int row = v / (BK / VW);
                const int kv = (v % (BK / VW)) * VW;
                const int64_t i = i0 + row, k = k0 + kv;
                if (i < m) {
                    if (vec_a && k + VW <= n) {
                        val = *reinterpret_cast<const V *>(A + i * n + k);
                    } else {
#pragma unroll
                        for (int e = 0; e < VW; ++e)
                            if (k + e < n) ((T *)&val)[e] = A[i * n + k + e];
                    }
                }
            } else if (v < A_VECS) {
                // column-major A: element (i, k) at i + k m; a vector runs along i
                const int kk = v / (TM / VW);
                const int iv = (v % (TM / VW)) * VW;
                const int64_t i = i0 + iv, k = k0 + kk;
                if (k < n) {
                    if (vec_a && i + VW <= m) {
                        val = *reinterpret_cast<const V *>(A + k * m + i);
                    } else {
#pragma unroll
                        for (int e = 0; e < VW; ++e)
                            if (i + e < m) ((T *)&val)[e] = A[k * m + i + e];
                    }
                }
            }
            ra[s] = val;
        }
#pragma unroll
        for (int s = 0; s < B_PER; ++s) {
            const int v = t + 256 * s;
            V val;
#pragma unroll
            for (int e = 0; e < VW; ++e) ((T *)&val)[e] = T(0);
            if (v < B_VECS && !b_col) {
                const int kk = v / (TN / VW);
                const int jv = (v % (TN / VW)) * VW;
                const int64_t k = k0 + kk, j = j0 + jv;
                if (k < n) {
                    if (vec_b && j + VW <= p) {
                        val = *reinterpret_cast<const V *>(B + k * p + j);
                    } else {
#pragma unroll
                        for (int e = 0; e < VW; ++e)
                            if (j + e < p) ((T *)&val)[e] = B[k * p + j + e];
                    }
                }
            } else if (v < B_VECS) {
                // column-major B: element (k, j) at k + j n; a vector runs along k
                const int jj = v / (BK / VW);
                const int kv = (v % (BK / VW)) * VW;
                const int64_t j = j0 + jj, k = k0 + kv;
                if (j < p) {
                    if (vec_b && k + VW <= n) {
                        val = *reinterpret_cast<const V *>(B + j * n + k);
                    } else {
#pragma unroll
                        for (int e = 0; e < VW; ++e)
                            if (k + e < n) ((T *)&val)[e] = B[j * n + k + e];
                    }
                }
            }
            rb[s] = val;
        }
    };
    auto store_slab = [&](int buf) {
#pragma unroll
        for (int s = 0; s < A_PER; ++s) {
            const int v = t + 256 * s;
            if (v < A_VECS && !a_col) {
                const int row = v / (BK / VW);
                const int kv = (v % (BK / VW)) * VW;
                *reinterpret_cast<V *>(&As[buf][row * LDA + kv]) = ra[s];
            } else if (v < A_VECS) {           // transposed into the row-major slab
                const int kk = v / (TM / VW);
                const int iv = (v % (TM / VW)) * VW;
#pragma unroll
                for (int e = 0; e < VW; ++e) As[buf][(iv + e) * LDA + kk] = ((const T *)&ra[s])[e];
            }
        }
#pragma unroll
        for (int s = 0; s < B_PER; ++s) {
            const int v = t + 256 * s;
            if (v < B_VECS && !b_col) {
                const int kk = v / (TN / VW);
                const int jv = (v % (TN / VW)) * VW;
                *reinterpret_cast<V *>(&Bs[buf][kk * TN + jv]) = rb[s];
            } else if (v < B_VECS) {
                const int jj = v / (BK / VW);
                const int kv = (v % (BK / VW)) * VW;
#pragma unroll
                for (int e = 0; e < VW; ++e) Bs[buf][(kv + e) * TN + jj] = ((const T *)&rb[s])[e];
            }
        }
    };

    // ---- one in-slab step: k ascending ------------------------------------
    auto step = [&](const T *as, const T *bs, int kk) {
        T a[R];
#pragma unroll
        for (int q = 0; q < R; ++q) a[q] = as[(tr + TR * q) * LDA + kk];
        T b[VJ];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const V bv = *reinterpret_cast<const V *>(&bs[kk * TN + g * (TC * VW) + tc * VW]);
#pragma unroll
            for (int e = 0; e < VW; ++e) b[g * VW + e] = ((const T *)&bv)[e];
        }
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int v = 0; v < VJ; ++v) acc[q][v] = fma_t(a[q], b[v], acc[q][v]);
    };

    const int64_t nslabs = (n + BK - 1) / BK;
    if (nslabs > 0) {
        load_slab(0);
        store_slab(0);
        __syncthreads();
    }
    for (int64_t s = 0; s < nslabs; ++s) {
        const int buf = (int)(s & 1);
        const int64_t k0 = s * BK;
        if (s + 1 < nslabs) load_slab(k0 + BK);
        const T *as = As[buf];
        const T *bs = Bs[buf];
        const int64_t kn = n - k0;
        if (kn >= BK) {
#pragma unroll
            for (int kk = 0; kk < BK; kk += VW) {
                // A values for VW consecutive k come from one vector read per row
                V av[R];
#pragma unroll
                for (int q = 0; q < R; ++q)
                    av[q] = *reinterpret_cast<const V *>(&as[(tr + TR * q) * LDA + kk]);
#pragma unroll
                for (int e = 0; e < VW; ++e) {
                    T b[VJ];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const V bv = *reinterpret_cast<const V *>(
                            &bs[(kk + e) * TN + g * (TC * VW) + tc * VW]);
#pragma unroll
                        for (int w = 0; w < VW; ++w) b[g * VW + w] = ((const T *)&bv)[w];
                    }
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const T a = ((const T *)&av[q])[e];
#pragma unroll
                        for (int v = 0; v < VJ; ++v) acc[q][v] = fma_t(a, b[v], acc[q][v]);
                    }
                }
            }
        } else {
            for (int kk = 0; kk < (int)kn; ++kk) step(as, bs, kk);
        }
        if (s + 1 < nslabs) store_slab(buf ^ 1);
        __syncthreads();
    }

    // ---- write the C block: contiguous runs of row i ----------------------
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int64_t i = i0 + tr + (int64_t)TR * q;
        if (i >= m) continue;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t j = j0 + g * (TC * VW) + tc * VW;
            if (vec_c && j + VW <= p) {
                V out;
#pragma unroll
                for (int e = 0; e < VW; ++e) ((T *)&out)[e] = acc[q][g * VW + e];
                *reinterpret_cast<V *>(C + i * p + j) = out;
            } else {
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    if (j + e < p) C[i * p + j + e] = acc[q][g * VW + e];
            }
        }
    }
}

// ONF on the matrix cores. One step of v_mfma_f64_16x16x4 (or
// v_mfma_f32_16x16x4) adds to every element of a 16 x 16 block of C four
// fused multiply-adds, one after another with k ascending and one rounding
// each: D = fma(a3, b3, fma(a2, b2, fma(a1, b1, fma(a0, b0, C)))), subnormals,
// signed zeros and infinities included (compared bit for bit with
// __builtin_fma chains over such values). Issued slab by slab with k
// ascending they are Eq. 3's loop itself, so the results are bitwise those of
// the scalar loop, at the matrix-core rate: 256 lanes' worth of fma per
// instruction instead of 64, so the vector ALU's operand traffic (8 + 8 LDS
// elements per lane for 64 fma) is gone and what bounds the kernel is the
// matrix rate itself (78.6 TF in FP64, 157.3 in FP32). Measured, vector kernel
// of the same blocks and direct-to-LDS ring before: 8192^3 FP32 12.2 -> 7.7 ms
// (90 -> 143 TF), FP64 22.7 -> 16.7 ms (48 -> 66 TF), 1999 x 1531 x 2113 FP64
// 461 -> 244 us, 256^3 FP64 18.7 -> 6.7 us per call.
//
// A workgroup of four waves owns a TM x TN block of C, a wave WM x WN of it as
// 16 x 16 blocks. k is walked in stages of SUB sub-slabs of 64 bytes of k per
// row (8 doubles, 16 floats), which go from memory straight into an LDS ring of
// NST stages (`buffer_load ... lds`, 1 KiB per load). An operand is laid down
// by its contiguous extent, so every layout runs the same loop:
//   k-contiguous (row-major A, column-major B): one 64-byte row per row of the
//     block, 16-byte chunk c of row r at chunk c ^ ((r / 4) mod 4);
//   k-strided (row-major B, column-major A): BK rows of the block's extent,
//     row k turned by 64 bytes (FP32) or 128 bytes (FP64) times k mod 4.
// Both make the 64 lanes of a fragment read (16 rows x 4 k) cover the 64 banks
// evenly. Rows past the operand's end read as zeros (buffer ranges); what lies
// past m or p feeds only elements that are never stored. In the last, partial
// stage k >= n enters as (-0) * (+0): a step that adds -0, which changes no
// value, not even a -0 sum.
template <typename T> struct Mm;
template <> struct Mm<double> {
    typedef double acc_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mfma(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // C row of register r (its column is lane mod 16)
    static __device__ __forceinline__ int row(int r, int lane) { return 4 * r + (lane >> 4); }
};
template <> struct Mm<float> {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mfma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + r; }
};

// One operand's share of a sub-slab: W rows (or columns) of the block, KC
// whether k is its contiguous extent.
template <typename T, int W, bool KC> struct MmOperand {
    static constexpr int ES = (int)sizeof(T), BK = 64 / ES, EPC = 16 / ES;
    static constexpr int BYTES = W * 64;                     // W rows of 64 bytes, or BK rows of W elements
    static constexpr int LOADS = BYTES / 1024;
    static constexpr int CPR = W * ES / 16;                  // 16-byte chunks of a k-strided row
    static_assert(BYTES % 1024 == 0 && CPR <= 64, "whole loads of at most one row each");

    // Vector offset of lane `lane` in load g of a sub-slab; live: rows of the
    // block inside the operand (KC), ld: the operand's leading extent.
    static __device__ __forceinline__ int voffset(int g, int lane, int64_t live, int64_t ld) {
        if constexpr (KC) {
            const int r = 16 * g + (lane >> 2);
            const int c = (lane & 3) ^ ((lane >> 4) & 3);
            return r < live ? (int)((r * ld + EPC * c) * ES) : ring::kDeadVoffset;
        } else {
            const int k = g * (64 / CPR) + lane / CPR;
            const int c = (lane % CPR + CPR - (ES * (k & 3)) % CPR) % CPR;
            return (int)((k * ld + EPC * c) * ES);
        }
    }
    // Byte offset of (row r, k) in the sub-slab.
    static __device__ __forceinline__ int at(int r, int k) {
        if constexpr (KC)
            return r * 64 + (((k / EPC) ^ ((r >> 2) & 3)) << 4) + (k % EPC) * ES;
        else
            return k * (W * ES) + (((r / EPC + ES * (k & 3)) % CPR) << 4) + (r % EPC) * ES;
    }
};

template <typename T, int TM, int TN, int WM, int WN, int SUB, int NST> struct MmCfg {
    static constexpr int ES = (int)sizeof(T), BK = 64 / ES;
    static constexpr int SUB_BYTES = (TM + TN) * 64, STAGE = SUB * SUB_BYTES, LDS = NST * STAGE;
    static constexpr int LPW = STAGE / 1024 / 4;             // loads per wave and stage
    static_assert(STAGE % 4096 == 0 && (NST - 2) * LPW <= 63, "whole loads per wave, countable");
    static_assert((TM / WM) * (TN / WN) == 4, "four waves");
};

template <typename T, int TM, int TN, int WM, int WN, int SUB, int NST, int GK, bool A_COL, bool B_COL>
__device__ __forceinline__ void onf_mm_block(const T *__restrict__ A, const T *__restrict__ B, T *__restrict__ C,
                                             int64_t m, int64_t n, int64_t p, int accumulate, int tiles_m, int tiles_n,
                                             uint8_t *lds) {
    using G = MmCfg<T, TM, TN, WM, WN, SUB, NST>;
    using OA = MmOperand<T, TM, !A_COL>;
    using OB = MmOperand<T, TN, B_COL>;
    using M = Mm<T>;
    constexpr int ES = G::ES, BK = G::BK, LPW = G::LPW, FM = WM / 16, FN = WN / 16, KS = BK / 4;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / (TN / WN), wn = wave % (TN / WN);
    int tm, tn;
    ring::block_of(tiles_m, tiles_n, &tm, &tn);
    const int64_t i0 = (int64_t)tm * TM, j0 = (int64_t)tn * TN;
    const int lr = lane & 15, lk = lane >> 4;               // a fragment's row and k of this lane

    // Load x = wave LPW + q of a stage brings KiB g of its sub-slab u. Its
    // lanes' offsets are the same in every stage; the resource starts at the
    // sub-slab and ends where the operand ends, and moves on by one stage per
    // issue (64-bit scalars: base, bytes left, bytes per stage).
    const int64_t lda = A_COL ? m : n, ldb = B_COL ? n : p;
    const int64_t a_live = m - i0 < TM ? m - i0 : TM, b_live = p - j0 < TN ? p - j0 : TN;
    const char *a_base = reinterpret_cast<const char *>(A + (A_COL ? i0 : i0 * n));
    const char *b_base = reinterpret_cast<const char *>(B + (B_COL ? j0 * n : j0));
    const int64_t a_end = (A_COL ? n * m - i0 : a_live * n) * ES;     // bytes from the base to the live end
    const int64_t b_end = (B_COL ? b_live * n : n * p - j0) * ES;
    const int64_t a_step = (A_COL ? m : 1) * BK * ES, b_step = (B_COL ? 1 : p) * BK * ES;   // bytes per sub-slab
    constexpr int KIB = G::SUB_BYTES / 1024;
    int voff[LPW];
    const char *src[LPW];
    int64_t left[LPW], step_bytes[LPW], k_of[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
        const int x = wave * LPW + q, u = x / KIB, g = x % KIB;         // wave-uniform
        const bool a = g < OA::LOADS;
        voff[q] = a ? OA::voffset(g, lane, a_live, lda) : OB::voffset(g - OA::LOADS, lane, b_live, ldb);
        const int64_t one = a ? a_step : b_step;
        src[q] = (a ? a_base : b_base) + u * one;
        left[q] = (a ? a_end : b_end) - u * one;
        step_bytes[q] = SUB * one;
        k_of[q] = n - u * BK;                                           // k left from this load's first
    }
    auto clip = [](int64_t x) {                                         // 0 .. 2^31 - 1, in 32-bit scalar steps
        const int hi = (int)(x >> 32);
        const uint32_t lo = min((uint32_t)x, 0x7FFFFFFFu);
        return hi < 0 ? 0 : hi > 0 ? 0x7FFFFFFF : (int)lo;
    };
    // The next stage into buf. Past the end the ranges are empty: the loads
    // touch no memory but keep the count of loads in flight.
    auto issue_next = [&](uint8_t *buf) {
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void *)src[q], (short)0, (int)(k_of[q] >> 32) < 0 || k_of[q] == 0 ? 0 : clip(left[q]), 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsrc, (ring::lds_void_t *)(buf + (wave * LPW + q) * 1024), 16, voff[q], 0, 0, 0);
            src[q] += step_bytes[q];
            left[q] -= step_bytes[q];
            k_of[q] -= SUB * BK;
        }
    };

    typename M::acc_t acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = typename M::acc_t{};

    // Fragments are read one unit (GK steps of 4 k) ahead of the matrix-core
    // steps that use them, also across stages: the last unit of a stage is
    // multiplied after the next stage's barrier, behind the reads of its first
    // unit. Two register sets, unit un in set un mod 2. The first stage finds
    // (-0) * (+0) in set 1, which changes no sum.
    constexpr int UNITS = SUB * KS / GK;
    static_assert(KS % GK == 0 && UNITS % 2 == 0, "whole units, an even number per stage");
    T av[2][GK][FM], bv[2][GK][FN];
#pragma unroll
    for (int ks = 0; ks < GK; ++ks) {
#pragma unroll
        for (int a = 0; a < FM; ++a) av[1][ks][a] = -T(0);
#pragma unroll
        for (int b = 0; b < FN; ++b) bv[1][ks][b] = T(0);
    }
    // `live`: k of this stage that exist (TAIL: fewer than the stage holds)
    auto read_unit = [&](const uint8_t *buf, int un, int64_t live, auto tail) {
        constexpr bool TAIL = decltype(tail)::value;
        const int u = un * GK / KS;
        const uint8_t *as = buf + u * G::SUB_BYTES, *bs = as + OA::BYTES;
#pragma unroll
        for (int ks = 0; ks < GK; ++ks) {
            const int k = 4 * (un * GK % KS + ks) + lk;
            const bool dead = TAIL && u * BK + k >= live;
#pragma unroll
            for (int a = 0; a < FM; ++a) {
                const T x = *reinterpret_cast<const T *>(as + OA::at(wm * WM + a * 16 + lr, k));
                av[un & 1][ks][a] = dead ? -T(0) : x;
            }
#pragma unroll
            for (int b = 0; b < FN; ++b) {
                const T x = *reinterpret_cast<const T *>(bs + OB::at(wn * WN + b * 16 + lr, k));
                bv[un & 1][ks][b] = dead ? T(0) : x;
            }
        }
    };
    auto mma_set = [&](int set) {
#pragma unroll
        for (int ks = 0; ks < GK; ++ks)
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b) acc[a][b] = M::mfma(av[set][ks][a], bv[set][ks][b], acc[a][b]);
    };

    // The stage a step's loads fill and the stage it reads are disjoint LDS,
    // passed as restrict pointers so that the fragment reads need not wait for
    // those loads (the explicit wait orders each stage's own loads).
    auto step = [&](uint8_t *__restrict__ dma, const uint8_t *__restrict__ cur) {
        issue_next(dma);
#pragma unroll
        for (int un = 0; un < UNITS; ++un) {
            read_unit(cur, un, 0, std::false_type{});
            mma_set((un & 1) ^ 1);
        }
    };
    constexpr int STEP_K = SUB * BK;
    const int64_t S = (n + STEP_K - 1) / STEP_K, full = n / STEP_K;
    if (S > 0)
        for (int q = 0; q < NST - 1; ++q) issue_next(lds + q * G::STAGE);
    // The accumulate form starts from C, read while the ring fills. Rows and
    // columns past the end read the last one instead (such elements are never
    // stored): without a branch per element all loads are in flight together.
    if (accumulate) {
        int64_t col[FN];
#pragma unroll
        for (int b = 0; b < FN; ++b) col[b] = min(j0 + wn * WN + b * 16 + lr, p - 1);
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T *row = C + min(i0 + wm * WM + a * 16 + M::row(r, lane), m - 1) * p;
#pragma unroll
                for (int b = 0; b < FN; ++b) acc[a][b][r] = row[col[b]];
            }
        __builtin_amdgcn_s_waitcnt(ring::waitcnt_vm(0));
    }
    int rd = 0, wr = NST - 1;                               // ring slots of stages s and s + NST - 1
    for (int64_t s = 0; s < full; ++s) {
        // stage s landed in every wave; every wave has read stage s - 1 (its
        // last unit's reads too: lgkmcnt(0))
        __builtin_amdgcn_s_waitcnt(ring::waitcnt_vm((NST - 2) * LPW) & ~(0xF << 8));
        ring::ring_barrier();
        step(lds + wr * G::STAGE, lds + rd * G::STAGE);
        rd = rd + 1 == NST ? 0 : rd + 1;
        wr = wr + 1 == NST ? 0 : wr + 1;
    }
    mma_set(1);
    // also the last loads' wait: none may land in LDS after the workgroup ends
    __builtin_amdgcn_s_waitcnt(ring::waitcnt_vm(0));
    if (full < S) {
        ring::ring_barrier();
#pragma unroll
        for (int un = 0; un < UNITS; ++un) {
            if (un * GK * 4 >= n - full * STEP_K) break;
            read_unit(lds + rd * G::STAGE, un, n - full * STEP_K, std::true_type{});
            mma_set(un & 1);
        }
    }

    auto store = [&](auto whole_form) {
        constexpr bool WHOLE = decltype(whole_form)::value;  // no row or column past the end
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t i = i0 + wm * WM + a * 16 + M::row(r, lane);
                if (!WHOLE && i >= m) continue;
#pragma unroll
                for (int b = 0; b < FN; ++b) {
                    const int64_t j = j0 + wn * WN + b * 16 + lr;
                    if (WHOLE || j < p) C[i * p + j] = acc[a][b][r];
                }
            }
    };
    if (i0 + TM <= m && j0 + TN <= p) store(std::true_type{});
    else store(std::false_type{});
}

// Workgroups per CU the registers must allow: two, which keep the matrix cores
// fed through each other's barriers (the 128 x 128 FP64 block holds 128
// accumulator registers); one where the ring leaves no room in LDS for a second
// (FP64 64 x 64: four sub-slabs x three stages are 96 KiB).
template <class G> constexpr int mm_workgroups() { return 2 * G::LDS <= 160 * 1024 ? 2 : 1; }
template <typename T, int TM, int TN, int WM, int WN, int SUB, int NST, int GK, bool A_COL, bool B_COL>
__global__ __launch_bounds__(256, (mm_workgroups<MmCfg<T, TM, TN, WM, WN, SUB, NST>>())) void onf_mm_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                        T *__restrict__ C, int64_t m, int64_t n, int64_t p,
                                                        int accumulate, int tiles_m, int tiles_n) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[MmCfg<T, TM, TN, WM, WN, SUB, NST>::LDS];
    onf_mm_block<T, TM, TN, WM, WN, SUB, NST, GK, A_COL, B_COL>(A, B, C, m, n, p, accumulate, tiles_m, tiles_n, lds);
}

template <typename T, int TM, int TN, int WM, int WN, int SUB, int NST, int GK, bool ANY_LAYOUT>
hipError_t launch_mm(const moa_gemm_desc &d, hipStream_t st) {
    const T *A = static_cast<const T *>(d.A);
    const T *B = static_cast<const T *>(d.B);
    T *C = static_cast<T *>(d.C);
    const int tiles_m = (int)((d.m + TM - 1) / TM), tiles_n = (int)((d.p + TN - 1) / TN);
    const dim3 grid((unsigned)((int64_t)tiles_m * tiles_n)), bl(256);
    const bool ac = ANY_LAYOUT && (d.flags & MOA_FLAG_A_COL), bc = ANY_LAYOUT && (d.flags & MOA_FLAG_B_COL);
    if constexpr (ANY_LAYOUT) {
        if (ac && bc)
            hipLaunchKernelGGL((onf_mm_kernel<T, TM, TN, WM, WN, SUB, NST, GK, true, true>), grid, bl, 0, st, A, B, C, d.m,
                               d.n, d.p, d.accumulate, tiles_m, tiles_n);
        else if (ac)
            hipLaunchKernelGGL((onf_mm_kernel<T, TM, TN, WM, WN, SUB, NST, GK, true, false>), grid, bl, 0, st, A, B, C,
                               d.m, d.n, d.p, d.accumulate, tiles_m, tiles_n);
        else if (bc)
            hipLaunchKernelGGL((onf_mm_kernel<T, TM, TN, WM, WN, SUB, NST, GK, false, true>), grid, bl, 0, st, A, B, C,
                               d.m, d.n, d.p, d.accumulate, tiles_m, tiles_n);
    }
    if (!ac && !bc)
        hipLaunchKernelGGL((onf_mm_kernel<T, TM, TN, WM, WN, SUB, NST, GK, false, false>), grid, bl, 0, st, A, B, C, d.m,
                           d.n, d.p, d.accumulate, tiles_m, tiles_n);
    return hipGetLastError();
}

// Instantiation tables. The first entry per type is the paper's static block
// for the 32 KB vector L1 (three blocks of A, B and C): 1024 FP64 components
// (32 x 32) and 2048 FP32 components (32 x 64). Larger entries trade LDS for
// register blocking; the planner picks among them. Per entry: the block, the
// wave's part of it and the LDS ring (sub-slabs per stage, stages) of the
// matrix-core kernel, then slab and lane block of the register-staged kernel
// (0: none, the last entry per type, which takes row-major operands only).
// The small blocks take deep stages: their products are short of workgroups,
// so what counts is how much of k is on its way at once, whole 128-byte lines
// per row and few barriers in the k walk (FP64 64 x 64, 1000^3: 37 us with four
// sub-slabs per stage, 50 with one); three stages beat more (the rest of LDS
// holds further workgroups: FP64 32 x 32, 1999 x 1531 x 2113: 244 us with
// three, 284 with six).
struct OnfShape { int tm, tn, wm, wn, sub, nst, bk, r, vj; };
constexpr OnfShape kF64[] = {{32, 32, 16, 16, 4, 3, 16, 2, 2},
                             {64, 64, 32, 32, 4, 3, 16, 4, 4},
                             {64, 128, 32, 64, 2, 3, 16, 4, 8},
                             {128, 128, 64, 64, 1, 3, 16, 8, 8},
                             {128, 128, 32, 128, 1, 4, 0, 8, 8}};
constexpr OnfShape kF32[] = {{32, 64, 16, 32, 2, 3, 16, 2, 4},
                             {64, 64, 32, 32, 2, 3, 16, 4, 4},
                             {64, 128, 32, 64, 1, 3, 16, 4, 8},
                             {128, 128, 64, 64, 1, 3, 16, 8, 8},
                             {128, 128, 32, 128, 1, 3, 0, 8, 8}};

template <typename T, int TM, int TN, int BK, int R, int VJ>
hipError_t launch_one(const moa_gemm_desc &d, hipStream_t st) {
    const T *A = static_cast<const T *>(d.A);
    const T *B = static_cast<const T *>(d.B);
    T *C = static_cast<T *>(d.C);
    constexpr int VW = Vec<T>::W;
    const int a_col = (d.flags & MOA_FLAG_A_COL) != 0, b_col = (d.flags & MOA_FLAG_B_COL) != 0;
    // 16-byte vectors run along the contiguous extent of each operand
    const int vec_a = ((a_col ? d.m : d.n) % VW == 0) && ((uintptr_t)A % 16 == 0);
    const int vec_b = ((b_col ? d.n : d.p) % VW == 0) && ((uintptr_t)B % 16 == 0);
    const int vec_c = (d.p % VW == 0) && ((uintptr_t)C % 16 == 0);
    dim3 grid((unsigned)((d.p + TN - 1) / TN), (unsigned)((d.m + TM - 1) / TM));
    hipLaunchKernelGGL((onf_kernel<T, TM, TN, BK, R, VJ>), grid, dim3(256), 0, st, A, B, C,
                       d.m, d.n, d.p, d.accumulate, vec_a, vec_b, vec_c, a_col, b_col);
    return hipGetLastError();
}

}  // namespace

int onf_variant_count(moa_dtype t) {
    return t == MOA_F64 ? (int)(sizeof(kF64) / sizeof(kF64[0]))
                        : (int)(sizeof(kF32) / sizeof(kF32[0]));
}

void onf_variant_shape(moa_dtype t, int v, bool staged, Plan *p) {
    const OnfShape s = (t == MOA_F64) ? kF64[v] : kF32[v];
    const int es = (t == MOA_F64) ? 8 : 4;
    p->variant = v;
    p->tile_m = s.tm;
    p->tile_n = s.tn;
    p->threads = 256;
    if (staged) {
        p->tile_k = s.bk;
        p->lane_m = s.r;
        p->lane_n = s.vj;
        p->wave_m = s.r * (64 / (s.tn / s.vj));
        p->wave_n = s.tn;
        p->lds_bytes = 2 * (s.tm * (s.bk + 16 / es) + s.bk * s.tn) * es;
        return;
    }
    p->tile_k = s.sub * 64 / es;
    p->wave_m = s.wm;
    p->wave_n = s.wn;
    p->lane_m = s.wm / 4;               // 4 rows of each 16 x 16 block
    p->lane_n = s.wn / 16;              // 1 column
    p->lds_bytes = s.nst * s.sub * (s.tm + s.tn) * 64;
}

int onf_ring_variant(moa_dtype t) { return onf_variant_count(t) - 1; }

static const OnfShape *shapes_of(const moa_gemm_desc &d) { return d.dtype == MOA_F64 ? kF64 : kF32; }

// The planner's candidates: of the two 128 x 128 blocks the row-major variant
// where it applies; FP64 without it stops at 64 x 128.
static bool onf_eligible(const moa_gemm_desc &d, int v, bool ring_ok) {
    const int ring = onf_ring_variant((moa_dtype)d.dtype);
    return v == ring ? ring_ok : v < ring - 1 || (d.dtype != MOA_F64 && !ring_ok);
}

int onf_largest_rows(const moa_gemm_desc &d, bool ring_ok) {
    int v = onf_ring_variant((moa_dtype)d.dtype);
    while (!onf_eligible(d, v, ring_ok)) --v;
    return shapes_of(d)[v].tm;
}

bool onf_launches(const moa_gemm_desc &d, int v) {
    const OnfShape s = shapes_of(d)[v];
    const int64_t rows = (d.m + s.tm - 1) / s.tm, cols = (d.p + s.tn - 1) / s.tn;
    const int64_t lim = (int64_t(1) << 24) - 1;              // workgroups of 256 threads in x
    return onf_mm_fits(d, v) ? rows * cols <= lim : rows <= 65535 && cols <= lim;
}

// The planner's block: the one whose workgroups, dealt out over the CUs, leave
// the busiest CU the least to do -- ceil(blocks / CUs) times the block's k steps,
// its area weighted by its measured time per element of C (4096^3: FP64 2.28 ms
// with 32 x 32 blocks, 2.12 with 64 x 64 and the larger ones; FP32 1.13 ms with
// 32 x 64, 1.03 with 64 x 64, 1.02 with 64 x 128, 0.99 with 128 x 128), and what a
// block takes outside its k walk: filling the ring and writing C (with the
// accumulate form reading it), which larger blocks hide better. That is counted
// in k steps, fitted to 23 shapes with n from 8 to 300; in FP64, where it is
// mostly C's traffic, for the part of the block inside C. The matrix cores are
// shared by a CU's workgroups, so a CU with two blocks takes twice as long as its
// neighbours with one: 1999 x 1531 x 2113 in FP64 has 272 blocks of 128 x 128 and
// takes 403 us with them, 258 with 64 x 64 and 244 with 32 x 32; 256^3 takes 41, 11
// and 4.8 us. With a short walk it is the other way round: 6000 x 30 x 6000 in FP64
// 75 us with 128 x 128, 123 with 64 x 64 and 110 with 32 x 32. Ties go to the larger
// block. 128 x 128 blocks only where every CU gets one. Blocks whose grid does not
// hold the product (fewer than 2^32 threads in x; the register-staged kernel's rows
// of blocks are its grid's y) are not candidates.
int onf_default_variant(const moa_gemm_desc &d, bool ring_ok) {
    constexpr double kWeight64[] = {1.07, 1.0, 1.0, 1.0, 1.0}, kWeight32[] = {1.13, 1.035, 1.03, 1.0, 1.0};
    // k steps' worth of time outside the walk: overwrite, accumulate
    constexpr int kEdge64[][5] = {{72, 78, 48, 34, 40}, {125, 138, 92, 76, 78}};
    constexpr int kEdge32[][5] = {{67, 56, 33, 34, 35}, {95, 95, 57, 68, 72}};
    const bool f64 = d.dtype == MOA_F64;
    const OnfShape *shapes = shapes_of(d);
    const double *weight = f64 ? kWeight64 : kWeight32;
    const int *edge = (f64 ? kEdge64 : kEdge32)[d.accumulate ? 1 : 0];
    const int ring = onf_ring_variant((moa_dtype)d.dtype);
    int best = 0;
    double best_cost = 0;
    for (int v = ring; v >= 0; --v) {
        if (!onf_eligible(d, v, ring_ok) || !onf_launches(d, v)) continue;
        const OnfShape s = shapes[v];
        const int64_t blocks = ((d.m + s.tm - 1) / s.tm) * ((d.p + s.tn - 1) / s.tn);
        if (s.tm * s.tn == 128 * 128 && blocks < kNumCUs) continue;
        const double area = s.tm * s.tn, live = f64 ? (double)d.m * (double)d.p / (double)blocks : area;
        const double cost = (double)((blocks + kNumCUs - 1) / kNumCUs) * weight[v] *
                            (area * (double)d.n + live * (double)edge[v]);
        if (best_cost == 0 || cost < best_cost) {
            best = v;
            best_cost = cost;
        }
    }
    return best;
}

// The matrix-core kernel's 32-bit buffer offsets: a k-contiguous operand spans
// the block's rows of n elements, a k-strided one the k of a sub-slab times its
// leading extent. Products beyond that run the register-staged kernel of the
// same block (64-bit addresses); the last entry has none and is refused there.
bool onf_mm_fits(const moa_gemm_desc &d, int v) {
    const OnfShape s = d.dtype == MOA_F64 ? kF64[v] : kF32[v];
    const int64_t es = d.dtype == MOA_F64 ? 8 : 4, bk = 64 / es, lim = 0x7FFFFFFF;
    if (d.m > lim || d.n > lim || d.p > lim) return false;
    const int64_t a = (d.flags & MOA_FLAG_A_COL) ? (bk + 1) * d.m : (int64_t)(s.tm + 2) * d.n;
    const int64_t b = (d.flags & MOA_FLAG_B_COL) ? (int64_t)(s.tn + 2) * d.n : (bk + 1) * d.p;
    return a * es < lim && b * es < lim;
}

hipError_t launch_onf(const moa_gemm_desc &d, const Plan &plan, hipStream_t st) {
    const bool mm = onf_mm_fits(d, plan.variant);
    if (d.dtype == MOA_F64) {
        switch (plan.variant) {
        case 0: return mm ? launch_mm<double, 32, 32, 16, 16, 4, 3, 2, true>(d, st) : launch_one<double, 32, 32, 16, 2, 2>(d, st);
        case 1: return mm ? launch_mm<double, 64, 64, 32, 32, 4, 3, 1, true>(d, st) : launch_one<double, 64, 64, 16, 4, 4>(d, st);
        case 2: return mm ? launch_mm<double, 64, 128, 32, 64, 2, 3, 1, true>(d, st) : launch_one<double, 64, 128, 16, 4, 8>(d, st);
        case 3: return mm ? launch_mm<double, 128, 128, 64, 64, 1, 3, 1, true>(d, st) : launch_one<double, 128, 128, 16, 8, 8>(d, st);
        default: return launch_mm<double, 128, 128, 32, 128, 1, 4, 1, false>(d, st);
        }
    }
    switch (plan.variant) {
    case 0: return mm ? launch_mm<float, 32, 64, 16, 32, 2, 3, 2, true>(d, st) : launch_one<float, 32, 64, 16, 2, 4>(d, st);
    case 1: return mm ? launch_mm<float, 64, 64, 32, 32, 2, 3, 2, true>(d, st) : launch_one<float, 64, 64, 16, 4, 4>(d, st);
    case 2: return mm ? launch_mm<float, 64, 128, 32, 64, 1, 3, 1, true>(d, st) : launch_one<float, 64, 128, 16, 4, 8>(d, st);
    case 3: return mm ? launch_mm<float, 128, 128, 64, 64, 1, 3, 1, true>(d, st) : launch_one<float, 128, 128, 16, 8, 8>(d, st);
    default: return launch_mm<float, 128, 128, 32, 128, 1, 3, 1, false>(d, st);
    }
}

}  // namespace moa
