// lu64.hip -- blocked LU in FP64 on the FP64 matrix cores, with or without
// partial pivoting, and the matching triangular solves.
//
// Two uses (paper: "Background" -- the figure of merit is measured against
// the FP64 solve of HPL; "Experimental Results" -- the pivoting study of
// Figures 2-4, LU in 64-bit arithmetic with and without partial pivoting):
//   * the FP64 baseline of the mixed-precision solve (same GPU, same timer);
//   * the largest pivot and the residual norms of FP64 LU with and without
//     partial pivoting on matrices with entries uniform in [-1, 1).
//
// Right-looking, block size nb (64 or 128).  Per block step k, m = n - k:
//   without pivoting: the nb x nb diagonal block is factored by one
//     work-group in LDS (k_diag64); L21 = A21 U11^-1 and U12 = L11^-1 A12 by
//     blocked substitution, its products on the matrix cores (k_trsm64);
//   with pivoting: a panel of up to 8192 rows is factored a few columns at a
//     time by one work-group (k_panel64_wg, k_panel64_rest), a larger one by
//     one cooperative launch (k_panel64_pp): every work-group holds a slice of
//     the panel's rows in LDS; per column each proposes its largest-magnitude candidate, a grid
//     barrier, every work-group picks the same winner (largest magnitude,
//     smallest row among equals -- the rule of LAPACK's getrf), the two rows
//     trade places and every work-group eliminates its rows.  The swaps are
//     then applied to the columns left and right of the panel (k_laswp64)
//     and U12 formed as above;
//   both: A22 <- A22 - L21 U12 with v_mfma_f64_16x16x4f64 (k_gemm64), without
//     pivoting for four blocks at a time while the matrix is large.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <mutex>
#include <type_traits>

#include "../../include/mxp.h"
#include "common.hpp"
#include "kernels.hpp"
#include "prof.hpp"

namespace mxp {

typedef double d4v __attribute__((ext_vector_type(4)));

// ============================================================== trailing update
// C (M x N, ldc) -= A (M x K, lda) B (K x N, ldb), all column-major FP64.
// Work-group tile 128 x 128, four waves of 64 x 64 (4 x 4 blocks of the
// 16 x 16 MFMA).  Lane l of an MFMA supplies P[l%16][l/16] and Q[l/16][l%16]
// of a 16 x 4 by 4 x 16 step and holds D[l/16 + 4q][l%16], q < 4.  The
// product is formed transposed (P = B^T, Q = A^T), so that the 16 lanes of a
// result row are 16 consecutive rows of C (128 bytes per access).
//
// Bound: a k-step of four takes a wave 16 MFMAs of 64 cycles; its operands
// read straight from memory (32-byte pieces of B, one step ahead) left the
// matrix cores waiting.  Both operands are staged through LDS instead, 16 of
// K at a time, the next stage's copies (16 bytes per lane straight into LDS)
// in flight behind the current one's 64 MFMAs; 69 KB per work-group, so two
// share a CU and one's C update overlaps the other's products.  A rows stand
// at a pitch of 144 (the two k of a 32-lane half on different banks), the
// 16-byte chunks of a B column are XOR-swizzled by the column.  Tiles past an
// edge, ragged K and columns that are not 16-byte aligned take guarded loads
// into the same layout.
constexpr int G64_T = 128;
constexpr int G64_K = 16;                        // K per stage
constexpr int G64_PA = 144;                      // doubles between two k of the A stage
constexpr int G64_SA = G64_K * G64_PA;           // doubles of an A stage
constexpr int G64_SB = G64_T * G64_K;            // doubles of a B stage
constexpr size_t G64_LDS = 2 * (size_t)(G64_SA + G64_SB) * 8;

MXP_DEV int g64_key(int col) { return (col >> 1) & 7; }
// element (k, col) of a B stage
MXP_DEV int g64_boff(int k, int col) { return col * G64_K + (((k >> 1) ^ g64_key(col)) << 1) + (k & 1); }

__global__ __launch_bounds__(256, 2) void k_gemm64(double* __restrict__ C, int64_t ldc, const double* __restrict__ A,
                                                   int64_t lda, const double* __restrict__ B, int64_t ldb, int64_t M,
                                                   int64_t N, int K, int aligned, int tm, int ne) {
    extern __shared__ __attribute__((aligned(16))) double gsm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int li = lane & 15, lk = lane >> 4;
    // tiles: the first ne tile columns whole (tm tile rows each), the first ne tile
    // rows of the columns after them
    const int t = (int)blockIdx.x, u = t - tm * ne;
    const int64_t row0 = (int64_t)(u < 0 ? t % tm : u % ne) * G64_T;
    const int64_t col0 = (int64_t)(u < 0 ? t / tm : ne + u / ne) * G64_T;
    const bool inside = aligned && row0 + G64_T <= M && col0 + G64_T <= N;
    auto stage = [&](int k0, int buf) {
        double* sA = gsm + buf * (G64_SA + G64_SB);
        double* sB = sA + G64_SA;
        if (inside && k0 + G64_K <= K) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int kk = 4 * wave + i;                  // one k: 128 rows, 1 KB
                dma16((const char*)(A + row0 + 2 * lane + (int64_t)(k0 + kk) * lda), (char*)(sA + kk * G64_PA));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = 4 * wave + i;                   // eight columns, 1 KB
                const int c = 8 * j + (lane >> 3);
                const int q = (lane & 7) ^ g64_key(c);        // logical chunk kept at this lane's place
                dma16((const char*)(B + (k0 + 2 * q) + (col0 + c) * ldb), (char*)(sB + j * 128));
            }
        } else {
            double va[8], vb[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = tid + 256 * i;
                const int r = e & 127, ka = e >> 7, kb = e & 15, c = e >> 4;
                va[i] = row0 + r < M && k0 + ka < K ? A[row0 + r + (int64_t)(k0 + ka) * lda] : 0.0;
                vb[i] = col0 + c < N && k0 + kb < K ? B[k0 + kb + (col0 + c) * ldb] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = tid + 256 * i;
                sA[(e >> 7) * G64_PA + (e & 127)] = va[i];
                sB[g64_boff(e & 15, e >> 4)] = vb[i];
            }
        }
    };
    d4v acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = d4v{0.0, 0.0, 0.0, 0.0};
    const int nst = (K + G64_K - 1) / G64_K;
    stage(0, 0);
    for (int st = 0; st < nst; ++st) {
        __builtin_amdgcn_s_waitcnt(0);        // this wave's part of stage st is in LDS
        __syncthreads();                      // everyone's is; stage st - 1's buffer is free
        if (st + 1 < nst) stage((st + 1) * G64_K, (st + 1) & 1);
        const double* sA = gsm + (st & 1) * (G64_SA + G64_SB);
        const double* sB = sA + G64_SA;
#pragma unroll
        for (int ks = 0; ks < G64_K / 4; ++ks) {
            double fa[4], fb[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) fa[a] = sA[(4 * ks + lk) * G64_PA + wm * 64 + a * 16 + li];
#pragma unroll
            for (int b = 0; b < 4; ++b) fb[b] = sB[g64_boff(4 * ks + lk, wn * 64 + b * 16 + li)];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[b], fa[a], acc[a][b], 0, 0, 0);
        }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int64_t r = row0 + wm * 64 + a * 16 + li;
            const int64_t c0 = col0 + wn * 64 + b * 16 + lk;
            if (inside) {
                double* p = C + r + c0 * ldc;
                double x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = p[(int64_t)(4 * q) * ldc];
#pragma unroll
                for (int q = 0; q < 4; ++q) p[(int64_t)(4 * q) * ldc] = x[q] - acc[a][b][q];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r < M && c0 + 4 * q < N) C[r + (c0 + 4 * q) * ldc] -= acc[a][b][q];
            }
        }
}

// edge < 0: all of C; otherwise its first edge columns and the rest of its first
// edge rows (edge a multiple of the tile)
static hipError_t gemm64_part(double* C, int64_t ldc, const double* A, int64_t lda, const double* B, int64_t ldb,
                              int64_t M, int64_t N, int K, int64_t edge, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    if (K % 4 || edge % G64_T > 0) return hipErrorInvalidValue;
    const int64_t tm = (M + G64_T - 1) / G64_T, tn = (N + G64_T - 1) / G64_T;
    const int64_t ne = edge < 0 || edge / G64_T > tn ? tn : edge / G64_T;
    const int64_t nr = ne < tm ? ne : tm;
    if (ne == 0) return hipSuccess;
    if (ne < tn && nr < ne) return hipErrorInvalidValue;
    static const hipError_t attr =
        hipFuncSetAttribute((const void*)k_gemm64, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G64_LDS);
    if (attr) return attr;
    hipEvent_t pt = prof::begin(prof::GEMM64, s);
    // 16-byte copies need even leading dimensions and 16-byte aligned operands
    const int aligned = lda % 2 == 0 && ldb % 2 == 0 && ((uintptr_t)A | (uintptr_t)B) % 16 == 0;
    k_gemm64<<<(unsigned)(tm * ne + nr * (tn - ne)), 256, G64_LDS, s>>>(C, ldc, A, lda, B, ldb, M, N, K, aligned,
                                                                        (int)tm, (int)ne);
    const double mn = ne == tn ? M * (double)N : (double)edge * (M + N - edge);
    prof::end(pt, prof::GEMM64, s, 2.0 * mn * K, 16.0 * mn + 8.0 * (M + N) * K);
    return hipGetLastError();
}

hipError_t gemm64(double* C, int64_t ldc, const double* A, int64_t lda, const double* B, int64_t ldb, int64_t M,
                  int64_t N, int K, hipStream_t s) {
    return gemm64_part(C, ldc, A, lda, B, ldb, M, N, K, -1, s);
}

// The same update by rocBLAS's dgemm (a plain library GEMM), for the FP64
// baseline at the speed of the vendor library.  One handle per device; the
// stream is set and the call enqueued under a lock (a handle holds one
// stream at a time).
static std::mutex g_blas_mutex;
static rocblas_handle g_blas[64];

hipError_t gemm64_rocblas(double* C, int64_t ldc, const double* A, int64_t lda, const double* B, int64_t ldb,
                          int64_t M, int64_t N, int K, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_blas_mutex);
    if (!g_blas[dev] && rocblas_create_handle(&g_blas[dev]) != rocblas_status_success) return hipErrorUnknown;
    if (rocblas_set_stream(g_blas[dev], s) != rocblas_status_success) return hipErrorUnknown;
    const double alpha = -1.0, beta = 1.0;
    hipEvent_t pt = prof::begin(prof::GEMM64, s);
    const rocblas_status st = rocblas_dgemm(g_blas[dev], rocblas_operation_none, rocblas_operation_none,
                                            (rocblas_int)M, (rocblas_int)N, (rocblas_int)K, &alpha, A,
                                            (rocblas_int)lda, B, (rocblas_int)ldb, &beta, C, (rocblas_int)ldc);
    prof::end(pt, prof::GEMM64, s, 2.0 * M * (double)N * K, 16.0 * M * (double)N + 8.0 * (M + N) * K);
    return st == rocblas_status_success ? hipSuccess : hipErrorUnknown;
}

// ============================================================== block triangles
// The triangular solves of a block step cut the nb x nb triangle into 16 x 16
// blocks: the blocks below its diagonal (of L11, and of U11 transposed) are
// MFMA operands, block (i, j), i > j, k-step ks of lane l at
// 256 (i (i + 1) / 2 + j) + 64 ks + l = M[16 i + l % 16][16 j + 4 ks + l / 16];
// the diagonal blocks are solved by substitution (tri_solve16), their entry
// M[r][e], r >= e, at 256 (i (i + 3) / 2) + tri_pos(r, e), with the reciprocals of
// U11's diagonal in places of the other triangle (tri_rp).
constexpr int TB = 16;                              // triangle block
constexpr int TRI_MAX = 8 * 9 / 2 * 256;            // doubles of one packed triangle (nb = 128)
MXP_DEV int tri_off(int i, int j) { return (i * (i + 1) / 2 + j) * 256; }
MXP_DEV int tri_pos(int r, int e) { return 16 * e + 4 * (r & 3) + (r >> 2); }
MXP_DEV int tri_rp(int e) { return e ? tri_pos(e - 1, e) : tri_pos(0, 15); }

// lane row G (of four) of the wave to all of them
MXP_DEV int rows_bcast32(int v, int G) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const int r = (G & 1) ? p[1] : p[0];
    const auto o = __builtin_amdgcn_permlane32_swap(r, r, false, false);
    return (G & 2) ? o[1] : o[0];
}
MXP_DEV double rows_bcast(double v, int G) {
    return __hiloint2double(rows_bcast32(__double2hiint(v), G), rows_bcast32(__double2loint(v), G));
}

// M^-1 x0 for a lower 16 x 16 triangle and sixteen lines at once: entry 4 q + g of
// line c in register q of lane 16 g + c (the layout of the MFMA's result and of
// its next operand).  coef(e): this lane's M[4 q + g][e], q = 0 ..
// 3 (not used where not below the diagonal); DIV: diagonal diag(e) with
// reciprocal rp(e), else 1.  A step's quotient is the product with the
// reciprocal and one residual correction; where any result is not finite -- a
// zero, subnormal or infinite diagonal entry, an infinite entry, an overflow --
// the solve is made again with true quotients.  All coefficients are loaded
// first: loaded step by step, each step waits for its own.
// (Substitution, not the product with the block's inverse: without pivoting these
// blocks are badly conditioned as a rule on uniform entries, and the product then
// loses the accuracy that its conditioning takes: largest |LU - A| / (eps |L||U|)
// 363 against 2.4 at n = 4600, scaled residual of the solve 33 against 7 at
// n = 2000.)
template <bool DIV, class FC, class FD, class FR>
MXP_DEV d4v tri_solve16(const d4v x0, FC coef, FD diag, FR rp) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
    d4v m[TB];
    double d[TB], r[TB];
#pragma unroll
    for (int e = 0; e < TB; ++e) {
        m[e] = coef(e);
        if constexpr (DIV) { d[e] = diag(e); r[e] = rp(e); }
    }
    __builtin_amdgcn_sched_barrier(0);
    d4v x = x0, y;
#pragma unroll
    for (int e = 0; e < TB; ++e) {
        double t = x[e >> 2];
        if constexpr (DIV) {
            const double q = t * r[e];
            t = fma(fma(-d[e], q, t), r[e], q);
        }
        const double b = rows_bcast(t, e & 3);
        y[e >> 2] = g == (e & 3) ? b : y[e >> 2];
        // (rows at or above e are done: their part of x is no longer read)
#pragma unroll
        for (int q = e >> 2; q < 4; ++q) x[q] = fma(-m[e][q], b, x[q]);
    }
    if constexpr (DIV) {
        if (!__all(isfinite(y[0]) && isfinite(y[1]) && isfinite(y[2]) && isfinite(y[3]))) {
            x = x0;
#pragma unroll 1
            for (int e = 0; e < TB; ++e) {
                const d4v me = coef(e);
                const int q0 = e >> 2;
                double t = q0 == 0 ? x[0] : q0 == 1 ? x[1] : q0 == 2 ? x[2] : x[3];
                t = t / diag(e);
                const double b = __shfl(t, 16 * (e & 3) + (lane & 15), 64);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (4 * q + g > e) x[q] -= me[q] * b;
                    y[q] = 4 * q + g == e ? b : y[q];
                }
            }
        }
    }
    return y;
}

// lane J of each 16-lane row to the whole row
template <int J> MXP_DEV double row_bcast(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + J, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + J, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// step J of the LU of a 16 x 16 block, row r in the lanes r + 16 g, columns
// in registers; a zero or non-finite pivot is recorded and its column left
template <int J> MXP_DEV void leaf64(double (&x)[TB], int r, int& bad) {
    if constexpr (J < TB) {
        const double pv = row_bcast<J>(x[J]);
        const bool ok = pv != 0.0 && isfinite(pv);
        if (!ok && bad < 0) bad = J;
        const double rp = 1.0 / pv;
        const double l = (ok && r > J) ? x[J] * rp : 0.0;
        if (ok && r > J) x[J] = l;
#pragma unroll
        for (int c = J + 1; c < TB; ++c) x[c] = fma(-l, row_bcast<J>(x[c]), x[c]);
        leaf64<J + 1>(x, r, bad);
    }
}

// ============================================================== diagonal block (no pivoting)
// LU of the kb x kb block at A[k, k] (kb <= 128) by one work-group: the block
// in LDS (padded with the identity to a multiple of 16, pitch D64P), right-
// looking over 16 x 16 blocks.  Per step, wave 0 factors the diagonal block
// in registers (one row per lane, the pivot row broadcast along a 16-lane row
// by DPP); the waves then solve the strips against it (tri_solve16, sixteen rows
// or columns each) and update the rest on the FP64 matrix cores, wave 0 taking
// the next diagonal block first and going on to its LU.  The chain of leaf and
// strip is what bounds it.  A zero / non-finite pivot sets *info; the packed
// triangles of L11 and U11^T go to PL and PU.
constexpr int D64P = 130;
constexpr size_t D64_LDS = (size_t)(128 * D64P + TB) * 8;

__global__ __launch_bounds__(512) void k_diag64(double* A, int64_t lda, int64_t k, int kb, double* PL, double* PU,
                                                unsigned long long* info) {
    extern __shared__ __attribute__((aligned(16))) double gsm[];
    double* D = gsm;                                  // D[c * D64P + r]
    double* sR = gsm + 128 * D64P;                    // reciprocals of the step's pivots
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int P = (kb + TB - 1) / TB, kp = P * TB;
    for (int e = tid; e < 128 * kp; e += 512) {
        const int r = e & 127, c = e >> 7;
        if (r < kp) D[c * D64P + r] = r < kb && c < kb ? A[(k + r) + (k + c) * lda] : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    // C(i,j) -= L(i,t) U(t,j)
    auto update = [&](int i, int j, int t) {
        d4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(D[(TB * t + 4 * ks + lk) * D64P + TB * i + li],
                                                       D[(TB * j + li) * D64P + TB * t + 4 * ks + lk], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) D[(TB * j + li) * D64P + TB * i + lk + 4 * q] -= acc[q];
    };
    for (int t = 0; t < P; ++t) {
        const int o = TB * t;
        if (wave == 0) {
            if (t > 0) update(t, t, t - 1);
            asm volatile("" ::: "memory");
            double x[TB];
#pragma unroll
            for (int c = 0; c < TB; ++c) x[c] = D[(o + c) * D64P + o + li];
            int bad = -1;
            leaf64<0>(x, li, bad);
            if (bad >= 0 && lane == 0) atomicMin(info, (unsigned long long)(k + o + bad + 1));
            double dg = 1.0;
#pragma unroll
            for (int c = 0; c < TB; ++c) {
                if (c == li) dg = x[c];
                if (lk == 0) D[(o + c) * D64P + o + li] = x[c];
            }
            if (lk == 0) sR[li] = 1.0 / dg;
        } else if (t > 0) {
            // the rest of update t - 1
            const int w = P - t;
            for (int u = wave; u < w * w; u += 7) update(t + u % w, t + u / w, t - 1);
        }
        __syncthreads();
        const int w = P - 1 - t;
        for (int u = wave; u < 2 * w; u += 8) {
            if (u < w) {
                // rows of block (i,t), against U_tt^T
                double* p = D + (o + lk) * D64P + TB * (t + 1 + u) + li;
                const d4v x = tri_solve16<true>(
                    d4v{p[0], p[4 * D64P], p[8 * D64P], p[12 * D64P]},
                    [&](int e) {
                        d4v m;
#pragma unroll
                        for (int q = 0; q < 4; ++q) m[q] = D[(o + 4 * q + lk) * D64P + o + e];
                        return m;
                    },
                    [&](int e) { return D[(o + e) * D64P + o + e]; }, [&](int e) { return sR[e]; });
#pragma unroll
                for (int q = 0; q < 4; ++q) p[4 * q * D64P] = x[q];
            } else {
                // columns of block (t,j), against L_tt
                double* p = D + (TB * (t + 1 + u - w) + li) * D64P + o + lk;
                const d4v x = tri_solve16<false>(
                    d4v{p[0], p[4], p[8], p[12]},
                    [&](int e) {
                        d4v m;
#pragma unroll
                        for (int q = 0; q < 4; ++q) m[q] = D[(o + e) * D64P + o + 4 * q + lk];
                        return m;
                    },
                    [](int) { return 1.0; }, [](int) { return 1.0; });
#pragma unroll
                for (int q = 0; q < 4; ++q) p[4 * q] = x[q];
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < 128 * kb; e += 512) {
        const int r = e & 127, c = e >> 7;
        if (r < kb) A[(k + r) + (k + c) * lda] = D[c * D64P + r];
    }
    // the packed triangles: the blocks below the diagonal as operands, the
    // diagonal blocks for the substitution (entry f = tri_pos(r, e))
    for (int u = wave; u < P * (P + 1) / 2; u += 8) {
        int i = 0, v = u;
        while (v > i) v -= ++i;
        double *pl = PL + tri_off(i, v), *pu = PU + tri_off(i, v);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int f = 64 * ks + lane;
            if (v < i) {
                pl[f] = D[(TB * v + 4 * ks + lk) * D64P + TB * i + li];
                pu[f] = D[(TB * i + li) * D64P + TB * v + 4 * ks + lk];
            } else {
                const int e = f >> 4, r = (f >> 2 & 3) + 4 * (f & 3), b = TB * i;
                const int d = r == e - 1 ? e : r == 0 && e == 15 ? 0 : -1;      // the reciprocal kept here
                pl[f] = r > e ? D[(b + e) * D64P + b + r] : 0.0;
                pu[f] = r >= e ? D[(b + r) * D64P + b + e] : d >= 0 ? 1.0 / D[(b + d) * D64P + b + d] : 0.0;
            }
        }
    }
}

// the packed triangle of L11 from a factored nb x nb block (pivoted panels)
__global__ __launch_bounds__(512) void k_pack64(const double* __restrict__ A, int64_t lda, int64_t k, int nb,
                                                double* __restrict__ PL) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int P = nb / TB;
    const double* B = A + k + k * lda;
    for (int u = wave; u < P * (P + 1) / 2; u += 8) {
        int i = 0, v = u;
        while (v > i) v -= ++i;
        double* pl = PL + tri_off(i, v);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int f = 64 * ks + lane, e = f >> 4, r = (f >> 2 & 3) + 4 * (f & 3);
            if (v < i) pl[f] = B[TB * i + li + (int64_t)(TB * v + 4 * ks + lk) * lda];
            else pl[f] = r > e ? B[TB * i + r + (int64_t)(TB * i + e) * lda] : 0.0;
        }
    }
}

// ============================================================== triangular solves of a block step
// L21 = A21 U11^-1 (as U11^T X = A21^T) and U12 = L11^-1 A12 in one launch:
// a wave takes 16 rows of A21 (work-groups [0, wgr)) or 16 columns of A12 (the
// rest) and holds all nb entries of each in registers, in the MFMA result
// layout, whose registers are also the operands of the next product.  Per
// 16-block i: X(i) <- M(i,i)^-1 X(i) by substitution (tri_solve16), then X(j) -=
// M(j,i) X(i) for the blocks after it on the matrix cores (the packed triangle's
// operands read as whole 512-byte lines).  The chain of a wave bounds it; one
// thread per row or column with its entries in LDS was a chain of nb^2/2 dependent
// LDS reads.  The blocks move one place through the registers per step, so that
// the loop is one copy of its code: eight copies, each run once, were bound by
// fetching them (43 us per launch at n = 8192).
template <int P>
__global__ __launch_bounds__(256) void k_trsm64(double* A, int64_t lda, int64_t n, int64_t k, int wgr,
                                                const double* __restrict__ PL, const double* __restrict__ PU) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const bool right = (int)blockIdx.x < wgr;              // rows of A21
    const int64_t wg = right ? blockIdx.x : blockIdx.x - wgr;
    const double* __restrict__ M = right ? PU : PL;
    // the diagonal blocks in LDS: a substitution step that takes its coefficients
    // from memory waits for them (24 us more per launch at n = 8192)
    __shared__ __attribute__((aligned(32))) double sT[P][256];
#pragma unroll
    for (int i = 0; i < P; ++i) sT[i][threadIdx.x] = M[tri_off(i, i) + threadIdx.x];
    __syncthreads();
    const int64_t o0 = k + TB * P + (wg * 4 + wave) * TB;  // first row / column of the wave
    if (o0 >= n) return;
    const bool in = o0 + li < n;
    const int64_t o = in ? o0 + li : n - 1;
    // entry e of this lane's row / column: base + (4 q + 16 i) step
    double* base = right ? A + o + (k + lk) * lda : A + (k + lk) + o * lda;
    const int64_t step = right ? lda : 1;
    d4v X[P];
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) X[i][q] = base[(int64_t)(TB * i + 4 * q) * step];
    auto solve = [&](auto DIV) {
#pragma unroll 1
        for (int i = 0; i < P; ++i) {
            // the operands of the blocks (i + j, i); X holds the blocks from i on
            d4v m[P];
#pragma unroll
            for (int j = 1; j < P; ++j) {
                const double* __restrict__ Mj = M + tri_off(i + j < P ? i + j : P - 1, i);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) m[j][ks] = Mj[64 * ks + lane];
            }
            const double* T = sT[i];
            const d4v y = tri_solve16<decltype(DIV)::value>(
                X[0], [&](int e) { return *(const d4v*)(T + tri_pos(lk, e)); },
                [&](int e) { return T[tri_pos(e, e)]; }, [&](int e) { return T[tri_rp(e)]; });
            if (in) {
#pragma unroll
                for (int q = 0; q < 4; ++q) base[(int64_t)(TB * i + 4 * q) * step] = y[q];
            }
#pragma unroll
            for (int j = 1; j < P; ++j) {
                if (i + j >= P) break;
                d4v acc = X[j];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(m[j][ks], -y[ks], acc, 0, 0, 0);
                X[j - 1] = acc;
            }
        }
    };
    if (right) solve(std::true_type{});
    else solve(std::false_type{});
}

// ============================================================== pivoted panel
// Grid barrier of a cooperative launch: bar[0] counts arrivals, bar[1] is
// the generation.  Everything the work-groups exchange is written and read
// with agent-scope accesses (put64, get64), so the arrival only waits for the
// wave's stores (sync_release; the language's fences also wrote back and
// invalidated the L2 once per column).  A bounded wait that expires sets *err
// and every work-group then stops.
__device__ bool grid_sync(unsigned* bar, unsigned nwg, int* err) {
    __shared__ int s_ok;
    // every wave's stores are released before the barrier (the work-group
    // barrier alone does not wait for them)
    sync_release();
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned gen = __hip_atomic_load(&bar[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned old = __hip_atomic_fetch_add(&bar[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int ok = 1;
        if (old == nwg - 1) {
            __hip_atomic_store(&bar[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sync_release();                        // the count is back at zero before the next round can start
            __hip_atomic_store(&bar[1], gen + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            unsigned it = 0;
            while (__hip_atomic_load(&bar[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gen) {
                if (++it > (1u << 24) || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    ok = 0;
                    atomicOr(err, 1);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        sync_acquire();
        s_ok = ok;
    }
    __syncthreads();
    return s_ok != 0;
}

MXP_DEV void put64(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
MXP_DEV double get64(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// What a pivot search goes by: the magnitude, a NaN counting as zero.  A row on
// or below the pivot position then always is a candidate, and ipiv always names
// one of them: the swaps' kernels index with it.  (A NaN compares false with
// everything; held by the lane that the others are compared with it hid them, and
// with one in every work-group there was no candidate at all.)
MXP_DEV double pivot_size(double a) { return fmax(fabs(a), 0.0); }

// the better of two pivot candidates: larger magnitude, smaller row among equals
MXP_DEV void better(double& v, int64_t& r, double ov, int64_t orr) {
    if (ov > v || (ov == v && orr < r)) { v = ov; r = orr; }
}

// (value, row) maximum over the work-group (every thread gets the result)
MXP_DEV void wg_argmax(double& v, int64_t& r, double* redv, int64_t* redr) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) better(v, r, __shfl_xor(v, o, 64), __shfl_xor(r, o, 64));
    if (lane == 0) { redv[wv] = v; redr[wv] = r; }
    __syncthreads();
    v = redv[0];
    r = redr[0];
    for (int q = 1; q < 4; ++q) better(v, r, redv[q], redr[q]);
    __syncthreads();
}

// Panel columns [k, k+nb), rows [k, n): work-group w holds rows
// [k + w rpw, k + (w+1) rpw) in LDS (P[c * rpw + rr]), one row per thread.
// cand: 2 x nwg slots of (|value|, row, nb row values); top: 2 x nb (the
// current pivot position's row); both double-buffered by column parity.
__global__ __launch_bounds__(256) void k_panel64_pp(double* A, int64_t lda, int64_t n, int64_t k, int nb, int rpw,
                                                    int64_t* ipiv, double* cand, double* top, unsigned* bar,
                                                    unsigned long long* info, int* err) {
    extern __shared__ double P[];
    __shared__ double prow[128];
    __shared__ double redv[4];
    __shared__ int64_t redr[4];
    const int t = threadIdx.x;
    const unsigned nwg = gridDim.x;
    const int w = (int)blockIdx.x;
    const int64_t rbase = k + (int64_t)w * rpw;                 // global row of local row 0
    const int nrows = (int)(n - rbase < rpw ? n - rbase : rpw);
    const int slot = nb + 2;
    // after a wait that expired, here or in a panel before: no swaps from column j on
    auto leave = [&](int j) {
        if (w == 0 && t >= j && t < nb) ipiv[k + t] = k + t;
    };
    if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return leave(0);
    for (int c = 0; c < nb; ++c)
        if (t < nrows) P[c * rpw + t] = A[(rbase + t) + (k + c) * lda];
    __syncthreads();
    for (int j = 0; j < nb; ++j) {
        const int par = j & 1;
        const int64_t gtop = k + j;                            // pivot position
        // (a) this work-group's candidate: the largest |P[j][r]| on or below the pivot position
        double bv = -1.0;
        int64_t br = INT64_MAX;
        if (t < nrows && rbase + t >= gtop) {
            bv = pivot_size(P[j * rpw + t]);
            br = rbase + t;
        }
        wg_argmax(bv, br, redv, redr);
        double* my = cand + (int64_t)(par * nwg + w) * slot;
        if (t == 0) {
            put64(&my[0], bv);
            put64(&my[1], bv >= 0.0 ? (double)br : -1.0);
        }
        if (bv >= 0.0 && t < nb) put64(&my[2 + t], P[t * rpw + (int)(br - rbase)]);
        if (gtop >= rbase && gtop < rbase + nrows && t < nb) put64(&top[par * nb + t], P[t * rpw + (int)(gtop - rbase)]);
        // (b) every candidate and the top row are published
        if (!grid_sync(bar, nwg, err)) return leave(j);
        // (c) the winner, the same in every work-group: one candidate per thread
        double cv = -1.0;
        int64_t cr = INT64_MAX;
        if (t < (int)nwg) {
            const double* cq = cand + (int64_t)(par * nwg + t) * slot;
            const double v = get64(&cq[0]);
            const double r = get64(&cq[1]);
            if (r >= 0.0) { cv = v; cr = (int64_t)r; }
        }
        wg_argmax(cv, cr, redv, redr);
        const int64_t p = cr;
        if (w == 0 && t == 0) ipiv[gtop] = p;
        const int wp = (int)((p - k) / rpw);
        if (t < nb) prow[t] = get64(&cand[(int64_t)(par * nwg + wp) * slot + 2 + t]);
        __syncthreads();
        // (d) rows gtop and p trade places
        if (p != gtop) {
            if (p >= rbase && p < rbase + nrows && t < nb) P[t * rpw + (int)(p - rbase)] = get64(&top[par * nb + t]);
            if (gtop >= rbase && gtop < rbase + nrows && t < nb) P[t * rpw + (int)(gtop - rbase)] = prow[t];
        }
        __syncthreads();
        // (e) eliminate below the pivot
        const double piv = prow[j];
        const bool ok = piv != 0.0 && isfinite(piv);
        if (!ok && w == 0 && t == 0) atomicMin(info, (unsigned long long)(gtop + 1));
        if (ok && t < nrows && rbase + t > gtop) {
            const double l = P[j * rpw + t] / piv;
            P[j * rpw + t] = l;
            for (int c = j + 1; c < nb; ++c) P[c * rpw + t] -= l * prow[c];
        }
        __syncthreads();
    }
    for (int c = 0; c < nb; ++c)
        if (t < nrows) A[(rbase + t) + (k + c) * lda] = P[c * rpw + t];
}

// ---------------------------------------------------------------- panels of one work-group
// A panel of up to 8192 rows is factored W = 16, 8 or 4 columns at a time by
// one work-group that holds all its rows in registers (thread t the rows t,
// t + 1024, ...: R = 32 / W of them), so that a column costs one work-group
// barrier instead of a round over the whole device: every wave proposes its
// largest magnitude with that row's W values in LDS, and after the barrier
// every thread has the winner, its row and the row it trades places with.
// Measured (n = 3000, rocprofv3): 29.5 us per 16 columns and 18.4 per 8, 1.9 to
// 2.3 us per column (48 and 26 us with the reductions through LDS and a division
// per row), against 12 us per column with a device-wide barrier (5 us with the
// cheaper one above).  Eight waves with twice the rows each, or the columns in a
// loop that moves them through the same registers, were not faster (20.4 and 42 us
// per 8 columns).  The swaps and the update of the panel's
// other columns follow per W columns (k_panel64_rest).
constexpr int PW_T = 1024;

// the largest of v (no NaN) over the 16 lanes of a row / over the wave, in all of
// its lanes: exchanges by DPP and lane swaps (through LDS, as __shfl does it, the
// reductions were two thirds of a column's time)
MXP_DEV double max64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <int CTRL> MXP_DEV double dpp_max64(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return max64(v, __hiloint2double(hi, lo));
}
MXP_DEV double row_max64(double v) {
    v = dpp_max64<0xB1>(v);                                // quad_perm [1,0,3,2]
    v = dpp_max64<0x4E>(v);                                // quad_perm [2,3,0,1]
    v = dpp_max64<0x141>(v);                               // row_half_mirror
    return dpp_max64<0x140>(v);                            // row_mirror
}
MXP_DEV double wave_max64(double v) {
    v = row_max64(v);
    {
        const auto a = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
        const auto b = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
        v = max64(__hiloint2double((int)b[0], (int)a[0]), __hiloint2double((int)b[1], (int)a[1]));
    }
    const auto a = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
    return max64(__hiloint2double((int)b[0], (int)a[0]), __hiloint2double((int)b[1], (int)a[1]));
}
// the smallest row over the lanes of mask (a wave-uniform result; one lane as a rule)
MXP_DEV int least_row(unsigned long long mask, int row) {
    int r = __builtin_amdgcn_readlane(row, __builtin_ctzll(mask));
    for (mask &= mask - 1; mask; mask &= mask - 1) {
        const int t = __builtin_amdgcn_readlane(row, __builtin_ctzll(mask));
        r = t < r ? t : r;
    }
    return r;
}
// 1 / x to within an ulp or so, finite and normal where it is used; the quotients
// taken with it are corrected by their residual
MXP_DEV double recip64(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

template <int J, int W, int R>
MXP_DEV void panel_step(double (&x)[R][W], int64_t k0, int m, int tid, int lane, int wave, int64_t* ipiv,
                        double (*swave)[17], int (*srow)[16], double (*sval)[16][W], double (*stop)[W], int& bad) {
    if constexpr (J < W) {
        constexpr int par = J & 1;
        // this wave's candidate: the largest |x[.][J]| on or below the pivot
        // position, the smallest row among equals
        double v = -1.0;
        int row = 0x7FFFFFFF;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int r = tid + PW_T * i;
            const double a = pivot_size(x[i][J]);
            if (r >= J && r < m && a > v) { v = a; row = r; }
        }
        const double wm = wave_max64(v);
        const int cr = wm < 0.0 ? 0x7FFFFFFF : least_row(__ballot(v == wm), row);
        if (cr != 0x7FFFFFFF) {
            const int ci = cr / PW_T;
#pragma unroll
            for (int i = 0; i < R; ++i)
                if (i == ci && tid + PW_T * i == cr)
#pragma unroll
                    for (int c = 0; c < W; ++c) sval[par][wave][c] = x[i][c];
        }
        if (lane == 0) { swave[par][wave] = wm; srow[par][wave] = cr; }
        if (tid == J)
#pragma unroll
            for (int c = 0; c < W; ++c) stop[par][c] = x[0][c];
        __syncthreads();
        // the winner, the same in every thread
        const double cv = swave[par][lane & 15];
        const int wr = srow[par][lane & 15];
        const int p = least_row(__ballot(cv == row_max64(cv)) & 0xFFFFull, wr);
        const int pw = (p % PW_T) / 64;
        double pr[W];
#pragma unroll
        for (int c = 0; c < W; ++c) pr[c] = sval[par][pw][c];
        if (tid == 0) ipiv[k0 + J] = k0 + p;
        if (p != J) {
            // rows J and p trade places
            const int pi = p / PW_T;
            if (wave == pw) {
#pragma unroll
                for (int i = 0; i < R; ++i)
                    if (i == pi && tid + PW_T * i == p)
#pragma unroll
                        for (int c = 0; c < W; ++c) x[i][c] = stop[par][c];
            }
            if (tid == J)
#pragma unroll
                for (int c = 0; c < W; ++c) x[0][c] = pr[c];
        }
        const double piv = pr[J];
        if (__builtin_amdgcn_readfirstlane(piv != 0.0 && isfinite(piv))) {
            // the quotient as a product with the reciprocal and one residual
            // correction (a true quotient where the reciprocal leaves the range)
            double l[R];
            const double rp = recip64(piv);
            if (__builtin_amdgcn_readfirstlane(fabs(rp) >= 0x1p-1000 && fabs(rp) <= 0x1p1000)) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    l[i] = x[i][J] * rp;
                    l[i] = fma(fma(-piv, l[i], x[i][J]), rp, l[i]);
                }
            } else {
#pragma unroll 1
                for (int i = 0; i < R; ++i) {
                    double a = x[0][J];
#pragma unroll
                    for (int k = 1; k < R; ++k) a = k == i ? x[k][J] : a;
                    a = a / piv;
#pragma unroll
                    for (int k = 0; k < R; ++k) l[k] = k == i ? a : l[k];
                }
            }
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const bool below = i > 0 || tid > J;
                x[i][J] = below ? l[i] : x[i][J];
                l[i] = below ? l[i] : 0.0;
#pragma unroll
                for (int c = J + 1; c < W; ++c) x[i][c] = fma(-l[i], pr[c], x[i][c]);
            }
        } else if (bad < 0) {
            bad = J;
        }
        panel_step<J + 1, W, R>(x, k0, m, tid, lane, wave, ipiv, swave, srow, sval, stop, bad);
    }
}

// columns [k0, k0 + w) (w <= W), rows [k0, n): at most 1024 R rows
template <int W, int R>
__global__ __launch_bounds__(PW_T) void k_panel64_wg(double* A, int64_t lda, int64_t n, int64_t k0, int w,
                                                     int64_t* ipiv, unsigned long long* info) {
    __shared__ double swave[2][17];
    __shared__ int srow[2][16];
    __shared__ double sval[2][16][W];
    __shared__ double stop[2][W];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = (int)(n - k0);
    double x[R][W];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int c = 0; c < W; ++c) {
            const int r = tid + PW_T * i;
            // past the edges zeros (the columns past w, those of the matrix's last
            // sub-panel only, take no part in its elimination)
            const bool in = r < m && c < w;
            const double v = A[in ? (k0 + r) + (k0 + c) * lda : k0 + k0 * lda];
            x[i][c] = in ? v : 0.0;
        }
    int bad = -1;
    if (w == W) {
        panel_step<0, W, R>(x, k0, m, tid, lane, wave, ipiv, swave, srow, sval, stop, bad);
    } else {
        // the last columns of the matrix: m = w < W rows, one column at a time
        // by the same rule in LDS
        if (tid < m)
#pragma unroll
            for (int c = 0; c < W; ++c) sval[0][tid][c] = x[0][c];
        __syncthreads();
        if (tid == 0) {
            for (int j = 0; j < w; ++j) {
                int p = j;
                double best = -1.0;
                for (int r = j; r < m; ++r) {
                    const double a = pivot_size(sval[0][r][j]);
                    if (a > best) { best = a; p = r; }
                }
                ipiv[k0 + j] = k0 + p;
                for (int c = 0; c < w; ++c) {
                    const double t = sval[0][j][c];
                    sval[0][j][c] = sval[0][p][c];
                    sval[0][p][c] = t;
                }
                const double piv = sval[0][j][j];
                if (piv == 0.0 || !isfinite(piv)) {
                    if (bad < 0) bad = j;
                    continue;
                }
                for (int r = j + 1; r < m; ++r) {
                    const double l = sval[0][r][j] / piv;
                    sval[0][r][j] = l;
                    for (int c = j + 1; c < w; ++c) sval[0][r][c] = fma(-l, sval[0][j][c], sval[0][r][c]);
                }
            }
        }
        __syncthreads();
        if (tid < m)
#pragma unroll
            for (int c = 0; c < W; ++c) x[0][c] = sval[0][tid][c];
    }
    if (bad >= 0 && tid == 0) atomicMin(info, (unsigned long long)(k0 + bad + 1));
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int c = 0; c < W; ++c) {
            const int r = tid + PW_T * i;
            if (r < m && c < w) A[(k0 + r) + (k0 + c) * lda] = x[i][c];
        }
}

// The net row exchange of the swaps ipiv[k0 .. k0 + w) (w <= 128) as a
// gather: slot s < w is row k0 + s, slot w + j row ipiv[k0 + j] where that
// lies below and no earlier swap names it (else unused: row -1); src[s]: the
// slot whose row's content ends up in slot s.  By one work-group.
MXP_DEV void swap_gather(const int64_t* ipiv, int64_t k0, int w, int* row, int* src, int* slot) {
    const int tid = threadIdx.x;
    if (tid < w) {
        const int p = (int)(ipiv[k0 + tid] - k0);
        row[tid] = tid;
        row[w + tid] = p;
    }
    __syncthreads();
    if (tid < w) {
        const int p = row[w + tid];
        int s = p < w ? p : w + tid;
        if (p >= w)
            for (int j = 0; j < tid; ++j)
                if (row[w + j] == p) { s = w + j; break; }
        slot[tid] = s;
        src[tid] = tid;
        src[w + tid] = w + tid;
    }
    __syncthreads();
    if (tid < w && slot[tid] != w + tid) row[w + tid] = -1;
    if (tid == 0)
        for (int j = 0; j < w; ++j) {
            const int s = slot[j], a = src[j];
            src[j] = src[s];
            src[s] = a;
        }
    __syncthreads();
}

// The panel [k, k + nb) after its columns [k0, k0 + W): a work-group takes CW
// of the panel's other columns, applies the W swaps to them, and right of
// the factored columns forms the W rows of U (unit-lower substitution, one
// column per thread) and updates the rows below, one row per thread.
constexpr int PR_CW = 4;
template <int W>
__global__ __launch_bounds__(512) void k_panel64_rest(double* A, int64_t lda, int64_t n, int64_t k, int64_t k0,
                                                      int64_t cend, const int64_t* __restrict__ ipiv, int lgroups) {
    __shared__ int row[2 * W], src[2 * W], slot[W];
    __shared__ double val[2 * W][PR_CW], sL[W][W], su[PR_CW][W];
    const int tid = threadIdx.x;
    const bool left = (int)blockIdx.x < lgroups;
    const int64_t c0 = left ? k + (int64_t)blockIdx.x * PR_CW : k0 + W + (int64_t)(blockIdx.x - lgroups) * PR_CW;
    const int64_t ce = left ? k0 : cend;
    const int nc = (int)(ce - c0 < PR_CW ? ce - c0 : PR_CW);
    if (tid < W * W) sL[tid / W][tid % W] = A[(k0 + tid % W) + (k0 + tid / W) * lda];   // sL[c][r]
    swap_gather(ipiv, k0, W, row, src, slot);
    if (tid < 2 * W * PR_CW) {
        const int s = tid / PR_CW, c = tid % PR_CW;
        val[s][c] = row[s] >= 0 && c < nc ? A[(k0 + row[s]) + (c0 + c) * lda] : 0.0;
    }
    __syncthreads();
    if (tid < 2 * W * PR_CW) {
        const int s = tid / PR_CW, c = tid % PR_CW;
        if (c < nc && row[s] >= 0 && (left || s >= W)) A[(k0 + row[s]) + (c0 + c) * lda] = val[src[s]][c];
    }
    if (left) return;
    if (tid < nc) {
        double u[W];
#pragma unroll
        for (int j = 0; j < W; ++j) u[j] = val[src[j]][tid];
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int r = j + 1; r < W; ++r) u[r] = fma(-sL[j][r], u[j], u[r]);
#pragma unroll
        for (int j = 0; j < W; ++j) {
            su[tid][j] = u[j];
            A[(k0 + j) + (c0 + tid) * lda] = u[j];
        }
    }
    __syncthreads();
    for (int64_t r = k0 + W + tid; r < n; r += 512) {
        double l[W], x[PR_CW];
#pragma unroll
        for (int j = 0; j < W; ++j) l[j] = A[r + (k0 + j) * lda];
#pragma unroll
        for (int c = 0; c < PR_CW; ++c) x[c] = A[r + (c0 + (c < nc ? c : 0)) * lda];
#pragma unroll
        for (int c = 0; c < PR_CW; ++c) {
#pragma unroll
            for (int j = 0; j < W; ++j) x[c] = fma(-l[j], su[c < nc ? c : 0][j], x[c]);
        }
#pragma unroll
        for (int c = 0; c < PR_CW; ++c)
            if (c < nc) A[r + (c0 + c) * lda] = x[c];
    }
}

// the swaps ipiv[k0 .. k0 + w) (w < 16) in order, one thread per column of
// [c_begin, c_end): the few columns left of the matrix's last sub-panel
__global__ __launch_bounds__(64) void k_swap_cols64(double* A, int64_t lda, const int64_t* __restrict__ ipiv,
                                                    int64_t k0, int w, int64_t c_begin, int64_t c_end) {
    const int64_t c = c_begin + (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (c >= c_end) return;
    double* col = A + c * lda;
    for (int j = 0; j < w; ++j) {
        const int64_t p = ipiv[k0 + j];
        if (p != k0 + j) {
            const double x = col[k0 + j];
            col[k0 + j] = col[p];
            col[p] = x;
        }
    }
}

// Row swaps ipiv[k .. k+nb) applied to the columns outside the panel (left of
// it: [0, k); right: [k + nb, n)): every work-group forms the net exchange of
// at most 2 nb rows once and moves 16 columns through LDS, all loads in flight
// at once (swap after swap in every column was a chain of nb dependent
// round trips to memory).
constexpr int LSW_C = 16;
__global__ __launch_bounds__(256) void k_laswp64(double* A, int64_t lda, int64_t n, const int64_t* __restrict__ ipiv,
                                                 int64_t k, int nb, int lgroups) {
    __shared__ int row[256], src[256], slot[128];
    __shared__ double val[256][LSW_C + 1];
    const bool left = (int)blockIdx.x < lgroups;
    const int64_t c0 = left ? (int64_t)blockIdx.x * LSW_C : k + nb + (int64_t)(blockIdx.x - lgroups) * LSW_C;
    const int64_t ce = left ? k : n;
    swap_gather(ipiv, k, nb, row, src, slot);
    const int s = threadIdx.x;
    const bool live = s < 2 * nb && row[s] >= 0;
    double* base = A + k + (live ? row[s] : 0);
    double v[LSW_C];
#pragma unroll
    for (int c = 0; c < LSW_C; ++c) v[c] = base[(c0 + c < ce ? c0 + c : c0) * lda];
#pragma unroll
    for (int c = 0; c < LSW_C; ++c) val[s][c] = v[c];
    __syncthreads();
    if (live && src[s] != s)
#pragma unroll
        for (int c = 0; c < LSW_C; ++c)
            if (c0 + c < ce) base[(c0 + c) * lda] = val[src[s]][c];
}

// ============================================================== solve
// x <- P x, then unit-lower forward and upper backward substitution over
// blocks of 128 rows, one launch per block: every work-group subtracts the
// previous block's contribution from its 128 rows, and the one that holds
// the next block solves it in the same launch.  Launches and the solve's
// chain bound it (14 to 16 us per block at n = 8192); blocks of 64 with the
// triangle solved by one lane per right-hand side from memory took 80 us.

// The n swaps in order, one work-group per right-hand side: x in LDS when it fits
// (lds_n = n).  Sixteen waves form the net exchange of 64 swaps each -- at most 128
// slots: slot j < 64 is row k0 + j, slot 64 + j row ipiv[k0 + j] where that lies
// outside and no earlier swap names it -- then one wave moves the values, 64 swaps
// at a time.  (Swap after swap on the values, each a round trip to LDS: 316 us at
// n = 3000 against 46.)
constexpr int AP_T = 1024, AP_W = AP_T / 64;
__global__ __launch_bounds__(AP_T) void k_apply_pivots(double* x, int64_t ldx, const int64_t* __restrict__ ipiv,
                                                       int64_t n, int lds_n) {
    extern __shared__ __attribute__((aligned(16))) double gsm[];
    __shared__ int row[AP_W][128];
    __shared__ int src[AP_W][128];
    double* g = x + (int64_t)blockIdx.x * ldx;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < lds_n; i += AP_T) gsm[i] = g[i];
    double* const v = lds_n ? gsm : g;
    for (int64_t r0 = 0; r0 < n; r0 += 64 * AP_W) {
        const int64_t k0 = r0 + 64 * wave;
        const int m = (int)(n - k0 < 64 ? n - k0 : 64);
        if (m > 0) {
            const int p = lane < m ? (int)ipiv[k0 + lane] : (int)k0 + lane;
            int slot = p - (int)k0;
            if (slot >= 64) {
                slot = 64 + lane;
            }
#pragma unroll 8
            for (int j = 62; j >= 0; --j)                 // the first swap that names the row
                if (slot >= 64 && j < lane && __builtin_amdgcn_readlane(p, j) == p) slot = 64 + j;
            row[wave][lane] = lane < m ? (int)k0 + lane : -1;
            row[wave][64 + lane] = lane < m && slot == 64 + lane ? p : -1;
            src[wave][lane] = lane;
            src[wave][64 + lane] = 64 + lane;
            __builtin_amdgcn_wave_barrier();
            for (int j = 0; j < m; ++j) {
                const int s = __builtin_amdgcn_readlane(slot, j);
                if (lane == 0) {
                    const int a = src[wave][j], b = src[wave][s];
                    src[wave][j] = b;
                    src[wave][s] = a;
                }
            }
        }
        __syncthreads();
        if (wave == 0) {
            for (int c = 0; c < AP_W && r0 + 64 * c < n; ++c) {
                const int ra = row[c][lane], rb = row[c][64 + lane];
                const double a = ra >= 0 ? v[row[c][src[c][lane]]] : 0.0;
                const double b = rb >= 0 ? v[row[c][src[c][64 + lane]]] : 0.0;
                __threadfence_block();
                __builtin_amdgcn_wave_barrier();
                if (ra >= 0) v[ra] = a;
                if (rb >= 0) v[rb] = b;
                __threadfence_block();
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
    }
    for (int i = tid; i < lds_n; i += AP_T) g[i] = gsm[i];
}

constexpr int SVB = 128;     // rows of a block step

MXP_DEV double rl64(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// One wave solves a 64 x 64 triangle (its first m rows), row r in lane r: d[s] =
// T[r][s], zero outside the strict triangle, dg its diagonal (1 for the unit-
// lower); NR right-hand sides side by side.  The quotient by the diagonal is the
// product with its reciprocal and one residual correction.  Where any result is
// not finite -- a zero, subnormal or infinite diagonal entry, an infinite entry,
// an overflow -- that right-hand side is solved again with true quotients and only
// the rows that a solved one reaches (T[r][s] again from memory, at T + s ld).
template <bool LOWER, int NR>
MXP_DEV void tri_solve64(double (&x)[NR], const double (&d)[64], double dg, const double* T, int64_t ld, int m) {
    const int lane = threadIdx.x & 63;
    const double ri = LOWER ? 1.0 : 1.0 / dg;
    double x0[NR], y[NR];
    bool fin[NR], all = true;
#pragma unroll
    for (int r = 0; r < NR; ++r) x0[r] = x[r];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int s0 = LOWER ? 16 * c : 48 - 16 * c;
        if (s0 >= m) continue;                           // (wave-uniform)
#pragma unroll
        for (int s2 = 0; s2 < 16; ++s2) {
            const int s = LOWER ? s0 + s2 : s0 + 15 - s2;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                double q = x[r];
                if (!LOWER) {
                    q = x[r] * ri;
                    q = fma(fma(-dg, q, x[r]), ri, q);
                }
                x[r] = fma(-d[s], rl64(q, s), x[r]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (!LOWER) {
            const double q = x[r] * ri;
            x[r] = fma(fma(-dg, q, x[r]), ri, q);
        }
        fin[r] = __all(isfinite(x[r]));
        all = all && fin[r];
    }
    if (all) return;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        y[r] = x[r];
        x[r] = x0[r];
    }
#pragma unroll 1
    for (int s2 = 0; s2 < m; ++s2) {
        const int s = LOWER ? s2 : m - 1 - s2;
        const bool reach = lane < m && (LOWER ? s < lane : s > lane);
        const double t = T[reach ? s * ld : 0];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const double q = LOWER ? x[r] : x[r] / dg;
            const double b = rl64(q, s);
            if (reach) x[r] -= t * b;
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) x[r] = fin[r] ? y[r] : LOWER ? x[r] : x[r] / dg;
}

// Block step: the block [b0, b0 + kb) and the rows beyond it (above it for
// the upper triangle) lose A[., p0 : p0 + pkb] x[p0 : p0 + pkb]; work-group 0
// then solves the block's triangle.  512 threads: 128 rows x 4 column groups; row
// y of the grid the right-hand sides NR y .. (one launch for all of them: one
// chain of launches per four took 289 us at n = 16 with 64 right-hand sides).
template <bool LOWER, int NR>
__global__ __launch_bounds__(512) void k_trsv64_step(const double* __restrict__ A, int64_t lda, int64_t n, int64_t b0,
                                                     int kb, int64_t p0, int pkb, double* xs, int64_t ldx, int nrhs) {
    __shared__ double sx[NR][SVB];
    __shared__ double part[NR][4][SVB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = tid & 127, cg = tid >> 7;
    const bool solver = blockIdx.x == 0;
    // right-hand side r; past the last one it is read in its place, and not written
    const int nr = nrhs - NR * (int)blockIdx.y;
    xs += (int64_t)NR * blockIdx.y * ldx;
    auto x = [&](int r) { return xs + (r < nr ? r : nr - 1) * ldx; };
    // first row of this work-group, end of its rows
    const int64_t r0 = solver ? b0 : LOWER ? b0 + kb + (int64_t)(blockIdx.x - 1) * SVB
                                           : (int64_t)(blockIdx.x - 1) * SVB;
    const int64_t rend = solver ? b0 + kb : LOWER ? n : b0;
    const int64_t i = r0 + row < rend ? r0 + row : rend - 1;
    const bool in = r0 + row < rend;
    // the triangle's rows of the solver's waves: wave 0 the first 64 rows,
    // wave 1 the rest (d), waves 2-5 the block between them (16 columns each)
    double d[64], dg = 1.0;
    const int h0 = kb < 64 ? kb : 64, h1 = kb - h0;         // rows of the two halves
    if (solver && wave < 2) {
        const int64_t o = b0 + 64 * wave;
        const int m = wave ? h1 : h0;
#pragma unroll
        for (int c = 0; c < 64; ++c) {
            const bool strict = lane < m && c < m && (LOWER ? c < lane : c > lane);
            const double v = A[strict ? (o + lane) + (o + c) * lda : b0 + b0 * lda];
            d[c] = strict ? v : 0.0;
        }
        if (!LOWER && lane < m) dg = A[(o + lane) + (o + lane) * lda];
    }
    if (pkb > 0) {
        for (int e = tid; e < NR * SVB; e += 512) {
            const int r = e / SVB, c = e % SVB;
            sx[r][c] = c < pkb ? x(r)[p0 + c] : 0.0;
        }
        __syncthreads();
        double acc[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) acc[r] = 0.0;
        const double* ap = A + i + p0 * lda;
#pragma unroll
        for (int c0 = 0; c0 < 32; c0 += 16) {
            double a[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const int cc = 32 * cg + c0 + c;
                a[c] = ap[(int64_t)(cc < pkb ? cc : 0) * lda];
            }
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const int cc = 32 * cg + c0 + c;
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (cc < pkb) acc[r] = fma(a[c], sx[r][cc], acc[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) part[r][cg][row] = acc[r];
        __syncthreads();
    }
    if (cg == 0) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            double v = x(r)[i];
            if (pkb > 0) v -= (part[r][0][row] + part[r][1][row]) + (part[r][2][row] + part[r][3][row]);
            if (solver) sx[r][row] = v;
            else if (in && pkb > 0 && r < nr) x(r)[i] = v;
        }
    }
    if (!solver) return;
    __syncthreads();
    // the half solved first (rows 0-63 of L, 64-127 of U), its contribution to
    // the other half, the other half
    const int first = LOWER ? 0 : 1;
    auto half = [&](int w, int m) {
        if (wave == w && m > 0) {
            double v[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) v[r] = lane < m ? sx[r][64 * w + lane] : 0.0;
            const int64_t o = b0 + 64 * w;
            tri_solve64<LOWER, NR>(v, d, dg, A + o + (lane < m ? lane : 0) + o * lda, lda, m);
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (lane < m) {
                    sx[r][64 * w + lane] = v[r];
                    if (r < nr) x(r)[b0 + 64 * w + lane] = v[r];
                }
        }
    };
    half(first, first ? h1 : h0);
    if (h1 > 0) {
        // rows of the half still to be solved, 16 columns of the solved half per wave
        const int mo = first ? h0 : h1, ms = first ? h1 : h0;
        double a[16];
        if (wave >= 2 && wave < 6) {
            const int64_t ro = b0 + (first ? 0 : 64) + (lane < mo ? lane : 0);
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const int cc = 16 * (wave - 2) + c;
                a[c] = A[ro + (b0 + 64 * first + (cc < ms ? cc : 0)) * lda];
            }
        }
        __syncthreads();
        if (wave >= 2 && wave < 6) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                double t = 0.0;
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    const int cc = 16 * (wave - 2) + c;
                    if (cc < ms) t = fma(a[c], sx[r][64 * first + cc], t);
                }
                part[r][wave - 2][lane] = t;
            }
        }
        __syncthreads();
        if (wave == 1 - first)
#pragma unroll
            for (int r = 0; r < NR; ++r)
                sx[r][64 * (1 - first) + lane] -=
                    (part[r][0][lane] + part[r][1][lane]) + (part[r][2][lane] + part[r][3][lane]);
    }
    half(1 - first, first ? h0 : h1);
}

// ============================================================== drivers
int lu64_block(int64_t n) {
    // the pivoted panel holds ceil(m / 256) rows x nb per work-group in at most 128 KB of LDS
    const int64_t rpw = (n + 255) / 256;
    return rpw <= 128 ? 128 : 64;
}

// candidates and top rows of the pivoted panel, its barrier and error words
static size_t lu64_panel_bytes(int64_t n) {
    const int nb = lu64_block(n);
    return ((size_t)2 * 256 * (nb + 2) * 8 + (size_t)2 * nb * 8 + 256 + 63) / 64 * 64;
}

size_t lu64_work_bytes(int64_t n) { return lu64_panel_bytes(n) + (size_t)2 * TRI_MAX * 8; }

// the pivoted panel [k, k + kb) by one work-group, W columns at a time
template <int W>
static void panel64_cols(double* A, int64_t lda, int64_t n, int64_t k, int kb, int64_t* ipiv,
                         unsigned long long* info, hipStream_t s) {
    for (int64_t k0 = k; k0 < k + kb; k0 += W) {
        const int w = (int)(k + kb - k0 < W ? k + kb - k0 : W);
        k_panel64_wg<W, 32 / W><<<1, PW_T, 0, s>>>(A, lda, n, k0, w, ipiv, info);
        if (w < W) {
            // the last columns of the matrix: only the swaps are left
            const int64_t left = k0 - k;
            if (left) k_swap_cols64<<<(unsigned)((left + 63) / 64), 64, 0, s>>>(A, lda, ipiv, k0, w, k, k0);
            continue;
        }
        const int lg = (int)((k0 - k + PR_CW - 1) / PR_CW), rg = (int)((k + kb - k0 - W + PR_CW - 1) / PR_CW);
        if (lg + rg) k_panel64_rest<W><<<lg + rg, 512, 0, s>>>(A, lda, n, k, k0, k + kb, ipiv, lg);
    }
}
static void panel64_wg(double* A, int64_t lda, int64_t n, int64_t k, int kb, int64_t* ipiv, unsigned long long* info,
                       hipStream_t s) {
    const int64_t m = n - k;
    if (m <= 2 * PW_T) panel64_cols<16>(A, lda, n, k, kb, ipiv, info, s);
    else if (m <= 4 * PW_T) panel64_cols<8>(A, lda, n, k, kb, ipiv, info, s);
    else panel64_cols<4>(A, lda, n, k, kb, ipiv, info, s);
}

hipError_t lu64_factor(int64_t n, double* A, int64_t lda, int64_t* ipiv, void* work, unsigned long long* info_dev,
                       int use_rocblas, hipStream_t s) {
    const int nb = lu64_block(n);
    static const hipError_t attr = []() {
        hipError_t e;
        if ((e = hipFuncSetAttribute((const void*)k_diag64, hipFuncAttributeMaxDynamicSharedMemorySize, (int)D64_LDS)))
            return e;
        return hipFuncSetAttribute((const void*)k_panel64_pp, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
    }();
    if (attr) return attr;
    char* wb = (char*)work;
    double* cand = (double*)wb;
    double* top = cand + 2 * 256 * (nb + 2);
    unsigned* bar = (unsigned*)(top + 2 * nb);
    int* err = (int*)(bar + 2);
    double* PL = (double*)(wb + lu64_panel_bytes(n));
    double* PU = PL + TRI_MAX;
    hipError_t e;
    if ((e = fill_u64(info_dev, 1, ~0ull, s))) return e;
    if ((e = fill_u64(bar, 2, 0ull, s))) return e;   // bar[0..1] and err
    // Without pivoting, while at least GROUP_MIN columns are left, blocks are taken
    // four at a time: inside such a group an update covers what the group still
    // factors, its columns and its rows, and the rest follows once per group with
    // K = 512 (one pass over C instead of four: the update alone runs at 42 TFLOP/s
    // with K = 128, 52 with 256, 63 with 512).  Factorisation 13.63 -> 12.09 ms at n = 8192, 9.88
    // -> 9.20 at 6500, 5.66 -> 5.56 at 5000; with groups down to 2048 columns 3.02 ->
    // 3.06 at n = 3000, down to 6144 only 12.39 at 8192.  (Pivoting brings rows of
    // the rest, which lag, into the group.)
    constexpr int64_t GROUP_MIN = 4096;
    int64_t g0 = 0, ge = 0;                              // the group's columns [g0, ge)
    for (int64_t k = 0; k < n; k += nb) {
        if (k == ge) {
            g0 = k;
            ge = k + (nb == G64_T && !ipiv && n - k >= GROUP_MIN ? 4 * nb : nb);
        }
        const int kb = (int)(n - k < nb ? n - k : nb);
        const int64_t m = n - k;
        if (ipiv) {
            if (m <= 8 * PW_T) {
                panel64_wg(A, lda, n, k, kb, ipiv, info_dev, s);
            } else {
                const int rpw = (int)(m <= 256 * 64 ? 64 : (m + 255) / 256);
                const unsigned nwg = (unsigned)((m + rpw - 1) / rpw);
                const size_t lds = (size_t)rpw * kb * 8;
                double* Ap = A;
                int64_t nn = n, kk = k;
                int kbv = kb, rpwv = rpw;
                void* args[] = {&Ap, (void*)&lda, &nn, &kk, &kbv, &rpwv, &ipiv, &cand, &top, &bar, &info_dev, &err};
                if ((e = hipLaunchCooperativeKernel((const void*)k_panel64_pp, dim3(nwg), dim3(256), args,
                                                    (unsigned)lds, s)))
                    return e;
            }
            // the swaps, left and right of the panel
            const int lg = (int)((k + LSW_C - 1) / LSW_C);
            const int rg = k + kb < n ? (int)((n - k - kb + LSW_C - 1) / LSW_C) : 0;
            if (lg + rg) k_laswp64<<<lg + rg, 256, 0, s>>>(A, lda, n, ipiv, k, kb, lg);
            if (k + kb < n) k_pack64<<<1, 512, 0, s>>>(A, lda, k, kb, PL);
        } else {
            k_diag64<<<1, 512, D64_LDS, s>>>(A, lda, k, kb, PL, PU, info_dev);
        }
        if ((e = hipGetLastError())) return e;
        if (k + kb < n) {
            // every block but the last is a full one (kb = nb)
            const int wg = (int)((n - k - kb + 63) / 64), wgr = ipiv ? 0 : wg;
            if (kb == 128) k_trsm64<8><<<wg + wgr, 256, 0, s>>>(A, lda, n, k, wgr, PL, PU);
            else k_trsm64<4><<<wg + wgr, 256, 0, s>>>(A, lda, n, k, wgr, PL, PU);
            if ((e = hipGetLastError())) return e;
            const int64_t k1 = k + kb;
            double* C = A + k1 + k1 * lda;
            if (use_rocblas)
                e = gemm64_rocblas(C, lda, A + k1 + k * lda, lda, A + k + k1 * lda, lda, m - kb, m - kb, kb, s);
            else if (k1 < ge)
                e = gemm64_part(C, lda, A + k1 + k * lda, lda, A + k + k1 * lda, lda, m - kb, m - kb, kb,
                                ge < n ? ge - k1 : -1, s);
            else
                e = gemm64(C, lda, A + k1 + g0 * lda, lda, A + g0 + k1 * lda, lda, m - kb, m - kb, (int)(k1 - g0), s);
            if (e) return e;
        }
    }
    return hipSuccess;
}

int* lu64_err_word(void* work, int64_t n) {
    const int nb = lu64_block(n);
    double* cand = (double*)work;
    double* top = cand + 2 * 256 * (nb + 2);
    return (int*)((unsigned*)(top + 2 * nb) + 2);
}

template <int NR>
static void lu64_solve_nr(int64_t n, const double* A, int64_t lda, double* X, int64_t ldx, int nr, hipStream_t s) {
    const int64_t last = (n - 1) / SVB * SVB;
    // work-groups of a step with the given rows beside the block
    auto wgs = [&](int64_t rows) {
        return dim3((unsigned)(1 + (rows + SVB - 1) / SVB), (unsigned)((nr + NR - 1) / NR));
    };
    for (int64_t b0 = 0; b0 < n; b0 += SVB) {
        const int kb = (int)(n - b0 < SVB ? n - b0 : SVB);
        k_trsv64_step<true, NR><<<wgs(b0 ? n - b0 - kb : 0), 512, 0, s>>>(A, lda, n, b0, kb, b0 - SVB, b0 ? SVB : 0, X,
                                                                          ldx, nr);
    }
    for (int64_t b0 = last; b0 >= 0; b0 -= SVB) {
        const int kb = (int)(n - b0 < SVB ? n - b0 : SVB);
        const int pkb = b0 == last ? 0 : (int)(n - b0 - SVB < SVB ? n - b0 - SVB : SVB);
        k_trsv64_step<false, NR><<<wgs(pkb ? b0 : 0), 512, 0, s>>>(A, lda, n, b0, kb, b0 + SVB, pkb, X, ldx, nr);
    }
}

hipError_t lu64_solve(int64_t n, const double* A, int64_t lda, const int64_t* ipiv, double* X, int64_t ldx, int nr,
                      hipStream_t s) {
    hipError_t e;
    if (ipiv) {
        constexpr int LDS_N = 18000;                  // of 160 KB of LDS, 16 for the exchanges
        static const hipError_t attr = hipFuncSetAttribute((const void*)k_apply_pivots,
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS_N * 8);
        if (attr) return attr;
        const int lds_n = n <= LDS_N ? (int)n : 0;
        k_apply_pivots<<<nr, AP_T, (size_t)lds_n * 8, s>>>(X, ldx, ipiv, n, lds_n);
        if ((e = hipGetLastError())) return e;
    }
    if (nr == 1) lu64_solve_nr<1>(n, A, lda, X, ldx, nr, s);
    else if (nr == 2) lu64_solve_nr<2>(n, A, lda, X, ldx, nr, s);
    else lu64_solve_nr<4>(n, A, lda, X, ldx, nr, s);
    return hipGetLastError();
}

}  // namespace mxp
