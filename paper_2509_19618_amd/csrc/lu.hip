// lu.hip -- right-looking blocked LU without pivoting in mixed precision
// (paper: "Algorithmic Framework" and its Figure 1: the panel and the
// triangular solves in 32-bit, the Schur complement A22 - A21 A11^-1 A12 in
// 16-bit (or 8-bit) inputs with 32-bit accumulation; balancing/scaling of
// the input allowed).
//
// Per block step k (block size nb):
//   1. diagonal block A11 -> FP32, LU in FP32 by up to 32 cooperating
//      work-groups over 32x32 tiles (diag.hip); inverses of the 64x64
//      diagonal sub-blocks of L11 and U11 kept;
//   2. L21 = A21 U11^-1 and U12 = L11^-1 A12 by blocked substitution in
//      FP32, one workgroup per 32-row (32-column) strip, fused with the
//      rounding to the update format under a power-of-two strip scale (the
//      strips beyond the next block's, while they are many, as products with
//      the block's inverses: panel.hip);
//   3. A22 <- A22 - L21 U12 on the matrix cores (MFMA), FP32 accumulation,
//      result rounded to the storage format.
#include <mutex>
#include <vector>

#include "common.hpp"
#include "kernels.hpp"
#include "prof.hpp"

namespace mxp {

int dtype_bytes(int dt) {
    switch (dt) {
    case F64: return 8;
    case F32: return 4;
    case F16: case BF16: return 2;
    case F8: return 1;
    default: return 0;
    }
}

__host__ __device__ static inline int64_t rup(int64_t a, int64_t b) { return (a + b - 1) / b * b; }
static inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

AuxLayout aux_layout(int64_t n, int64_t nb) {
    AuxLayout L;
    int64_t nblk = (n + nb - 1) / nb;
    size_t off = 0;
    L.T = off; off = al256(off + (size_t)nblk * nb * nb * 4);
    L.Trm = off; off = al256(off + (size_t)nblk * nb * nb * 4);
    L.linv = off; off = al256(off + (size_t)nblk * nb * 64 * 4);
    L.uinv = off; off = al256(off + (size_t)nblk * nb * 64 * 4);
    L.lsc = off; off = al256(off + (size_t)nblk * ((n + 31) / 32) * 4);
    L.rowscale = off; off = al256(off + (size_t)n * 8);
    const int64_t D = prec_block(nb), ngrp = (n + D - 1) / D;
    L.linv_full = off; off = al256(off + (size_t)ngrp * D * D * 4);
    L.uinv_full = off; off = al256(off + (size_t)ngrp * D * D * 4);
    L.total = off;
    return L;
}

// operand rows per set: the trailing size padded to 256, plus 256 so that
// the sub-range updates of the look-ahead (starting nb rows in) stay inside
int64_t operand_rows(int64_t n) { return rup(n, 256) + 256; }

WorkLayout work_layout(int64_t n, int64_t nb, int update) {
    WorkLayout W;
    int64_t rows = operand_rows(n);
    size_t eb = (size_t)dtype_bytes(update);
    size_t off = 0;
    W.Lq = off; off = al256(off + 4 * (size_t)rows * nb * eb);     // four sets: two pairs of steps
    W.Uq = off; off = al256(off + 4 * (size_t)rows * nb * eb);
    W.inv_sa = off; off = al256(off + 4 * (size_t)(rows / 32) * 4);
    W.inv_sb = off; off = al256(off + 4 * (size_t)(rows / 32) * 4);
    W.info = off; off = al256(off + 8);
    W.dsync = off; off = al256(off + (size_t)((n + nb - 1) / nb) * diag_sync_words(nb) * 4);
    W.binv = off; off = al256(off + (size_t)2 * 3 * nb * nb * 2);
    W.binv_sc = off; off = al256(off + (size_t)2 * nb * 4);
    W.total = off;
    return W;
}

// ============================================================== scaling
// Row equilibration: S_ii = 2^(t - p) with 2^p the power of two nearest the
// diagonal (the largest entry of its row), so the diagonal lands near 2^t;
// A <- S A in place, exactly.  t = 14 for FP16 storage, whose normal range
// ends below 2^-14: with the diagonal near 1 the off-diagonal entries (about
// n/4 times smaller) would be stored as subnormals, with the diagonal near
// 2^14 they stay normal; t = 0 for BF16 and FP32 storage.
template <int ST>
__global__ __launch_bounds__(256) void k_row_scale(int64_t n, typename Store<ST>::T* A, int64_t lda,
                                                   const double* __restrict__ diag, double* __restrict__ rowscale,
                                                   int target) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    int e;
    double f = frexp(diag[i], &e);        // diag = f 2^e, f in [0.5, 1)
    int p = (f < 0.70710678118654752) ? e - 1 : e;
    double S = ldexp(1.0, target - p);
    if (blockIdx.y == 0) rowscale[i] = S;
    float Sf = (float)S;
    int64_t j0 = (int64_t)blockIdx.y * 64;
    int64_t j1 = j0 + 64 < n ? j0 + 64 : n;
    for (int64_t j = j0; j < j1; ++j) {
        float v = Store<ST>::load(A, i + j * lda);
        A[i + j * lda] = Store<ST>::from_f32(v * Sf);
    }
}

__global__ void k_fill_f64(double* p, int64_t n, double v) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t row_equilibrate(const FactorPlan& p, const double* diag, hipStream_t s) {
    dim3 g((unsigned)((p.n + 255) / 256), (unsigned)((p.n + 63) / 64));
    switch (p.store) {
    case F32: k_row_scale<F32><<<g, 256, 0, s>>>(p.n, (float*)p.A, p.lda, diag, p.rowscale, 0); break;
    case F16: k_row_scale<F16><<<g, 256, 0, s>>>(p.n, (half_t*)p.A, p.lda, diag, p.rowscale, 14); break;
    case BF16: k_row_scale<BF16><<<g, 256, 0, s>>>(p.n, (bf16_t*)p.A, p.lda, diag, p.rowscale, 0); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ============================================================== strip TRSMs + rounding
constexpr int SR = 32;  // rows (columns) per strip of L21 (U12) and per scale
constexpr int SW = 8;   // waves of a strip's work-group
constexpr int ST_THREADS = 64 * SW;

// The strip solves run on the FP32 matrix cores (v_mfma_f32_16x16x4f32: lane
// l = 16 g + c holds A[c][k + g] and B[k + g][c], register q of the result row
// 4 g + q, column c).  Both solves are one: with the strip's 32 rows (of L21) or
// columns (of U12) as runs of nb floats in LDS, Y_J = (S_J - sum_{I<J} M_JI S_I)
// Minv_J^T, where M(j, k) is U11(k, j), read from the column-major copy, or
// L11(j, k), from the row-major one: k contiguous, so that a lane takes four
// consecutive k of its run in one 16-byte load of either operand (the order of k
// is the same for both, and free).  Eight waves: one 16 x 16 tile of the 64 x 32
// block each, no sum over waves.
// maximum of v over the work-group (red: SW floats of LDS, free)
MXP_DEV float strip_max(float v, float* red) {
    v = warp_maxf(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int u = 1; u < SW; ++u) r = fmaxf(r, red[u]);
    __syncthreads();
    return r;
}

// four consecutive elements of a storage or operand array, one access
template <class T> struct alignas(4 * sizeof(T)) Pack4 {
    T v[4];
};

// Solve of a strip: run r at S + r SP, Minv the 64 x 64 diagonal-block inverses
// (element (j, k) at j + 64 k).  The factor does not depend on the strip: two
// 64 x 64 blocks' loads stay ahead of the products, and a step's inverse is
// loaded while the step before it runs.  A step has two barriers: before its
// last product (the run's newest values) and between the right-hand side, kept
// apart from S (R, pitch 68), and its product with the inverse.  Two sums per
// tile (alternate sixteens of k) keep consecutive products independent.
// What bounds it, at nb = 512: 10.5 MFLOP per strip, 17 us of a CU's FP32 matrix
// rate, and about 2 us of latencies in each of eight steps; 35 us for one strip
// per CU.  Against four waves of 32 x 32 x 2 products (four-byte operand loads,
// half of the sum in another wave, four barriers a step), rocprofv3, both sides'
// strips in one launch: nb = 512 66 -> 64 us (two strips per CU), nb = 256 (a group
// of six orders of 520 to 5003) 31 -> 24 us, nb = 256 FP32 (n = 2048)
// 17.1 -> 15.7 us; 64, 24.5 and 16.3 with the inverse's diagonal term added last.
MXP_DEV float strip_solve(float* S, int SP, int nbk, const float* __restrict__ M, int ld,
                          const float* __restrict__ Minv, float* R) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int RP = 68;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4, tj = wave & 3, h = wave >> 2;
    float m = 0.0f;   // max |y| over this lane's final stores
    // one 64 x 64 block of M: this wave's 16 rows, k = 16 u + 4 g ..
    auto ld_blk = [&](f4 (&a)[4], int J, int I) {
        const float* ub = M + (int64_t)(J * 64 + 16 * tj) * ld + I * 64;
        const int lo = c * ld + 4 * g;
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = *(const f4*)(ub + lo + 16 * u);
    };
    // the step's inverse, lower triangular in (row, k): this wave's 16 rows, the
    // sixteens of k left of its diagonal one (vi, k = 16 u + t + 4 g) and that (vd, k
    // = 16 tj + 4 t + g)
    auto ld_inv = [&](float (&vi)[12], float (&vd)[4], int J) {
        const float* ub = Minv + (int64_t)J * 4096 + 16 * tj;
        const int lo = c + 256 * g;
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t) vi[4 * u + t] = ub[lo + (16 * u + t) * 64];
#pragma unroll
        for (int t = 0; t < 4; ++t) vd[t] = ub[c + 64 * g + (16 * tj + 4 * t) * 64];
    };
    float* const Sr = S + (16 * h + c) * SP + 4 * g;             // this lane's run, its k
    float* const Rr = R + (16 * h + c) * RP + 4 * g;
    f4 acc0, acc1;
    auto mul_blk = [&](const f4 (&a)[4], int I) {
        f4 b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = *(const f4*)(Sr + I * 64 + 16 * u);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][t], b[0][t], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2][t], b[2][t], acc1, 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1][t], b[1][t], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3][t], b[3][t], acc1, 0, 0, 0);
        }
    };
    float iv[12], id[4];
    f4 m0[4], m1[4];
    ld_inv(iv, id, 0);
    for (int J = 0; J < nbk; ++J) {
        acc0 = acc1 = f4{0.0f, 0.0f, 0.0f, 0.0f};
        // m0 holds block (J, 0), m1 block (J, 1) (loaded during step J - 1); the
        // last block of the step takes the values the step before wrote
        int I = 0;
        for (; I + 2 < J; I += 2) {
            mul_blk(m0, I);
            ld_blk(m0, J, I + 2);
            mul_blk(m1, I + 1);
            if (I + 3 < J) ld_blk(m1, J, I + 3);
        }
        if (I + 1 < J) mul_blk(m0, I);
        __syncthreads();
        if (J > 0) {
            if (I + 1 < J) mul_blk(m1, I + 1);
            else mul_blk(m0, I);
        }
        if (J + 1 < nbk) {
            ld_blk(m0, J + 1, 0);
            if (J > 0) ld_blk(m1, J + 1, 1);
        }
        // rows 4 g + q of the tile: four consecutive values of the run
        const int o = J * 64 + 16 * tj;
        *(f4*)(Rr + 16 * tj) = *(const f4*)(Sr + o) - (acc0 + acc1);
        __syncthreads();
        // (the diagonal sixteen last and in the order of k: its diagonal entry, by far
        // the largest as a rule, is then the last one added; with terms after it,
        // each rounded at its magnitude, L21 and U12 were off by 0.60 and 0.46
        // instead of 0.42 and 0.29 units of 2^-24 of the largest, rms)
        acc0 = acc1 = f4{0.0f, 0.0f, 0.0f, 0.0f};
        auto mul_inv = [&](int u, f4& a) {
            const f4 b = *(const f4*)(Rr + 16 * u);
#pragma unroll
            for (int t = 0; t < 4; ++t) a = __builtin_amdgcn_mfma_f32_16x16x4f32(iv[4 * u + t], b[t], a, 0, 0, 0);
        };
        float bd[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) bd[t] = R[(16 * h + c) * RP + 16 * tj + 4 * t + g];
        if (tj > 0) mul_inv(0, acc0);                    // (wave-uniform)
        if (tj > 1) mul_inv(1, acc1);
        if (tj > 2) mul_inv(2, acc0);
        f4 y = acc0 + acc1;
#pragma unroll
        for (int t = 0; t < 4; ++t) y = __builtin_amdgcn_mfma_f32_16x16x4f32(id[t], bd[t], y, 0, 0, 0);
        if (J + 1 < nbk) ld_inv(iv, id, J + 1);
        *(f4*)(Sr + o) = y;
#pragma unroll
        for (int q = 0; q < 4; ++q) m = fmaxf(m, fabsf(y[q]));
    }
    __syncthreads();
    return strip_max(m, R);
}

// LDS of a strip kernel: the strip (32 runs, 16-byte aligned, of pitch nb + 4:
// the sixteen runs a load touches fall in distinct banks) and a step's right-hand
// side
MXP_DEV int strip_pitch(int nb) { return nb + 4; }
static inline size_t trsm_smem(int nb) { return (size_t)(SR * (nb + 4) + SR * 68) * sizeof(float); }
static inline size_t trsm_smem(int nb, int wgs) {
    return wgs <= NUM_CU && trsm_smem(nb) < OWN_CU_LDS ? OWN_CU_LDS : trsm_smem(nb);
}

// L21 strip: X (32 x nb) = A21[rows, :] U11^-1, then amax -> power-of-two
// scales; writes the operand Lq (K-major, update format, scaled), the stored
// L21 (storage format, scaled) and the scales.  A full strip moves through
// 4-element accesses (a lane: 4 rows of one column of A, 4 columns of one
// row of Lq), with every load of the strip in flight at once; the ragged
// last strip takes element accesses.
template <int ST, int OP>
MXP_DEV void trsm_L_strip(typename Store<ST>::T* A, int64_t lda, int64_t n, int64_t k, int nb,
                          const float* __restrict__ T, const float* __restrict__ uinv,
                          typename Operand<OP>::T* Lq, float* inv_sa, float* lsc_blk, float* smem, int w) {
    typedef typename Store<ST>::T STT;
    typedef typename Operand<OP>::T OPT;
    const int SP = strip_pitch(nb);
    float* S = smem;
    float* red = smem + SR * SP;
    const int tid = threadIdx.x;
    const int64_t r0 = k + nb + (int64_t)SR * w;
    int64_t rv = n - r0;
    rv = rv > SR ? SR : (rv < 0 ? 0 : rv);
    const bool vec = rv == SR && (r0 & 3) == 0 && (lda & 3) == 0 && ((uintptr_t)A & 15) == 0;
    const int rq = tid & 7, cg = tid >> 3;          // vector mapping: rows 4 rq.., column cg + 64 i
    if (vec) {
        for (int c0 = 0; c0 < nb; c0 += 512) {
            // loads without conditions (a column past nb reads column 0,
            // unused): a load under a branch ends in a wait for every load in
            // flight, which would serialise them
            Pack4<STT> x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = c0 + cg + 64 * i;
                x[i] = *(const Pack4<STT>*)(A + (r0 + 4 * rq) + (k + (c < nb ? c : 0)) * lda);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = c0 + cg + 64 * i;
                if (c < nb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) S[(4 * rq + q) * SP + c] = Store<ST>::load(x[i].v, q);
            }
        }
    } else {
        const int ii = tid & 31;
        for (int c = tid >> 5; c < nb; c += ST_THREADS / 32)
            S[ii * SP + c] = (ii < rv) ? Store<ST>::load(A, (r0 + ii) + (k + c) * lda) : 0.0f;
    }
    __syncthreads();
    const float amax = strip_solve(S, SP, nb / 64, T, nb, uinv, red);
    const float s_op = Operand<OP>::scaled ? pow2_scale(amax, Operand<OP>::scale_exp) : 1.0f;
    const float s_st = Store<ST>::scaled ? pow2_scale(amax, Store<ST>::scale_exp) : 1.0f;
    if (tid == 0) {
        inv_sa[w] = 1.0f / s_op;
        if (rv > 0) lsc_blk[r0 / SR] = s_st;
    }
    // operand rows (nb contiguous values each): 4 columns per lane
    OPT* Lw = Lq + (int64_t)SR * w * nb;
    for (int e = 4 * tid; e < SR * nb; e += 4 * ST_THREADS) {
        const int ii = e / nb, c = e - ii * nb;      // nb is a multiple of 64: a lane's 4 stay in one row
        Pack4<OPT> o;
#pragma unroll
        for (int q = 0; q < 4; ++q) o.v[q] = Operand<OP>::from_f32(S[ii * SP + c + q] * s_op);
        *(Pack4<OPT>*)(Lw + e) = o;
    }
    if (vec) {
        for (int c = cg; c < nb; c += ST_THREADS / 8) {
            Pack4<STT> o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o.v[q] = Store<ST>::from_f32(S[(4 * rq + q) * SP + c] * s_st);
            *(Pack4<STT>*)(A + (r0 + 4 * rq) + (k + c) * lda) = o;
        }
    } else {
        const int ii = tid & 31;
        if (ii < rv)
            for (int c = tid >> 5; c < nb; c += ST_THREADS / 32) A[(r0 + ii) + (k + c) * lda] = Store<ST>::from_f32(S[ii * SP + c] * s_st);
    }
}

// U12 strip: Y (nb x 32) = L11^-1 A12[:, cols]; operand Uq (K-major: column
// j has nb contiguous values) scaled, stored U12 unscaled.  Accesses as in
// the L21 strip, a lane taking 4 consecutive rows of one column.
template <int ST, int OP>
MXP_DEV void trsm_U_strip(typename Store<ST>::T* A, int64_t lda, int64_t n, int64_t k, int nb,
                          const float* __restrict__ Trm, const float* __restrict__ linv,
                          typename Operand<OP>::T* Uq, float* inv_sb, float* smem, int w) {
    typedef typename Store<ST>::T STT;
    typedef typename Operand<OP>::T OPT;
    const int SP = strip_pitch(nb);
    float* S = smem;
    float* red = smem + SR * SP;
    const int tid = threadIdx.x;
    const int64_t c0 = k + nb + (int64_t)SR * w;
    int64_t cv = n - c0;
    cv = cv > SR ? SR : (cv < 0 ? 0 : cv);
    // nb divides 1024: a load of the work-group covers 2048 / nb columns, a lane 4 rows
    const int qpc = nb >> 2, lq = __builtin_ctz((unsigned)qpc);
    const int kq = tid & (qpc - 1), cs = tid >> lq, cpp = ST_THREADS >> lq;
    const bool vec = (1024 % nb) == 0 && (k & 3) == 0 && (lda & 3) == 0 && ((uintptr_t)A & 15) == 0;
    if (vec) {
        for (int p0 = 0; p0 < SR; p0 += 8 * cpp) {
            // loads without conditions, as in the L21 strip (a column past the
            // matrix reads column k + nb, unused)
            Pack4<STT> x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int cc = p0 + cs + cpp * i;
                const int64_t col = (cc < SR && cc < cv) ? c0 + cc : k + nb;
                x[i] = *(const Pack4<STT>*)(A + (k + 4 * kq) + col * lda);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int cc = p0 + cs + cpp * i;
                if (cc < SR)
#pragma unroll
                    for (int q = 0; q < 4; ++q) S[cc * SP + 4 * kq + q] = (cc < cv) ? Store<ST>::load(x[i].v, q) : 0.0f;
            }
        }
    } else {
        for (int cc = 0; cc < SR; ++cc)
            for (int kk = tid; kk < nb; kk += ST_THREADS)
                S[cc * SP + kk] = (cc < cv) ? Store<ST>::load(A, (k + kk) + (c0 + cc) * lda) : 0.0f;
    }
    __syncthreads();
    const float amax = strip_solve(S, SP, nb / 64, Trm, nb, linv, red);
    const float s_op = Operand<OP>::scaled ? pow2_scale(amax, Operand<OP>::scale_exp) : 1.0f;
    if (tid == 0) inv_sb[w] = 1.0f / s_op;
    OPT* Uw = Uq + (int64_t)SR * w * nb;
    if (vec) {
        for (int cc = cs; cc < SR; cc += cpp) {
            Pack4<OPT> o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o.v[q] = Operand<OP>::from_f32(S[cc * SP + 4 * kq + q] * s_op);
            *(Pack4<OPT>*)(Uw + (int64_t)cc * nb + 4 * kq) = o;
            if (cc < cv) {
                Pack4<STT> a;
#pragma unroll
                for (int q = 0; q < 4; ++q) a.v[q] = Store<ST>::from_f32(S[cc * SP + 4 * kq + q]);
                *(Pack4<STT>*)(A + (k + 4 * kq) + (c0 + cc) * lda) = a;
            }
        }
    } else {
        for (int cc = 0; cc < SR; ++cc)
            for (int kk = tid; kk < nb; kk += ST_THREADS) {
                Uw[(int64_t)cc * nb + kk] = Operand<OP>::from_f32(S[cc * SP + kk] * s_op);
                if (cc < cv) A[(k + kk) + (c0 + cc) * lda] = Store<ST>::from_f32(S[cc * SP + kk]);
            }
    }
}

// Both strip solves of one block step in one launch: the first nstrip
// work-groups solve L21 strips, the next nstrip U12 strips (independent).  One
// launch serves a group of factorisations (one per request of the solve
// server, or a single one): their work-groups are numbered one after another.
struct TrsmOne {
    void* A;
    int64_t lda, n, k;
    int nb, s0, nstrip, wg_end;              // strips s0 .. s0 + nstrip - 1 of each side
    const float *T, *uinv, *Trm, *linv;
    void* Lq;
    float* inv_sa;
    float* lsc_blk;
    void* Uq;
    float* inv_sb;
};
struct TrsmGroup {
    TrsmOne g[GEMM_GROUP_MAX];
    int count;
};

template <int ST, int OP>
__global__ __launch_bounds__(ST_THREADS, 4) void k_trsm(const TrsmGroup grp) {
    extern __shared__ float smem[];
    int d = 0;
    while ((int)blockIdx.x >= grp.g[d].wg_end) ++d;
    const TrsmOne& G = grp.g[d];
    const int w = (int)blockIdx.x - (d > 0 ? grp.g[d - 1].wg_end : 0);
    typename Store<ST>::T* A = (typename Store<ST>::T*)G.A;
    if (w < G.nstrip)
        trsm_L_strip<ST, OP>(A, G.lda, G.n, G.k, G.nb, G.T, G.uinv, (typename Operand<OP>::T*)G.Lq, G.inv_sa,
                             G.lsc_blk, smem, G.s0 + w);
    else
        trsm_U_strip<ST, OP>(A, G.lda, G.n, G.k, G.nb, G.Trm, G.linv, (typename Operand<OP>::T*)G.Uq, G.inv_sb, smem,
                             G.s0 + w - G.nstrip);
}

// the solve of runs that are zero before their element 64 j0 (and stay so)
MXP_DEV void strip_solve_from(int j0, float* S, int SP, int nbk, const float* __restrict__ M, int ld,
                              const float* __restrict__ Minv, float* R) {
    strip_solve(S + 64 * j0, SP, nbk - j0, M + (int64_t)64 * j0 * (ld + 1), ld, Minv + 4096 * j0, R);
}

// Full FP32 inverses of a diagonal block (size kbp) by strips of 32:
// U11^-1 rows r0..r0+31 = I[r0:r0+32, :] U11^-1 (with T, the factor
// column-major), L11^-1 columns c0..c0+31 = L11^-1 I[:, c0:c0+32] (with Trm,
// row-major); out: the inverse, column-major, ld D.
MXP_DEV void inv_upper_strip(int kbp, const float* __restrict__ T, int ld, const float* __restrict__ uinv,
                             float* __restrict__ out, int64_t D, int r0, float* smem) {
    const int SP = strip_pitch(kbp);
    float* S = smem;
    float* red = smem + SR * SP;
    for (int e = threadIdx.x; e < SR * kbp; e += ST_THREADS) {
        int ii = e % SR, c = e / SR;
        S[ii * SP + c] = (r0 + ii == c) ? 1.0f : 0.0f;
    }
    __syncthreads();
    strip_solve_from(r0 / 64, S, SP, kbp / 64, T, ld, uinv, red);
    for (int e = threadIdx.x; e < SR * kbp; e += ST_THREADS) {
        int ii = e % SR, c = e / SR;
        out[(r0 + ii) + (int64_t)c * D] = S[ii * SP + c];
    }
}
MXP_DEV void inv_lower_strip(int kbp, const float* __restrict__ Trm, int ld, const float* __restrict__ linv,
                             float* __restrict__ out, int64_t D, int c0, float* smem) {
    const int SP = strip_pitch(kbp);
    float* S = smem;
    float* red = smem + SR * SP;
    for (int e = threadIdx.x; e < SR * kbp; e += ST_THREADS) {
        int kk = e % kbp, cc = e / kbp;
        S[cc * SP + kk] = (kk == c0 + cc) ? 1.0f : 0.0f;
    }
    __syncthreads();
    strip_solve_from(c0 / 64, S, SP, kbp / 64, Trm, ld, linv, red);
    for (int e = threadIdx.x; e < SR * kbp; e += ST_THREADS) {
        int kk = e % kbp, cc = e / kbp;
        out[kk + (int64_t)(c0 + cc) * D] = S[cc * SP + kk];
    }
}

// The inverses formed after the factorisation, up to GEMM_GROUP_MAX of them in a
// launch (work-groups numbered one after another): the full inverses of the diagonal
// blocks blk0 .. blk0 + nblk (every block with FP32 storage, the blocks whose strips
// were all solved by substitution otherwise; the strips of U11^-1, then those of
// L11^-1), then the off-diagonal blocks of the pairs (k_pair).  Block blk is diagonal
// block blk % g of the preconditioner's group blk / g (column-major, ld D).  The two
// triangles of all members are independent: one launch for both and for all of a
// group, then two for the pairs (one after the other, six launches a member, most of
// a few dozen work-groups: a group of n = 520 to 5003 at nb = 256 3.41 against
// 2.99 ms, the solve at n = 600 991 against 963 us).
struct InvOne {
    const void* A;
    int64_t lda, n, blk0;
    int nb, nblk, npair, wg_inv, wg_pair, pad;
    const float *T, *Trm, *linv, *uinv, *lsc;
    float *Li, *Ui;
};
struct InvGroup {
    InvOne g[GEMM_GROUP_MAX];
    int count;
};
__global__ __launch_bounds__(ST_THREADS) void k_inv(const InvGroup grp) {
    extern __shared__ float smem[];
    int d = 0;
    while ((int)blockIdx.x >= grp.g[d].wg_inv) ++d;
    const InvOne& G = grp.g[d];
    const int w = (int)blockIdx.x - (d > 0 ? grp.g[d - 1].wg_inv : 0);
    const int nb = G.nb, per = nb / SR, side = w / (per * G.nblk), v = w - side * per * G.nblk;
    const int64_t blk = G.blk0 + v / per;
    const int64_t k = blk * nb;
    const int kb = (int)(G.n - k < nb ? G.n - k : nb);
    const int kbp = (kb + 63) / 64 * 64;
    const int r0 = SR * (v % per);
    if (r0 >= kbp) return;
    const int64_t D = prec_block(nb), g = D / nb, o = (blk % g) * nb, out = (blk / g) * D * D + o + o * D;
    if (side == 0) inv_upper_strip(kbp, G.T + blk * nb * nb, nb, G.uinv + blk * nb * 64, G.Ui + out, D, r0, smem);
    else inv_lower_strip(kbp, G.Trm + blk * nb * nb, nb, G.linv + blk * nb * 64, G.Li + out, D, r0, smem);
}

// the inverses of one block step's diagonal blocks (16-bit storage: formed
// right after each diagonal-block LU, they serve the strip products and
// later the preconditioner): work-groups [0, kbp/32) of a descriptor solve
// the strips of L11^-1, the next kbp/32 those of U11^-1
__global__ __launch_bounds__(ST_THREADS) void k_block_inv(const PanelGroup grp) {
    extern __shared__ float smem[];
    int d = 0;
    while ((int)blockIdx.x >= grp.g[d].wg_inv) ++d;
    const PanelOne& G = grp.g[d];
    const int w0 = (int)blockIdx.x - (d > 0 ? grp.g[d - 1].wg_inv : 0);
    const int nstr = G.kbp / SR;
    if (w0 < nstr) inv_lower_strip(G.kbp, G.Trm, G.nb, G.linv, G.Li, G.ldi, SR * w0, smem);
    else inv_upper_strip(G.kbp, G.T, G.nb, G.uinv, G.Ui, G.ldi, SR * (w0 - nstr), smem);
}

hipError_t block_inverses(const PanelGroup& grp, int wg, int nbmax, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_block_inv,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       (int)trsm_smem(1024));
    if (attr) return attr;
    k_block_inv<<<wg, ST_THREADS, trsm_smem(nbmax, wg), s>>>(grp);
    return hipGetLastError();
}

// Off-diagonal blocks of the inverses of the pairs of diagonal blocks
// (blocks b0 = 2p, b1 = 2p + 1 of sizes nb and kb1):
//   [[L0, 0], [B, L1]]^-1 = [[L0^-1, 0], [-L1^-1 B L0^-1, L1^-1]],
//   [[U0, B'], [0, U1]]^-1 = [[U0^-1, -U0^-1 B' U1^-1], [0, U1^-1]],
// with B and B' the stored panels of the factor (B with its strip factors
// undone) and the diagonal inverses from k_inv.  Two launches over both
// triangles of all pairs, a 64 x 64 output tile per work-group on the FP32
// matrix cores; the K range of a tile skips the
// zero triangle of its triangular operand.
// LDS pitches of the staged operands (64 banks): A is written with the rows
// running over the lanes and read two k rows at a time (pitch 96: the two
// rows fall on distinct banks); B is written with k running over the lanes
// (pitch 97, odd: 32 consecutive k rows on distinct banks)
constexpr int PP_SP = 96, PP_SPB = 97;
typedef float f16v_t __attribute__((ext_vector_type(16)));
MXP_DEV f16v_t mfma2(float a, float b, f16v_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// acc (wave (wr, wc)'s 32 x 32 part of the 64 x 64 tile) += A[i0.., k] B[k, j0..] over k in [k_lo, k_hi);
// the next chunk's operands are loaded into registers before this chunk's
// products, so that their latency overlaps them
template <class FA, class FB>
MXP_DEV f16v_t pair_tile(FA fa, FB fb, int M, int N, int i0, int j0, int k_lo, int k_hi, float* sA, float* sB) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave & 1, wc = wave >> 1, lr = lane & 31, lh = lane >> 5;
    f16v_t acc = {};
    float ra[8], rb[8];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int e = tid + 256 * t;
            // loads without conditions (an index past the range reads a
            // valid element, weighted zero): a load under a branch would
            // wait for every load in flight
            const int i = i0 + (e & 63), k = k0 + (e >> 6);          // A: rows contiguous
            const float a = fa(i < M ? i : M - 1, k < k_hi ? k : k_hi - 1);
            ra[t] = (i < M && k < k_hi) ? a : 0.0f;
            const int kq = k0 + (e & 31), j = j0 + (e >> 5);         // B: k contiguous
            const float b = fb(kq < k_hi ? kq : k_hi - 1, j < N ? j : N - 1);
            rb[t] = (j < N && kq < k_hi) ? b : 0.0f;
        }
    };
    if (k_lo < k_hi) fetch(k_lo);
    for (int k0 = k_lo; k0 < k_hi; k0 += 32) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int e = tid + 256 * t;
            sA[(e >> 6) * PP_SP + (e & 63)] = ra[t];
            sB[(e & 31) * PP_SPB + (e >> 5)] = rb[t];
        }
        __syncthreads();
        if (k0 + 32 < k_hi) fetch(k0 + 32);
#pragma unroll
        for (int s2 = 0; s2 < 16; ++s2) {
            const int kk = 2 * s2 + lh;
            acc = mfma2(sA[kk * PP_SP + wr * 32 + lr], sB[kk * PP_SPB + wc * 32 + lr], acc);
        }
        __syncthreads();
    }
    return acc;
}

// C[i][j] = alpha acc, register q of lane l holding row 8(q/4) + 4(l/32) + q%4, column l%32
template <class FC>
MXP_DEV void pair_store(const f16v_t& acc, float alpha, int M, int N, int i0, int j0, FC fc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave & 1, wc = wave >> 1;
    const int j = j0 + wc * 32 + (lane & 31);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int i = i0 + wr * 32 + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
        if (i < M && j < N) fc(i, j, alpha * acc[q]);
    }
}

// phase 0: W = B L0^-1 (kb1 x nb), phase 1: X = -L1^-1 W.  W stands in the pair's
// upper right block, which is zero in the inverse and never read.
template <int ST>
MXP_DEV void pair_lower(const InvOne& G, int64_t p, int i0, int j0, int phase, float* sA, float* sB) {
    typedef typename Store<ST>::T T;
    const T* A = (const T*)G.A;
    const int nb = G.nb;
    const int64_t n = G.n, lda = G.lda, D = 2 * (int64_t)nb;
    const int64_t k0 = p * D, k1 = k0 + nb, nstrips32 = (n + 31) / 32;
    if (k1 >= n) return;
    const int kb1 = (int)(n - k1 < nb ? n - k1 : nb);
    float* inv = G.Li + p * D * D;
    float* Wp = inv + nb * D;
    const float* lsc = G.lsc;
    if (phase == 0) {
        if (i0 >= kb1) return;
        const float* srow = lsc + (2 * p) * nstrips32;
        auto fa = [&](int i, int k) {
            return Store<ST>::load(A, (k1 + i) + (k0 + k) * lda) / srow[(k1 + i) / 32];
        };
        auto fb = [&](int k, int j) { return inv[k + (int64_t)j * D]; };
        const f16v_t acc = pair_tile(fa, fb, kb1, nb, i0, j0, j0, nb, sA, sB);   // L0^-1[k][j] = 0 for k < j
        pair_store(acc, 1.0f, kb1, nb, i0, j0, [&](int i, int j, float v) { Wp[i + (int64_t)j * D] = v; });
    } else {
        if (i0 >= kb1) return;
        auto fa = [&](int i, int k) { return inv[(nb + i) + (int64_t)(nb + k) * D]; };
        auto fb = [&](int k, int j) { return Wp[k + (int64_t)j * D]; };
        const int kh = i0 + 64 < kb1 ? i0 + 64 : kb1;                             // L1^-1[i][k] = 0 for k > i
        const f16v_t acc = pair_tile(fa, fb, kb1, nb, i0, j0, 0, kh, sA, sB);
        pair_store(acc, -1.0f, kb1, nb, i0, j0, [&](int i, int j, float v) { inv[(nb + i) + (int64_t)j * D] = v; });
    }
}

// phase 0: W = U0^-1 B' (nb x kb1, in the pair's lower left block), phase 1:
// Y = -W U1^-1
template <int ST>
MXP_DEV void pair_upper(const InvOne& G, int64_t p, int i0, int j0, int phase, float* sA, float* sB) {
    typedef typename Store<ST>::T T;
    const T* A = (const T*)G.A;
    const int nb = G.nb;
    const int64_t n = G.n, lda = G.lda, D = 2 * (int64_t)nb;
    const int64_t k0 = p * D, k1 = k0 + nb;
    if (k1 >= n) return;
    const int kb1 = (int)(n - k1 < nb ? n - k1 : nb);
    float* inv = G.Ui + p * D * D;
    float* Wp = inv + nb;
    if (j0 >= kb1) return;
    if (phase == 0) {
        auto fa = [&](int i, int k) { return inv[i + (int64_t)k * D]; };
        auto fb = [&](int k, int j) { return Store<ST>::load(A, (k0 + k) + (k1 + j) * lda); };
        const f16v_t acc = pair_tile(fa, fb, nb, kb1, i0, j0, i0, nb, sA, sB);   // U0^-1[i][k] = 0 for k < i
        pair_store(acc, 1.0f, nb, kb1, i0, j0, [&](int i, int j, float v) { Wp[i + (int64_t)j * D] = v; });
    } else {
        auto fa = [&](int i, int k) { return Wp[i + (int64_t)k * D]; };
        auto fb = [&](int k, int j) { return inv[(nb + k) + (int64_t)(nb + j) * D]; };
        const int kh = j0 + 64 < kb1 ? j0 + 64 : kb1;                             // U1^-1[k][j] = 0 for k > j
        const f16v_t acc = pair_tile(fa, fb, nb, kb1, i0, j0, 0, kh, sA, sB);
        pair_store(acc, -1.0f, nb, kb1, i0, j0, [&](int i, int j, float v) { inv[i + (int64_t)(nb + j) * D] = v; });
    }
}

template <int ST> __global__ __launch_bounds__(256) void k_pair(const InvGroup grp, int phase) {
    __shared__ float sA[32 * PP_SP], sB[32 * PP_SPB];
    int d = 0;
    while ((int)blockIdx.x >= grp.g[d].wg_pair) ++d;
    const InvOne& G = grp.g[d];
    const int w = (int)blockIdx.x - (d > 0 ? grp.g[d - 1].wg_pair : 0);
    const int t = G.nb / 64, q = w / (t * t), e = w - q * t * t;         // q: triangle and pair
    const int j0 = 64 * (e % t), i0 = 64 * (e / t);
    if (q < G.npair) pair_lower<ST>(G, q, i0, j0, phase, sA, sB);
    else pair_upper<ST>(G, q - G.npair, i0, j0, phase, sA, sB);
}

// The strips of block step k.  While they are no more than the CUs, one launch
// solves them all, a CU each.  Above, the first ones -- the next block's rows and
// columns, all that the next diagonal block waits for -- are solved on their own
// by substitution (44 to 48 us at nb = 512 where all strips of a step take 70 to
// 75 us and more beside the merged update), the others after them.
static int strip_count(const FactorPlan& p, int64_t k) {
    const int64_t m = p.n - k - p.nb;
    return m > 0 ? (int)(rup(m, 256) / SR) : 0;
}
static int first_strips(const FactorPlan& p, int64_t k) {
    return 2 * strip_count(p, k) <= NUM_CU ? strip_count(p, k) : (int)(p.nb / SR);
}

// Block step k solves its other strips through the block inverses (16-bit storage)
// while at least 16 blocks are left: the products free the compute units that the
// substitution would hold beside the merged update.  With fewer left they are
// solved by substitution too: the inverses' 16-bit parts are not as accurate.
// Against FP64 from the FP32 factor of the block, in units of 2^-24 of a column's
// largest (a model with these roundings, nb = 512, dominant and sqrt(n) matrices):
// substitution 0.35-0.45, two FP16 parts 3.9-4.5, three BF16 parts 0.58-0.60.
// (Products wherever there are other strips would be the faster: n = 12013
// nb = 512 BF16 5.82 against 5.95 ms, n = 16000 nb = 1024 BF16 9.7 against 12.0,
// n = 20001 nb = 512 FP8 on FP16 10.68 against 10.74.)
// Depends on (n, nb, k) alone, so that grouped and single factorisations take the
// same path.
constexpr int INV_BLOCKS = 16;
static bool inverse_path(const FactorPlan& p, int64_t k) {
    return panel_path(p.store) && strip_count(p, k) > first_strips(p, k) && p.n - k - p.nb >= INV_BLOCKS * p.nb;
}
// the first block whose inverses are formed after the factorisation
static int64_t inv_first_after(const FactorPlan& p) {
    const int64_t nblk = (p.n + p.nb - 1) / p.nb;
    int64_t b = 0;
    while (b < nblk && inverse_path(p, b * p.nb)) ++b;
    return b;
}

// the full FP32 inverses of the preconditioner's diagonal blocks (after the
// factorisations): every factor block's, then the off-diagonal blocks of the
// pairs
template <int ST>
static hipError_t prec_inverses(const FactorPlan* P, int count, hipStream_t s) {
    InvGroup grp;
    grp.count = count;
    int wi = 0, wp = 0, nbmax = 64;
    double fl = 0, by = 0;
    for (int i = 0; i < count; ++i) {
        const FactorPlan& p = P[i];
        InvOne& g = grp.g[i];
        const int64_t n = p.n, nb = p.nb;
        g.A = p.A; g.lda = p.lda; g.n = n; g.nb = (int)nb; g.pad = 0;
        // blocks before blk0 got their inverses during the factorisation
        g.blk0 = inv_first_after(p);
        g.nblk = (int)((n + nb - 1) / nb - g.blk0);
        g.npair = prec_block(nb) == 2 * nb && n > nb ? (int)((n + 2 * nb - 1) / (2 * nb)) : 0;
        g.wg_inv = wi += 2 * g.nblk * (int)(nb / SR);
        g.wg_pair = wp += 2 * g.npair * (int)((nb / 64) * (nb / 64));
        g.T = p.T; g.Trm = p.Trm; g.linv = p.linv; g.uinv = p.uinv; g.lsc = p.lsc;
        g.Li = p.linv_full; g.Ui = p.uinv_full;
        nbmax = (int)nb > nbmax ? (int)nb : nbmax;
        fl += (2.0 / 3.0 + (g.npair ? 4.0 : 0.0)) * (double)n * nb * nb;
        by += 16.0 * (double)n * nb;
    }
    hipEvent_t pt = prof::begin(prof::DIAG, s);
    if (wi) k_inv<<<wi, ST_THREADS, trsm_smem(nbmax, wi), s>>>(grp);
    if (wp)
        for (int ph = 0; ph < 2; ++ph) k_pair<ST><<<wp, 256, 0, s>>>(grp, ph);
    prof::end(pt, prof::DIAG, s, fl, by);
    return hipGetLastError();
}

// ============================================================== driver

hipError_t lookahead_create(Lookahead* la) {
    hipError_t e;
    if ((e = hipStreamCreateWithFlags(&la->side, hipStreamNonBlocking))) return e;
    if ((e = hipStreamCreateWithFlags(&la->chain, hipStreamNonBlocking))) return e;
    for (hipEvent_t* ev : {&la->ev_upd, &la->ev_cross, &la->ev_diag, &la->ev_first, &la->ev_panel, &la->ev_side})
        if ((e = hipEventCreateWithFlags(ev, hipEventDisableTiming))) return e;
    return hipSuccess;
}

void lookahead_destroy(Lookahead* la) {
    for (hipEvent_t ev : {la->ev_upd, la->ev_cross, la->ev_diag, la->ev_first, la->ev_panel, la->ev_side})
        if (ev) (void)hipEventDestroy(ev);
    if (la->chain) (void)hipStreamDestroy(la->chain);
    if (la->side) (void)hipStreamDestroy(la->side);
    *la = Lookahead();
}

// Look-ahead contexts of callers that bring none: a pool per device
// (default stream priority).  A call takes a context for the time it
// enqueues its work and returns it afterwards; work still in flight on the
// context's own streams is no hazard for the next user, whose waits and
// records are enqueued after it (a wait on an event refers to the event's
// latest record at the time of the wait call).  Two calls never enqueue on
// one context at the same time.
static std::vector<Lookahead*> g_la_free[64];
static std::mutex g_la_mutex;

static hipError_t lookahead_acquire(int dev, Lookahead** out) {
    {
        std::lock_guard<std::mutex> lock(g_la_mutex);
        if (!g_la_free[dev].empty()) {
            *out = g_la_free[dev].back();
            g_la_free[dev].pop_back();
            return hipSuccess;
        }
    }
    Lookahead* L = new Lookahead();
    hipError_t e = lookahead_create(L);
    if (e) {
        lookahead_destroy(L);
        delete L;
        return e;
    }
    *out = L;
    return hipSuccess;
}

static void lookahead_release(int dev, Lookahead* L) {
    std::lock_guard<std::mutex> lock(g_la_mutex);
    g_la_free[dev].push_back(L);
}

// the strip-TRSM descriptor of strips [s0, s0 + count) per side of block step k
// of a factorisation; wg_begin: the work-groups of the group before it
template <int ST, int OP>
static void trsm_desc(const FactorPlan& p, int64_t k, int s0, int count, TrsmOne& g, int wg_begin) {
    typedef typename Operand<OP>::T OP_T;
    const int nb = (int)p.nb;
    const int64_t blk = k / nb;
    const int set = (int)(blk & 3);
    const int64_t opset = p.op_rows * nb, scset = p.op_rows / 32;
    g.A = p.A; g.lda = p.lda; g.n = p.n; g.k = k; g.nb = nb; g.s0 = s0; g.nstrip = count;
    g.wg_end = wg_begin + 2 * count;
    g.Trm = p.Trm + blk * nb * nb;
    g.uinv = p.uinv + blk * nb * 64;
    g.T = p.T + blk * nb * nb;
    g.linv = p.linv + blk * nb * 64;
    g.Lq = (OP_T*)p.Lq + set * opset;
    g.inv_sa = p.inv_sa + set * scset;
    g.lsc_blk = p.lsc + blk * ((p.n + SR - 1) / SR);
    g.Uq = (OP_T*)p.Uq + set * opset;
    g.inv_sb = p.inv_sb + set * scset;
}

// The descriptor of block step k for the inverse-based strip solves; tr:
// the output tile rows of the panel_trsm launch (panel_rows of the largest
// nb it serves); wg0: the first work-group numbers of the three launches.
// Blocks without a trailing part (the last) only get their inverses.
static void panel_desc(const FactorPlan& p, int64_t k, int tr, PanelOne& g, const int wg0[3]) {
    const int nb = (int)p.nb;
    const int kb = (int)(p.n - k < nb ? p.n - k : nb);
    const int64_t m = p.n - k - kb;
    const int64_t blk = k / nb;
    const int set = (int)(blk & 3);
    const int eb = dtype_bytes(p.update);
    const int64_t opset = p.op_rows * nb, scset = p.op_rows / 32;
    const int64_t D = prec_block(nb), gsz = D / nb, o = (blk % gsz) * nb;
    g.A = p.A; g.lda = p.lda; g.n = p.n; g.k = k; g.ldi = D;
    g.nb = nb; g.kbp = (int)rup(kb, 64);
    g.tile0 = first_strips(p, k) * SR / tr;
    g.ntile = m > 0 ? (int)(rup(m, 256) / tr) - g.tile0 : 0;
    g.pad = 0;
    g.wg_inv = wg0[0] + 2 * (g.kbp / SR);
    g.wg_split = wg0[1] + (m > 0 ? 2 * (nb / 16) : 0);
    g.wg_trsm = wg0[2] + 2 * g.ntile;
    g.T = p.T + blk * nb * nb;
    g.Trm = p.Trm + blk * nb * nb;
    g.linv = p.linv + blk * nb * 64;
    g.uinv = p.uinv + blk * nb * 64;
    g.Li = p.linv_full + (blk / gsz) * D * D + o + o * D;
    g.Ui = p.uinv_full + (blk / gsz) * D * D + o + o * D;
    g.ub = p.binv;
    g.lb = (char*)p.binv + (size_t)3 * nb * nb * 2;
    g.ubs = p.binv_sc;
    g.lbs = p.binv_sc + nb;
    g.Lq = (char*)p.Lq + (size_t)set * opset * eb;
    g.inv_sa = p.inv_sa + set * scset;
    g.lsc_blk = p.lsc + blk * ((p.n + SR - 1) / SR);
    g.Uq = (char*)p.Uq + (size_t)set * opset * eb;
    g.inv_sb = p.inv_sb + set * scset;
}

// The trailing updates of the block steps, taken in pairs: block column and
// row k+1 receive the update of step k alone (they form panel k+1), and
// everything beyond them the updates of steps k and k+1 in one pass with K =
// 2 nb (one rounding to the storage format instead of two, half the C
// traffic).  With steps (k, k+1) a pair (k even in blocks), every element is
// computed by the same arithmetic however the updates are cut into launches.
//
// The operands of step j sit in set (j / nb) & 3 (four sets: two pairs in
// flight); row r of a set belongs to global row (column) j + nb + r.
template <int ST, int OP>
static GemmCall pair_call(const FactorPlan& p, int64_t j, bool pair, int64_t r0, int64_t c0, int64_t M,
                          int64_t N) {
    typedef typename Store<ST>::T ST_T;
    typedef typename Operand<OP>::T OP_T;
    const int64_t nb = p.nb;
    const int64_t opset = p.op_rows * nb, scset = p.op_rows / 32;
    GemmCall g{};
    g.C = (ST_T*)p.A + r0 + c0 * p.lda;
    g.ldc = p.lda;
    g.M = M;
    g.N = N;
    auto seg = [&](int64_t step, const void*& a, const void*& b, const float*& sa, const float*& sb) {
        const int set = (int)((step / nb) & 3);
        const int64_t ro = r0 - step - nb, co = c0 - step - nb;
        a = (const OP_T*)p.Lq + set * opset + ro * nb;
        b = (const OP_T*)p.Uq + set * opset + co * nb;
        sa = p.inv_sa + set * scset + ro / 32;
        sb = p.inv_sb + set * scset + co / 32;
    };
    g.K = (int)nb;
    seg(j, g.Aq, g.Bq, g.inv_sa, g.inv_sb);
    if (pair) {
        g.K2 = (int)nb;
        seg(j + nb, g.Aq2, g.Bq2, g.inv_sa2, g.inv_sb2);
    }
    return g;
}

// the update of block column and row b (width w, from global index b) by
// step j alone or by the pair (j, j+nb): two descriptors
template <int ST, int OP>
static int cross_calls(const FactorPlan& p, int64_t j, bool pair, int64_t b, GemmCall* out) {
    const int64_t n = p.n, w = n - b < p.nb ? n - b : p.nb;
    int c = 0;
    out[c++] = pair_call<ST, OP>(p, j, pair, b, b, n - b, w);               // block column b, diagonal included
    if (n - b - w > 0) out[c++] = pair_call<ST, OP>(p, j, pair, b, b + w, w, n - b - w);   // rest of block row b
    return c;
}

// Right-looking blocked LU with look-ahead on three streams, the updates taken
// in pairs (see above).
//   chain: what the next diagonal block waits for, and nothing else: with (a, b)
//   a pair of blocks, the diagonal block a's update by the pair before, its LU,
//   the strips of step a in block b, the diagonal block b's update by step a, its
//   LU, the strips of step b in the block after it.
//   side: the other strips of step a, the rest of block column and row b by step
//   a, the other strips of step b.
//   the caller's stream: the update by the pair before of the rest of block column
//   and row a and of block column and row b in one launch, then of everything
//   beyond.
// With every strip and the whole of block column and row b on the chain (which
// is still the order where one launch solves a step's strips) the factorisation at
// n = 12013 nb = 512 BF16 took 6.65 ms against 6.17, the solve at n = 20001 with FP8
// operands 16.9 against 15.6 (6.15 and 15.3 now): there a step's 300 us and more of chain (LU
// 150, inverses, their parts and products 160, update 20) became 270 (LU 175 beside
// the products, strips 60 to 85, update 17).
// One event per hand-over, waited for before its next record is enqueued.  The
// operand sets of a pair are rewritten by the strips two pairs later, which
// both streams enqueue after they have seen the pair's last update end.  The
// diagonal blocks' updates read whole tiles of operand rows: those past the block
// may be strips just being written, whose products are not stored.
template <int ST, int OP>
static hipError_t factor_typed(const FactorPlan& p, hipStream_t s, Lookahead* la) {
    typedef typename Store<ST>::T ST_T;
    typedef typename Operand<OP>::T OP_T;
    static const hipError_t attr = []() {
        hipError_t e2;
        if ((e2 = hipFuncSetAttribute((const void*)k_trsm<ST, OP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)trsm_smem(1024)))) return e2;
        return hipFuncSetAttribute((const void*)k_inv, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)trsm_smem(1024));
    }();
    if (attr) return attr;
    hipError_t e;
    Lookahead* LA = la;
    ST_T* A = (ST_T*)p.A;
    constexpr bool NP = ST == F16 || ST == BF16;     // strip solves through the block inverses
    const int64_t n = p.n, lda = p.lda;
    const int nb = (int)p.nb;

    // diagonal-block LU of block k (latency-bound: a handful of small grids)
    auto diag = [&](int64_t k, hipStream_t st) -> hipError_t {
        const int kb = (int)(n - k < nb ? n - k : nb);
        const int kbp = (int)rup(kb, 64);
        const int64_t blk = k / nb;
        float* T = p.T + blk * nb * nb;
        float* linv = p.linv + blk * nb * 64;
        float* uinv = p.uinv + blk * nb * 64;
        hipEvent_t pt = prof::begin(prof::DIAG, st);
        hipError_t e2 = diag_lu(ST, A, lda, k, kb, kbp, T, p.Trm + blk * nb * nb, nb, linv, uinv,
                                p.dsync + blk * diag_sync_words(nb), p.info, st);
        if (e2) return e2;
        prof::end(pt, prof::DIAG, st, 2.0 / 3.0 * kb * (double)kb * kb, 2.0 * kb * (double)kb * sizeof(ST_T));
        return hipGetLastError();
    };
    // strips [s0, s0 + count) of each side of block step k by substitution
    auto strips = [&](int64_t k, int s0, int count, hipStream_t st) -> hipError_t {
        if (count <= 0) return hipSuccess;
        TrsmGroup grp;
        trsm_desc<ST, OP>(p, k, s0, count, grp.g[0], 0);
        grp.count = 1;
        const double m = (double)count * SR;
        hipEvent_t pt = prof::begin(prof::TRSM, st);
        k_trsm<ST, OP><<<grp.g[0].wg_end, ST_THREADS, trsm_smem(nb, grp.g[0].wg_end), st>>>(grp);
        prof::end(pt, prof::TRSM, st, 2.0 * m * nb * nb, 4.0 * m * nb * sizeof(ST_T) + 2.0 * m * nb * sizeof(OP_T));
        return hipGetLastError();
    };
    // the strips beyond the first (wide grids: all CUs)
    auto other_strips = [&](int64_t k, hipStream_t st) -> hipError_t {
        const int s0 = first_strips(p, k);
        if (!(NP && inverse_path(p, k))) return strips(k, s0, strip_count(p, k) - s0, st);
        // the block's inverses, their 16-bit parts (the strip products' B
        // operands) and the products
        PanelGroup pg;
        const int wg0[3] = {0, 0, 0};
        panel_desc(p, k, panel_rows(ST, nb), pg.g[0], wg0);
        pg.count = 1;
        const double m = (double)(n - k - nb);
        hipEvent_t pt = prof::begin(prof::TRSM, st);
        hipError_t e2 = block_inverses(pg, pg.g[0].wg_inv, nb, st);
        if (!e2) e2 = panel_split(ST, pg, pg.g[0].wg_split, nb, st);
        if (!e2) e2 = panel_trsm(ST, OP, pg, pg.g[0].wg_trsm, nb, st);
        prof::end(pt, prof::TRSM, st, 4.0 * m * nb * nb + 4.0 / 3.0 * nb * (double)nb * nb,
                  4.0 * m * nb * sizeof(ST_T) + 2.0 * m * nb * sizeof(OP_T) + 8.0 * nb * (double)nb);
        return e2;
    };
    // one trailing-update launch of up to two descriptors, timed on its own
    auto gemm = [&](const GemmCall* c, int cnt, hipStream_t st) -> hipError_t {
        double fl = 0, by = 0;
        for (int i = 0; i < cnt; ++i) {
            const double K = c[i].K + c[i].K2;
            fl += 2.0 * c[i].M * (double)c[i].N * K;
            by += 2.0 * c[i].M * (double)c[i].N * sizeof(ST_T) + (c[i].M + c[i].N) * K * sizeof(OP_T);
        }
        if (fl == 0) return hipSuccess;
        // launches of fewer 256-row tiles than CUs (the late steps, the
        // diagonal block) take 128-row tiles: twice the work-groups, the
        // same arithmetic per element
        int tile = p.gemm_tile;
        int64_t tiles = 0;
        for (int i = 0; i < cnt; ++i) tiles += ((c[i].M + 255) / 256) * ((c[i].N + 127) / 128);
        if (tiles < 256) tile = GEMM_TILE_128;
        hipEvent_t pt = prof::begin(prof::GEMM, st);
        hipError_t e2 = gemm_group(OP, ST, tile, c, cnt, st);
        prof::end(pt, prof::GEMM, st, fl, by);
        return e2;
    };
    // the diagonal block b by step j (pair: by steps j and j + nb)
    auto diag_update = [&](int64_t j, bool pair, int64_t b, hipStream_t st) -> hipError_t {
        const int64_t w = n - b < nb ? n - b : nb;
        GemmCall c = pair_call<ST, OP>(p, j, pair, b, b, w, w);
        return gemm(&c, 1, st);
    };

    if ((e = fill_u64(p.info, 1, ~0ull, s))) return e;
    {
        const int64_t words = ((n + nb - 1) / nb) * (int64_t)diag_sync_words(nb);
        if ((e = fill_u64(p.dsync, (words + 1) / 2, 0ull, s))) return e;
    }
    if (n <= nb) {
        if ((e = diag(0, s))) return e;
        return prec_inverses<ST>(&p, 1, s);
    }
    // the first pair of a matrix whose strips are solved in one launch has nothing
    // to overlap with: it stays on the caller's stream
    const bool lone = first_strips(p, 0) == strip_count(p, 0);
    hipStream_t chain = lone ? s : LA->chain;
    // Under stream capture the side stream's work goes to the chain: a captured call
    // only forks from the caller's stream and joins it (a capture in which two forked
    // streams wait for each other's events ended the process).
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture)) {             // (no answer for the null stream beside a capture)
        (void)hipGetLastError();
        capture = hipStreamCaptureStatusNone;
    }
    const bool apart = capture == hipStreamCaptureStatusNone;
    const hipStream_t side = apart ? LA->side : LA->chain;
    bool side_used = false;
    // the strips of step j: the first (or all); the others behind them, through
    // the inverses, which start with a launch of few work-groups, beside them
    auto panel = [&](int64_t j) -> hipError_t {
        const int first = first_strips(p, j);
        if (first == strip_count(p, j)) return strips(j, 0, first, chain);
        const bool inv = NP && inverse_path(p, j);
        side_used = apart;
        hipError_t e2;
        if (apart && inv) {
            if ((e2 = hipEventRecord(LA->ev_diag, chain))) return e2;
            if ((e2 = hipStreamWaitEvent(side, LA->ev_diag, 0))) return e2;
        }
        if ((e2 = strips(j, 0, first, chain))) return e2;
        if (!apart) return other_strips(j, side);
        if ((e2 = hipEventRecord(LA->ev_first, chain))) return e2;
        if (!inv && (e2 = hipStreamWaitEvent(side, LA->ev_first, 0))) return e2;
        if ((e2 = other_strips(j, side))) return e2;
        return inv ? hipStreamWaitEvent(side, LA->ev_first, 0) : hipSuccess;
    };
    for (int64_t a = 0; a < n; a += 2 * nb) {
        const int64_t b = a + nb, k = a - 2 * nb;        // (k, k + nb): the pair before
        const int64_t wa = n - a < nb ? n - a : nb;
        if (a == 0 || (a == 2 * nb && lone)) {
            if ((e = hipEventRecord(LA->ev_upd, s))) return e;
            if (a > 0) chain = LA->chain;
        }
        // chain: diagonal block a (the pair before's predecessor has updated it)
        if (chain != s && (e = hipStreamWaitEvent(chain, LA->ev_upd, 0))) return e;
        if (a > 0 && (e = diag_update(k, true, a, chain))) return e;
        if ((e = diag(a, chain))) return e;
        if (b >= n) break;
        if (a > 0) {
            // the caller's stream: the pair before's panels are formed
            if ((k > 0 || !lone) && (e = hipStreamWaitEvent(s, LA->ev_panel, 0))) return e;
            if (side_used && (e = hipStreamWaitEvent(s, LA->ev_side, 0))) return e;
            GemmCall c[4];
            int cnt = 0;
            c[cnt++] = pair_call<ST, OP>(p, k, true, b, a, n - b, wa);
            c[cnt++] = pair_call<ST, OP>(p, k, true, a, b, wa, n - b);
            cnt += cross_calls<ST, OP>(p, k, true, b, c + cnt);
            if ((e = gemm(c, cnt, s))) return e;
            if ((e = hipEventRecord(LA->ev_cross, s))) return e;
            if (n - b > nb) {
                GemmCall d = pair_call<ST, OP>(p, k, true, b + nb, b + nb, n - b - nb, n - b - nb);
                if ((e = gemm(&d, 1, s))) return e;
            }
            if ((e = hipEventRecord(LA->ev_upd, s))) return e;
            if ((e = hipStreamWaitEvent(chain, LA->ev_cross, 0))) return e;
        }
        const int64_t wb = n - b < nb ? n - b : nb, c0 = b + wb;
        const bool whole = first_strips(p, a) == strip_count(p, a);
        if ((e = panel(a))) return e;
        GemmCall c[2];
        if (whole) {
            // block column and row b by step a
            const int cnt = cross_calls<ST, OP>(p, a, false, b, c);
            if ((e = gemm(c, cnt, chain))) return e;
        } else if ((e = diag_update(a, false, b, chain))) {
            return e;
        }
        if ((e = diag(b, chain))) return e;
        if (c0 < n) {
            if (!whole) {
                // side: the rest of block column and row b by step a
                c[0] = pair_call<ST, OP>(p, a, false, c0, b, n - c0, wb);
                c[1] = pair_call<ST, OP>(p, a, false, b, c0, wb, n - c0);
                if ((e = gemm(c, 2, side))) return e;
                if (apart && (e = hipEventRecord(LA->ev_side, side))) return e;
                if (apart && (e = hipStreamWaitEvent(chain, LA->ev_side, 0))) return e;
            }
            if ((e = panel(b))) return e;
        }
        if (chain != s && (e = hipEventRecord(LA->ev_panel, chain))) return e;
        if (side_used && (e = hipEventRecord(LA->ev_side, side))) return e;
    }
    // the caller's stream ends after every kernel of the other two
    if (chain != s) {
        if ((e = hipEventRecord(LA->ev_panel, chain))) return e;
        if ((e = hipStreamWaitEvent(s, LA->ev_panel, 0))) return e;
    }
    if (side_used && (e = hipStreamWaitEvent(s, LA->ev_side, 0))) return e;
    // full FP32 inverses of the preconditioner's diagonal blocks
    return prec_inverses<ST>(&p, 1, s);
}

static hipError_t factor_dispatch(const FactorPlan& p, hipStream_t s, Lookahead* la) {
    const int u = p.update, t = p.store;
    if (u == F32 && t == F32) return factor_typed<F32, F32>(p, s, la);
    if (u == F16 && t == F16) return factor_typed<F16, F16>(p, s, la);
    if (u == BF16 && t == BF16) return factor_typed<BF16, BF16>(p, s, la);
    if (u == F8 && t == F16) return factor_typed<F16, F8>(p, s, la);
    if (u == F8 && t == BF16) return factor_typed<BF16, F8>(p, s, la);
    if (u == F16 && t == F32) return factor_typed<F32, F16>(p, s, la);
    if (u == BF16 && t == F32) return factor_typed<F32, BF16>(p, s, la);
    return hipErrorInvalidValue;
}

template <int ST, int OP>
static hipError_t factor_group_typed(const FactorPlan* P, int count, hipStream_t s) {
    typedef typename Store<ST>::T ST_T;
    typedef typename Operand<OP>::T OP_T;
    constexpr bool NP = ST == F16 || ST == BF16;     // strip solves through the block inverses
    hipError_t e;
    if ((e = hipFuncSetAttribute((const void*)k_trsm<ST, OP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)trsm_smem(1024))))
        return e;
    if ((e = hipFuncSetAttribute((const void*)k_inv, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)trsm_smem(1024))))
        return e;
    int64_t steps = 0;
    for (int g = 0; g < count; ++g) {
        const FactorPlan& p = P[g];
        if ((e = fill_u64(p.info, 1, ~0ull, s))) return e;
        const int64_t nblk = (p.n + p.nb - 1) / p.nb;
        const int64_t words = nblk * (int64_t)diag_sync_words(p.nb);
        if ((e = fill_u64(p.dsync, (words + 1) / 2, 0ull, s))) return e;
        steps = nblk > steps ? nblk : steps;
    }
    // panel t (diagonal-block LU, strip TRSMs) of every factorisation that has block t
    auto panels = [&](int64_t t) -> hipError_t {
        DiagCall dc[GEMM_GROUP_MAX];
        TrsmGroup tg;
        PanelGroup pg;
        int nd = 0, nt = 0, np = 0, wg = 0, nbmax = 64, pnbmax = 64;
        for (int g = 0; g < count; ++g) {
            const FactorPlan& p = P[g];
            const int nb = (int)p.nb;
            const int64_t k = t * nb;
            if (k >= p.n) continue;
            const int kb = (int)(p.n - k < nb ? p.n - k : nb);
            const int64_t blk = k / nb, m = p.n - k - kb;
            dc[nd++] = DiagCall{p.A, p.lda, k, kb, (int)rup(kb, 64), nb, p.T + blk * nb * nb, p.Trm + blk * nb * nb,
                                p.linv + blk * nb * 64, p.uinv + blk * nb * 64, p.dsync + blk * diag_sync_words(nb),
                                p.info};
            const bool inv = NP && inverse_path(p, k);
            if (inv) {
                pg.g[np++].nb = nb;                       // descriptors filled below (tile rows need nbmax)
                pnbmax = nb > pnbmax ? nb : pnbmax;
            }
            if (m <= 0) continue;
            trsm_desc<ST, OP>(p, k, 0, inv ? first_strips(p, k) : strip_count(p, k), tg.g[nt], wg);
            wg = tg.g[nt++].wg_end;
            nbmax = nb > nbmax ? nb : nbmax;
        }
        if (!nd) return hipSuccess;
        hipError_t e2 = diag_lu_group(ST, dc, nd, s);
        if (e2) return e2;
        if (np) {
            // the steps on the inverse path: inverses, their parts, the strip products
            int wg0[3] = {0, 0, 0}, i = 0;
            for (int g = 0; g < count; ++g) {
                const FactorPlan& p = P[g];
                const int64_t k = t * p.nb;
                if (k >= p.n || !inverse_path(p, k)) continue;
                panel_desc(p, k, panel_rows(ST, pnbmax), pg.g[i], wg0);
                wg0[0] = pg.g[i].wg_inv; wg0[1] = pg.g[i].wg_split; wg0[2] = pg.g[i].wg_trsm;
                ++i;
            }
            pg.count = np;
            hipEvent_t pt = prof::begin(prof::TRSM, s);
            if ((e2 = block_inverses(pg, wg0[0], pnbmax, s))) return e2;
            if ((e2 = panel_split(ST, pg, wg0[1], pnbmax, s))) return e2;
            if ((e2 = panel_trsm(ST, OP, pg, wg0[2], pnbmax, s))) return e2;
            prof::end(pt, prof::TRSM, s, 0.0, 0.0);
        }
        if (!nt) return hipSuccess;
        tg.count = nt;
        hipEvent_t pt = prof::begin(prof::TRSM, s);
        k_trsm<ST, OP><<<wg, ST_THREADS, trsm_smem(nbmax, wg), s>>>(tg);
        prof::end(pt, prof::TRSM, s, 0.0, 0.0);
        return hipGetLastError();
    };
    auto gemms = [&](const GemmCall* gc, int ng) -> hipError_t {
        if (!ng) return hipSuccess;
        double fl = 0, by = 0;
        for (int i = 0; i < ng; ++i) {
            const double K = gc[i].K + gc[i].K2;
            fl += 2.0 * gc[i].M * (double)gc[i].N * K;
            by += 2.0 * gc[i].M * (double)gc[i].N * sizeof(ST_T) + (gc[i].M + gc[i].N) * K * sizeof(OP_T);
        }
        hipEvent_t pg = prof::begin(prof::GEMM, s);
        hipError_t e2 = gemm_group(OP, ST, P[0].gemm_tile, gc, ng, s);
        prof::end(pg, prof::GEMM, s, fl, by);
        return e2;
    };
    // the updates in pairs of steps, with the arithmetic of mxp_factor:
    // panel t, block column and row t+1 by step t alone, panel t+1, the rest
    // by steps t and t+1 in one pass
    for (int64_t t = 0; t < steps; t += 2) {
        if ((e = panels(t))) return e;
        GemmCall gc[GEMM_DESC_MAX];
        int ng = 0;
        for (int g = 0; g < count; ++g) {
            const FactorPlan& p = P[g];
            const int64_t b = (t + 1) * p.nb;
            if (b < p.n) ng += cross_calls<ST, OP>(p, t * p.nb, false, b, gc + ng);
        }
        if ((e = gemms(gc, ng))) return e;
        if ((e = panels(t + 1))) return e;
        ng = 0;
        for (int g = 0; g < count; ++g) {
            const FactorPlan& p = P[g];
            const int64_t b = (t + 2) * p.nb;
            if (b < p.n) gc[ng++] = pair_call<ST, OP>(p, t * p.nb, true, b, b, p.n - b, p.n - b);
        }
        if ((e = gemms(gc, ng))) return e;
    }
    return prec_inverses<ST>(P, count, s);
}

hipError_t factor_group(const FactorPlan* P, int count, hipStream_t s) {
    if (count < 1 || count > GEMM_GROUP_MAX) return hipErrorInvalidValue;
    for (int g = 1; g < count; ++g)
        if (P[g].update != P[0].update || P[g].store != P[0].store) return hipErrorInvalidValue;
    const int u = P[0].update, t = P[0].store;
    if (u == F32 && t == F32) return factor_group_typed<F32, F32>(P, count, s);
    if (u == F16 && t == F16) return factor_group_typed<F16, F16>(P, count, s);
    if (u == BF16 && t == BF16) return factor_group_typed<BF16, BF16>(P, count, s);
    if (u == F8 && t == F16) return factor_group_typed<F16, F8>(P, count, s);
    if (u == F8 && t == BF16) return factor_group_typed<BF16, F8>(P, count, s);
    if (u == F16 && t == F32) return factor_group_typed<F32, F16>(P, count, s);
    if (u == BF16 && t == F32) return factor_group_typed<F32, BF16>(P, count, s);
    return hipErrorInvalidValue;
}

hipError_t factor_run(const FactorPlan& p, hipStream_t s, Lookahead* la) {
    if (la) return factor_dispatch(p, s, la);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    Lookahead* L = nullptr;
    if ((e = lookahead_acquire(dev, &L))) return e;
    e = factor_dispatch(p, s, L);
    lookahead_release(dev, L);
    return e;
}

}  // namespace mxp
