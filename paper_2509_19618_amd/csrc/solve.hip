// solve.hip -- FP64 pieces of the GMRES-based refinement (paper:
// "Algorithmic Framework": the low-precision factors used as a left
// preconditioner, GMRES in 64-bit, at most 50 iterations).
//
// prec_apply: z = U^-1 L^-1 S v by block forward and backward substitution
// on the stored factor (FP64 arithmetic): the nb x nb diagonal blocks are
// applied through the full FP32 inverses kept by the factorisation, the
// off-diagonal panels are read in the storage format (L21 strips unscaled by
// their power-of-two factor); one dataflow kernel per triangular solve.
// Modified Gram-Schmidt, Givens rotations, the least-squares solve and the
// basis update are deterministic (fixed reduction orders).
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "prof.hpp"

namespace mxp {

__host__ __device__ static inline int64_t rup(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

// ================================================================ preconditioner
// ---------------------------------------------------------------- block substitution
// One kernel per triangular solve, every right-hand side at once (each
// right-hand side with its own flags).  Work-group = one strip of TS rows;
// strips are processed as a dataflow: a strip of block j accumulates the
// products of its rows of the off-diagonal factor with every dependency
// block's solution as soon as that block is published (flag `ready`),
// publishes its rows of the block right-hand side (its strip flag), and
// applies its rows of the FP32 inverse of the diagonal block once the strips
// those rows depend on have published theirs (the inverse is triangular:
// the strips above it in the block for L, below it for U); it then counts
// itself into the block's `ready`.  Forward (L): dependencies are the blocks
// before j, strips run in increasing order; backward (U): the blocks after
// j, strips in decreasing order.
//
// A work-group takes its position (right-hand side, strip) from a counter
// of the launch when it starts, not from its index, and every wait is on
// strips of earlier positions, so every wait is on work-groups that have
// started: the earliest unfinished one waits on none and runs to its end.
// The launch then always drains, whatever else holds the device: the
// hardware deals the indices out to the XCDs, each dispatching its share in
// order, and with other launches on other streams it can hold back a
// launch's remaining work-groups while that launch's resident ones spin.
// Each wait is still bounded and on expiry sets *err and lets the
// work-group exit.  All sums are taken in a fixed order (deterministic
// results).
#ifndef MXP_TRSV_TS
#define MXP_TRSV_TS 64
#endif
constexpr int TS = MXP_TRSV_TS;

// Values exchanged between work-groups (block solutions, block right-hand
// sides) are written and read with device-scope atomic accesses, which go to
// the device's coherence point instead of an XCD's L2.  A flag is raised
// after every wave's stores are released (sync_release) and a work-group
// barrier; a waiter that sees the flag reads after it (sync_acquire, then
// the barrier that lets its other threads read); see common.hpp.
MXP_DEV void put_shared(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
MXP_DEV double get_shared(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// v, treated as written at this point: arithmetic on prefetched registers
// cannot move above it (the compiler would otherwise unpack a load's result
// right after issuing it, which waits for the load)
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
MXP_DEV void pin4(u32x4v& v) { asm volatile("" : "+v"(v)); }
MXP_DEV void pin4f(f32x4v& v) { asm volatile("" : "+v"(v)); }

// element k of a 16-byte vector of storage values, taken from its 32-bit
// words (no access through a cast pointer, which would split the vector at
// its load)
template <int ST> MXP_DEV float u4_elem(const u32x4v& v, int k);
template <> MXP_DEV float u4_elem<F32>(const u32x4v& v, int k) {
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    return __uint_as_float(w[k]);
}
template <> MXP_DEV float u4_elem<F16>(const u32x4v& v, int k) {
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    const unsigned h = (k & 1) ? (w[k >> 1] >> 16) : (w[k >> 1] & 0xFFFFu);
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}
template <> MXP_DEV float u4_elem<BF16>(const u32x4v& v, int k) {
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
    return __uint_as_float((k & 1) ? (w[k >> 1] & 0xFFFF0000u) : (w[k >> 1] << 16));
}

// Bounded waits of one wave: until *flag >= target; until the cnt <= 64 flags
// f[0 .. cnt) are raised (one lane per flag).  False: expired here or anywhere
// (*err is looked at every 64 polls).
MXP_DEV bool wave_wait(const unsigned* f, int cnt, unsigned target, int* err) {
    const int l = threadIdx.x & 63;
    for (unsigned it = 0;; ++it) {
        const bool up = l >= cnt || __hip_atomic_load(f + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target;
        if (__all(up)) break;
        if ((it & 63) == 63 &&
            (it > (1u << 24) || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            if (l == 0) atomicOr(err, 1);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    sync_acquire();
    asm volatile("" ::: "memory");
    return true;
}

// A strip's step is a chain of round trips: the flag of the block before it,
// that block's solution, the strip's right-hand side to the others and theirs
// back, the solution out.  Each wave polls for itself (the loads that follow
// need no barrier before them), a whole diagonal block's panels are in
// registers when its flag is raised and are taken in one pass (one wait, one
// load of the solution, one reduction), both halves of the inverse's rows are
// loaded before the last wait and reduced together, and only the wave that
// stores waits for its stores.  Eight right-hand sides at n = 8192, BF16:
// 237 -> 219 us per solve; n = 600: 27 -> 23.5 us.  VEC: 16-byte aligned columns
// (else element loads).
template <int ST, bool LOWER, bool VEC>
__global__ __launch_bounds__(256, 2) void k_trsv(int64_t n, int nb, int db, const typename Store<ST>::T* __restrict__ A,
                                                 int64_t lda, const float* __restrict__ inv_all,
                                                 const float* __restrict__ lsc, int64_t nstrips32,
                                                 const double* __restrict__ scale, const double* __restrict__ rhs,
                                                 int64_t ld_rhs, double* __restrict__ tbuf, double* __restrict__ out,
                                                 int64_t ld_out, unsigned* flags, unsigned* other,
                                                 int64_t flag_stride, unsigned* ticket, unsigned* other_ticket,
                                                 int* err) {
    typedef typename Store<ST>::T T;
    constexpr int RPL = 16 / (int)sizeof(T);   // rows per lane: one 16-byte load
    constexpr int RG = TS / RPL;               // lanes per column
    constexpr int CPI = 64 / RG;               // columns per wave and load
    constexpr int HS = TS / 2, RQ = HS / 4, CS = 64 / RQ;   // diagonal apply: half strips, lanes per column, columns
    constexpr int PCOLS = CPI > CS ? CPI : CS;              // column groups of either
    static_assert(TS == 64, "a wave holds one value per row of a strip");
    constexpr int ZERO = 1024;                 // zs[ZERO] = 0: the weight of columns past a range
    __shared__ double zs[ZERO + 1];
    __shared__ double part[4][PCOLS][TS];
    __shared__ unsigned s_pos;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // position in start order: strip pos % S of right-hand side pos / S (the
    // grid is S x nrhs work-groups)
    if (tid == 0) {
        s_pos = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        zs[ZERO] = 0.0;
    }
    __syncthreads();
    const int64_t S = (n + TS - 1) / TS, J = (n + nb - 1) / nb;
    const int64_t pos = __builtin_amdgcn_readfirstlane((int)s_pos), py = __builtin_amdgcn_readfirstlane((int)((unsigned)pos / (unsigned)S)), px = pos - py * S;
    // right-hand side py: its own vectors, block buffer and flags
    rhs += py * ld_rhs;
    out += py * ld_out;
    tbuf += py * n;
    flags += py * flag_stride;
    other += py * flag_stride;
    // the flags and the counter of the other triangular solve, which is not
    // running, cleared for its next launch
    if (tid == 0) {
        __hip_atomic_store(other + px, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (px < J) __hip_atomic_store(other + S + px, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (pos == 0) __hip_atomic_store(other_ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the substitution's diagonal blocks (size db, a multiple of nb) are the
    // dataflow's steps
    const int64_t sidx = LOWER ? px : S - 1 - px;
    const int64_t j = __builtin_amdgcn_readfirstlane((int)((unsigned)sidx / (unsigned)(db / TS))), Jd = (n + db - 1) / db;
    const int64_t r0 = sidx * TS;
    const int rows = (int)(n - r0 < TS ? n - r0 : TS);
    unsigned* sflag = flags;          // one per strip: its rows of the block right-hand side are published
    unsigned* ready = flags + S;      // one per block: strips that have published their solution rows
    auto cols_of = [&](int64_t b) -> int { return (int)(n - b * db < db ? n - b * db : db); };
    auto strips_of = [&](int64_t b) -> unsigned { return (unsigned)((cols_of(b) + TS - 1) / TS); };
    // wave 0: the strip's rows, one per lane (the forward solve starts from S v)
    double w = 0.0;
    if (tid < rows) w = LOWER ? scale[r0 + tid] * rhs[r0 + tid] : rhs[r0 + tid];
    // The ragged last strip takes the same 16-byte loads: with 16-byte aligned
    // columns the rows up to lda may be read (its panel columns lie before the
    // last one), the lanes past lda re-read the strip's first rows, and the
    // sums of rows past n are dropped.  (Element loads, waited for one by one,
    // made that one strip the end of the forward solve: n = 20001 FP16 846 us
    // per solve against 312 us.)
    const int rg = lane % RG, cl = lane / RG;
    const int64_t rl = r0 + RPL * rg < lda ? r0 + RPL * rg : r0;   // first row this lane reads
    constexpr int PF = 16;                     // panel loads of one register set
    // The factor panels do not depend on the flags: a block's panel (each wave
    // a quarter of its columns, the first 2 PF loads of it) is loaded while the
    // block before it is awaited and applied, each register set as soon as it
    // is free.  The loads carry no condition (a column past the range reads
    // the block's first and is weighted zero below): a load under a branch
    // ends in a wait for every load in flight, which would serialise them.
    struct Quarter {
        int cb, ce;
    };
    auto quarter = [&](int64_t b) {
        const int kb = cols_of(b), q = (kb + 3) / 4;
        Quarter Q;
        Q.cb = wv * q < kb ? wv * q : kb;
        Q.ce = Q.cb + q < kb ? Q.cb + q : kb;
        return Q;
    };
    // a wave whose wait has expired (*err is set) waits no more and goes
    // through its steps: a way out of the loop would cost the registers that
    // hold the loads
    bool ok = true;
    double acc[RPL] = {};
    auto issue = [&](int64_t b, bool on, int m0, u32x4v* dst) {
        // a uniform base and 32-bit byte offsets (a block of 1024 columns spans
        // less than 4 GB for any matrix that fits the card)
        const Quarter Q = quarter(b);
        if (!VEC) return;
        const char* base = (const char*)(A + (int64_t)on * b * db * lda);
        const uint32_t ldb = (uint32_t)on * (uint32_t)(lda * sizeof(T)), row = (uint32_t)(rl * sizeof(T));
        // (opaque here: the columns of all loads would otherwise be computed
        // once and kept, which costs more registers than there are)
        int c0 = Q.cb + cl;
#pragma unroll
        for (int k = 0; k < RPL; ++k) asm volatile("" : "+v"(c0) : "v"(acc[k]));
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const int c = c0 + (m0 + m) * CPI;
            dst[m] = *(const u32x4v*)(base + (uint32_t)(c < Q.ce ? c : 0) * ldb + row);
        }
    };
    const int64_t bstep = LOWER ? 1 : -1;
    auto in_range = [&](int64_t b) { return LOWER ? b < j : b > j; };
    auto take = [&](const Quarter& Q, int m0, u32x4v* pre) {
        int c0 = Q.cb + cl;
        asm volatile("" : "+v"(c0));           // (see issue)
        if (!VEC) return;
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            pin4(pre[m]);
            const int c = c0 + (m0 + m) * CPI;
            const double zc = zs[c < Q.ce ? c : ZERO];
#pragma unroll
            for (int k = 0; k < RPL; ++k) acc[k] += (double)u4_elem<ST>(pre[m], k) * zc;
        }
    };
    {
        u32x4v pa[PF], pb[PF];
        int64_t b = LOWER ? 0 : Jd - 1;
        issue(b, in_range(b), 0, pa);
        issue(b, in_range(b), PF, pb);
        for (; in_range(b); b += bstep) {
            const Quarter Q = quarter(b);
            const int kb = cols_of(b);
            ok = ok && wave_wait(&ready[b], 1, strips_of(b), err);
            for (int c = tid; c < kb; c += 256) zs[c] = get_shared(out + b * db + c);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RPL; ++k) acc[k] = 0.0;
            const bool more = in_range(b + bstep);
            // (kept apart: overlapped, the registers of the old and of the new
            // loads would all be live)
            take(Q, 0, pa);
            __builtin_amdgcn_sched_barrier(0);
            issue(b + bstep, more, 0, pa);
            __builtin_amdgcn_sched_barrier(0);
            take(Q, PF, pb);
            __builtin_amdgcn_sched_barrier(0);
            issue(b + bstep, more, PF, pb);
            __builtin_amdgcn_sched_barrier(0);
            const T* base = A + rl + b * db * lda;
            if (VEC) {
#pragma unroll 4
                for (int c = Q.cb + cl + 2 * PF * CPI; c < Q.ce; c += CPI) {
                    const u32x4v v = *(const u32x4v*)(base + (int64_t)c * lda);
                    const T* e = (const T*)&v;
                    const double zc = zs[c];
#pragma unroll
                    for (int k = 0; k < RPL; ++k) acc[k] += (double)Store<ST>::load(e, k) * zc;
                }
            } else {
                for (int c = Q.cb + cl; c < Q.ce; c += CPI) {
                    const double zc = zs[c];
#pragma unroll
                    for (int k = 0; k < RPL; ++k)
                        if (RPL * rg + k < rows) acc[k] += (double)Store<ST>::load(base, (int64_t)c * lda + k) * zc;
                }
            }
            if (LOWER) {
                // stored strips carry a power of two per factor block and 32
                // rows; a dependency of the forward solve is a whole block, so
                // a wave's quarter lies in one factor block
                const int64_t i = b * (db / nb) + (int64_t)Q.cb / nb;
                const double us = 1.0 / (double)lsc[i * nstrips32 + (r0 + RPL * rg < n ? r0 + RPL * rg : r0) / 32];
#pragma unroll
                for (int k = 0; k < RPL; ++k) acc[k] *= us;
            }
#pragma unroll
            for (int k = 0; k < RPL; ++k) part[wv][cl][RPL * rg + k] = acc[k];
            __syncthreads();
            if (tid < TS) {
                double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int v2 = 0; v2 < CPI; ++v2)
#pragma unroll
                    for (int u = 0; u < 4; ++u) t[u] += part[u][v2][tid];
                w -= (t[0] + t[1]) + (t[2] + t[3]);
            }
        }
    }
    // this strip's rows of the block right-hand side are final (wave 0)
    if (wv == 0) {
        if (tid < rows) put_shared(tbuf + r0 + tid, w);
        sync_release();
        if (tid == 0) __hip_atomic_store(&sflag[sidx], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // The strip's rows of its diagonal-block inverse (lower / upper triangular:
    // a row takes the columns up to / from itself), in two half strips of HS
    // rows.  A lane: four consecutive rows (16-byte loads), one of CS column
    // groups; the waves split a half strip's columns.  The first loads of both
    // are issued while the strips they depend on publish.
    const int64_t cj = j * db;
    const int kbj = cols_of(j);
    const int nst = (int)strips_of(j);
    const int s_in = (int)((r0 - cj) / TS);
    const int rsub = lane % RQ, csub = lane / RQ;
    const float* blkinv = inv_all + j * (int64_t)db * db;
    struct Half {
        int r0, clo, cb, ce;
    };
    auto half = [&](int h) {
        Half H;
        H.r0 = HS * h < kbj ? HS * h : 0;                         // past the block: nothing is stored
        H.clo = LOWER ? 0 : H.r0;
        const int chi = LOWER ? (H.r0 + HS < kbj ? H.r0 + HS : kbj) : kbj;
        const int q = (chi - H.clo + 3) / 4;
        H.cb = H.clo + wv * q;
        H.ce = H.cb + q < chi ? H.cb + q : chi;
        return H;
    };
    const Half HA = half(2 * s_in), HB = half(2 * s_in + 1);
    constexpr int NIV = 16;               // inverse loads of a batch per lane (16 bytes each)
    auto load_inv = [&](const Half& H, int t0, f32x4v (&iv)[NIV]) {
        const uint32_t row = (uint32_t)(H.r0 + 4 * rsub) * 4u, ldb = (uint32_t)db * 4u;
#pragma unroll
        for (int t = 0; t < NIV; ++t) {
            const int c = H.cb + csub + CS * (t0 + t);
            iv[t] = *(const f32x4v*)((const char*)blkinv + (uint32_t)(c < H.ce ? c : H.clo) * ldb + row);
        }
    };
    f32x4v ia[NIV], ib[NIV];
    load_inv(HA, 0, ia);
    load_inv(HB, 0, ib);
    // the strips whose right-hand side rows this strip's rows take: those
    // above it in the block (L), below it (U)
    ok = ok && (LOWER ? wave_wait(sflag + sidx - s_in, s_in, 1u, err)
                      : wave_wait(sflag + sidx + 1, nst - 1 - s_in, 1u, err));
    {
        // this strip's own rows come from wave 0's registers
        const int own = s_in * TS, zlo = LOWER ? 0 : own + rows, zhi = LOWER ? own : kbj;
        for (int c = zlo + tid; c < zhi; c += 256) zs[c] = get_shared(tbuf + cj + c);
        if (tid < rows) zs[own + tid] = w;
    }
    __syncthreads();
    auto apply = [&](const Half& H, int h, f32x4v (&iv)[NIV]) {
        double a4[4] = {0.0, 0.0, 0.0, 0.0};
        for (int t0 = 0;;) {
#pragma unroll
            for (int t = 0; t < NIV; ++t) {
                pin4f(iv[t]);
                const int c = H.cb + csub + CS * (t0 + t);
                const double zc = zs[c < H.ce ? c : ZERO];
                a4[0] += (double)iv[t].x * zc;
                a4[1] += (double)iv[t].y * zc;
                a4[2] += (double)iv[t].z * zc;
                a4[3] += (double)iv[t].w * zc;
            }
            t0 += NIV;
            if (H.cb + CS * t0 >= H.ce) break;            // wave-uniform
            load_inv(H, t0, iv);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) part[wv][csub][HS * h + 4 * rsub + k] = a4[k];
    };
    apply(HA, 0, ia);
    apply(HB, 1, ib);
    __syncthreads();
    if (wv == 0) {
        if (tid < rows) {
            double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int v2 = 0; v2 < CS; ++v2)
#pragma unroll
                for (int u = 0; u < 4; ++u) t[u] += part[u][v2][tid];
            put_shared(out + r0 + tid, (t[0] + t[1]) + (t[2] + t[3]));
        }
        sync_release();
        if (tid == 0) __hip_atomic_fetch_add(&ready[j], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void k_zero_u32(unsigned* p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// flag words of one right-hand side: the strip flags (S = ceil(n / TS)) and
// block flags (J = ceil(n / nb), nb >= 64) of both solves; those of the
// first right-hand side also hold the two solves' start-order counters
// (words 2 (S + J) and 2 (S + J) + 1)
static int64_t trsv_flag_words(int64_t n) {
    constexpr int64_t u = TS < 64 ? TS : 64;
    return 4 * (n / u + 2);
}

size_t prec_work_bytes(int64_t n, int nr) {
    // forward solution, block right-hand sides (n x nr each), flags, error word
    return (size_t)(2 * n * nr) * 8 + (size_t)(trsv_flag_words(n) * nr) * 4 + 256;
}

static int* prec_err_word(double* W, int64_t n, int nr) {
    return (int*)((unsigned*)(W + 2 * n * nr) + trsv_flag_words(n) * nr);
}

// flags, counters and the error word: once before the applies with this n, nr
// (each solve then clears the other's)
hipError_t prec_reset(double* W, int64_t n, int nr, hipStream_t s) {
    const int64_t words = trsv_flag_words(n) * nr + 1;
    k_zero_u32<<<(unsigned)((words + 255) / 256), 256, 0, s>>>((unsigned*)(W + 2 * n * nr), words);
    return hipGetLastError();
}

hipError_t prec_err_read(double* W, int64_t n, int nr, int* err, hipStream_t s) {
    hipError_t e = hipMemcpyAsync(err, prec_err_word(W, n, nr), sizeof(int), hipMemcpyDeviceToHost, s);
    if (!e) e = hipStreamSynchronize(s);
    return e;
}

template <int ST>
static hipError_t prec_typed(const PrecPlan& p, const double* V, int64_t ldv, double* Z, int64_t ldz, int nr,
                             double* W, hipStream_t s) {
    typedef typename Store<ST>::T T;
    const int64_t n = p.n, nb = p.nb;
    const int64_t J = (n + nb - 1) / nb;
    const int64_t nstrips32 = (n + 31) / 32;
    const int64_t S = (n + TS - 1) / TS;
    double* Y = W;                 // forward solutions, nr columns (ld n)
    double* Tb = Y + n * nr;       // block right-hand sides
    unsigned* flags = (unsigned*)(Tb + n * nr);
    const int64_t fw = trsv_flag_words(n);
    int* err = prec_err_word(W, n, nr);
    const bool vec = ((p.lda * (int64_t)sizeof(T)) % 16 == 0 && ((uintptr_t)p.A) % 16 == 0);
    unsigned *fl = flags, *fu = flags + S + J, *tk = flags + 2 * (S + J);
    const int db = (int)prec_block(nb);
    const dim3 grid((unsigned)S, (unsigned)nr);
    hipEvent_t pt = prof::begin(prof::PREC, s);
    auto solves = [&](auto VEC) {
        constexpr bool V16 = decltype(VEC)::value;
        k_trsv<ST, true, V16><<<grid, 256, 0, s>>>(n, (int)nb, db, (const T*)p.A, p.lda, p.linv_full, p.lsc, nstrips32,
                                                   p.rowscale, V, ldv, Tb, Y, n, fl, fu, fw, tk, tk + 1, err);
        k_trsv<ST, false, V16><<<grid, 256, 0, s>>>(n, (int)nb, db, (const T*)p.A, p.lda, p.uinv_full, nullptr,
                                                    nstrips32, nullptr, Y, n, Tb, Z, ldz, fu, fl, fw, tk + 1, tk, err);
    };
    if (vec)
        solves(std::true_type{});
    else
        solves(std::false_type{});
    prof::end(pt, prof::PREC, s, 2.0 * n * (double)n * nr, (double)n * n * sizeof(T) + 8.0 * n * nb);
    return hipGetLastError();
}

hipError_t prec_apply(const PrecPlan& p, const double* V, int64_t ldv, double* Z, int64_t ldz, int nr, double* W,
                      hipStream_t s) {
    switch (p.store) {
    case F32: return prec_typed<F32>(p, V, ldv, Z, ldz, nr, W, s);
    case F16: return prec_typed<F16>(p, V, ldv, Z, ldz, nr, W, s);
    case BF16: return prec_typed<BF16>(p, V, ldv, Z, ldz, nr, W, s);
    default: return hipErrorInvalidValue;
    }
}

// ================================================================ GMRES vector kernels
// Every right-hand side runs its own GMRES in lockstep with the others:
// blockIdx.y (or the thread index of the scalar kernels) is the right-hand
// side r, and act[r] says whether r takes part in the current step (the
// others' blocks return at once).  Every reduction gives block b the fixed
// index range [b*chunk, (b+1)*chunk) and sums it in a fixed order, so
// results are identical from run to run.
int red_blocks(int64_t n) {
    int64_t b = (n + 4095) / 4096;
    if (b > 256) b = 256;
    if (b < 1) b = 1;
    return (int)b;
}

__device__ __forceinline__ double block_sum(double v, double* red) {
    v = warp_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return t;
}

__device__ __forceinline__ double sum_parts(const double* part, int nparts, double* red) {
    double v = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) v += part[i];
    return block_sum(v, red);
}

// part[r][b] = sum over block b's range of x_r . y_r
__global__ __launch_bounds__(256) void k_dot_part(int64_t n, int64_t chunk, const double* __restrict__ x, int64_t ldx,
                                                  const double* __restrict__ y, int64_t ldy, double* __restrict__ part,
                                                  const int* __restrict__ act) {
    __shared__ double red[4];
    const int r = blockIdx.y;
    if (!act[r]) return;
    x += r * ldx;
    y += r * ldy;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = i0 + chunk < n ? i0 + chunk : n;
    double v = 0.0;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) v += x[i] * y[i];
    v = block_sum(v, red);
    if (threadIdx.x == 0) part[r * 256 + blockIdx.x] = v;
}

// MGS step j of column k: h_jk = sum(part_in); w -= h_jk v_j over the
// block's range; then the partial dot for the next vector (v_{j+1} . w, or
// w . w after the last one).  V: basis vectors v_{r,j} at V + (j nr + r) n.
__global__ __launch_bounds__(256) void k_mgs(int64_t n, int64_t chunk, int nr, const double* __restrict__ V, int j,
                                             int last, double* __restrict__ W, const double* __restrict__ part_in,
                                             double* __restrict__ part_out, double* __restrict__ H, int ldh, int k,
                                             const int* __restrict__ act) {
    __shared__ double red[4];
    const int r = blockIdx.y;
    if (!act[r]) return;
    const double* vj = V + ((int64_t)j * nr + r) * n;
    const double* vnext = last ? nullptr : V + ((int64_t)(j + 1) * nr + r) * n;
    double* w = W + (int64_t)r * n;
    const double h = sum_parts(part_in + r * 256, gridDim.x, red);
    if (blockIdx.x == 0 && threadIdx.x == 0) H[(int64_t)r * ldh * (ldh - 1) + j + (int64_t)k * ldh] = h;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = i0 + chunk < n ? i0 + chunk : n;
    double v = 0.0;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const double wi = w[i] - h * vj[i];
        w[i] = wi;
        v += (vnext ? vnext[i] : wi) * wi;
    }
    v = block_sum(v, red);
    if (threadIdx.x == 0) part_out[r * 256 + blockIdx.x] = v;
}

// h = sqrt(sum(part)); H[k+1][k] = h; v_{k+1} = w / h (0 on exact breakdown)
__global__ __launch_bounds__(256) void k_normalize(int64_t n, int64_t chunk, int nr, const double* __restrict__ part,
                                                   const double* __restrict__ W, double* __restrict__ V, int k,
                                                   double* __restrict__ H, int ldh, const int* __restrict__ act) {
    __shared__ double red[4];
    const int r = blockIdx.y;
    if (!act[r]) return;
    const double h = sqrt(sum_parts(part + r * 256, gridDim.x, red));
    if (blockIdx.x == 0 && threadIdx.x == 0) H[(int64_t)r * ldh * (ldh - 1) + (k + 1) + (int64_t)k * ldh] = h;
    const double* w = W + (int64_t)r * n;
    double* v = V + ((int64_t)(k + 1) * nr + r) * n;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = i0 + chunk < n ? i0 + chunk : n;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) v[i] = (h > 0.0) ? w[i] / h : 0.0;
}

// out[r] = sqrt(sum(part[r]))
__global__ __launch_bounds__(256) void k_norm_final(const double* __restrict__ part, int nparts, double* out,
                                                    int out_stride, const int* __restrict__ act) {
    __shared__ double red[4];
    const int r = blockIdx.x;
    if (!act[r]) return;
    const double v = sum_parts(part + r * 256, nparts, red);
    if (threadIdx.x == 0) out[r * out_stride] = sqrt(v);
}

// v_{r,0} = z_r / beta_r; g_r = beta_r e_1
__global__ __launch_bounds__(256) void k_start_basis(int64_t n, const double* __restrict__ Z, const double* sc,
                                                     int sc_stride, double* __restrict__ V, int nr,
                                                     double* __restrict__ g, int ldg, const int* __restrict__ act) {
    const int r = blockIdx.y;
    if (!act[r]) return;
    const double b = sc[r * sc_stride];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < ldg) g[r * ldg + threadIdx.x] = threadIdx.x == 0 ? b : 0.0;
    if (i < n) V[(int64_t)r * n + i] = (b > 0.0) ? Z[(int64_t)r * n + i] / b : 0.0;
}

// Column k of each active H_r (column-major, ldh = m + 1): apply rotations
// 0..k-1, form rotation k that zeroes H[k+1][k], rotate g.  flag[r] = 1 when
// |g[k+1]| <= tau ||x_r|| or H[k+1][k] was 0 (exact breakdown).
MXP_DEV void givens_column(int r, int k, double* H, int ldh, double* cs, double* sn, double* g, const double* sc,
                           int sc_stride, double tau, int* flag) {
    double* h = H + (int64_t)r * ldh * (ldh - 1) + (int64_t)k * ldh;
    double* c_ = cs + r * ldh;
    double* s_ = sn + r * ldh;
    double* gr = g + r * ldh;
    const double hsub = h[k + 1];
    for (int i = 0; i < k; ++i) {
        const double a = h[i], b = h[i + 1];
        h[i] = c_[i] * a + s_[i] * b;
        h[i + 1] = -s_[i] * a + c_[i] * b;
    }
    const double a = h[k], b = h[k + 1];
    const double rho = hypot(a, b);
    const double c = (rho > 0.0) ? a / rho : 1.0, s = (rho > 0.0) ? b / rho : 0.0;
    c_[k] = c;
    s_[k] = s;
    h[k] = rho;
    h[k + 1] = 0.0;
    const double gk = gr[k];
    gr[k + 1] = -s * gk;
    gr[k] = c * gk;
    const double xnorm = sc[r * sc_stride];
    flag[r] = (fabs(gr[k + 1]) <= tau * xnorm || hsub == 0.0) ? 1 : 0;
}

__global__ void k_givens(int nr, int k, double* H, int ldh, double* cs, double* sn, double* g,
                         const double* sc, int sc_stride, double tau, int* flag, const int* __restrict__ act) {
    const int r = threadIdx.x;
    if (r < nr && act[r]) givens_column(r, k, H, ldh, cs, sn, g, sc, sc_stride, tau, flag);
}

// A whole Arnoldi step and its rotation for sizes whose sums are one block's
// (n <= 4096): k_dot_part, the k_mgs, k_normalize and k_givens of column k in
// one launch, the new vector in registers (same order of every sum).  At these
// sizes a launch (4-5 us) costs more than its work: n = 600, 100 us per step
// in k + 4 launches before.
constexpr int ONE_U = 16;      // elements per thread
__global__ __launch_bounds__(256) void k_arnoldi_one(int64_t n, int nr, double* __restrict__ V, int k,
                                                     const double* __restrict__ W, double* H, int ldh, double* cs,
                                                     double* sn, double* g, const double* sc, int sc_stride,
                                                     double tau, int* flag, const int* __restrict__ act) {
    __shared__ double red[4];
    const int r = blockIdx.x, tid = threadIdx.x;
    if (!act[r]) return;
    double* Hk = H + (int64_t)r * ldh * (ldh - 1) + (int64_t)k * ldh;
    const double* w = W + (int64_t)r * n;
    auto vec = [&](int j) -> double* { return V + ((int64_t)j * nr + r) * n; };
    double x[ONE_U], v[ONE_U], sum = 0.0;
    auto load = [&](const double* p, double (&d)[ONE_U]) {
#pragma unroll
        for (int u = 0; u < ONE_U; ++u) {
            const int i = tid + 256 * u;
            d[u] = i < n ? p[i] : 0.0;
        }
    };
    load(w, x);
    load(vec(0), v);
#pragma unroll
    for (int u = 0; u < ONE_U; ++u) sum += v[u] * x[u];
    double h = block_sum(sum, red);
    for (int j = 0; j <= k; ++j) {
        if (tid == 0) Hk[j] = h;
#pragma unroll
        for (int u = 0; u < ONE_U; ++u) x[u] -= h * v[u];
        if (j < k) load(vec(j + 1), v);
        sum = 0.0;
#pragma unroll
        for (int u = 0; u < ONE_U; ++u) sum += (j < k ? v[u] : x[u]) * x[u];
        h = block_sum(sum, red);
    }
    h = sqrt(h);
    if (tid == 0) Hk[k + 1] = h;
    double* vk = vec(k + 1);
#pragma unroll
    for (int u = 0; u < ONE_U; ++u) {
        const int i = tid + 256 * u;
        if (i < n) vk[i] = (h > 0.0) ? x[u] / h : 0.0;
    }
    if (tid == 0) givens_column(r, k, H, ldh, cs, sn, g, sc, sc_stride, tau, flag);
}

// y_r = R_r^-1 g_r (R_r = rotated H_r[0:k_r, 0:k_r]), k_r = kdim[r]
__global__ void k_backsub(int nr, const double* H, int ldh, const double* g, double* y, const int* kdim) {
    const int r = threadIdx.x;
    if (r >= nr) return;
    const int k = kdim[r];
    const double* Hr = H + (int64_t)r * ldh * (ldh - 1);
    const double* gr = g + r * ldh;
    double* yr = y + r * ldh;
    for (int i = k - 1; i >= 0; --i) {
        double t = gr[i];
        for (int l = i + 1; l < k; ++l) t -= Hr[i + (int64_t)l * ldh] * yr[l];
        yr[i] = t / Hr[i + (int64_t)i * ldh];
    }
}

// x_r += V_r[:, 0:k_r] y_r
__global__ __launch_bounds__(256) void k_axpy_basis(int64_t n, int nr, const double* __restrict__ V,
                                                    const double* __restrict__ y, int ldy, const int* kdim,
                                                    double* __restrict__ X, int64_t ldx) {
    const int r = blockIdx.y;
    const int k = kdim[r];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n || k == 0) return;
    double acc = 0.0;
    for (int j = 0; j < k; ++j) acc += y[r * ldy + j] * V[((int64_t)j * nr + r) * n + i];
    X[r * ldx + i] += acc;
}

__global__ void k_set_i32(int* p, int n, const int* src) {
    const int i = threadIdx.x;
    if (i < n) p[i] = src ? src[i] : 0;
}

// ---- host wrappers (all right-hand sides at once; V is (m + 1) x nr x n)
hipError_t gm_norms(int64_t n, int nr, const double* X, int64_t ldx, double* out, int out_stride, double* part,
                    const int* act, hipStream_t s) {
    const int nbk = red_blocks(n);
    const int64_t chunk = (n + nbk - 1) / nbk;
    k_dot_part<<<dim3(nbk, nr), 256, 0, s>>>(n, chunk, X, ldx, X, ldx, part, act);
    k_norm_final<<<nr, 256, 0, s>>>(part, nbk, out, out_stride, act);
    return hipGetLastError();
}

hipError_t gm_start(int64_t n, int nr, const double* Z, const double* sc, int sc_stride, double* V, double* g,
                    int ldg, const int* act, hipStream_t s) {
    k_start_basis<<<dim3((unsigned)((n + 255) / 256), nr), 256, 0, s>>>(n, Z, sc, sc_stride, V, nr, g, ldg, act);
    return hipGetLastError();
}

hipError_t gm_arnoldi(int64_t n, int nr, double* V, int k, double* W, double* part, double* H, int ldh, double* cs,
                      double* sn, double* g, const double* sc, int sc_stride, double tau, int* flag, const int* act,
                      hipStream_t s) {
    const int nbk = red_blocks(n);
    if (nbk == 1 && n <= 256 * ONE_U) {
        k_arnoldi_one<<<nr, 256, 0, s>>>(n, nr, V, k, W, H, ldh, cs, sn, g, sc, sc_stride, tau, flag, act);
        return hipGetLastError();
    }
    const int64_t chunk = (n + nbk - 1) / nbk;
    k_dot_part<<<dim3(nbk, nr), 256, 0, s>>>(n, chunk, V, n, W, n, part, act);
    for (int j = 0; j <= k; ++j) {
        const double* pin = part + (j & 1) * 256 * nr;
        double* pout = part + ((j + 1) & 1) * 256 * nr;
        k_mgs<<<dim3(nbk, nr), 256, 0, s>>>(n, chunk, nr, V, j, j == k, W, pin, pout, H, ldh, k, act);
    }
    k_normalize<<<dim3(nbk, nr), 256, 0, s>>>(n, chunk, nr, part + ((k + 1) & 1) * 256 * nr, W, V, k, H, ldh, act);
    k_givens<<<1, 64, 0, s>>>(nr, k, H, ldh, cs, sn, g, sc, sc_stride, tau, flag, act);
    return hipGetLastError();
}

hipError_t gm_update(int64_t n, int nr, const double* H, int ldh, const double* g, double* y, const int* kdim,
                     const double* V, double* X, int64_t ldx, hipStream_t s) {
    k_backsub<<<1, 64, 0, s>>>(nr, H, ldh, g, y, kdim);
    k_axpy_basis<<<dim3((unsigned)((n + 255) / 256), nr), 256, 0, s>>>(n, nr, V, y, ldh, kdim, X, ldx);
    return hipGetLastError();
}

hipError_t set_i32(int* dst, int n, const int* src_dev, hipStream_t s) {
    k_set_i32<<<1, 64, 0, s>>>(dst, n, src_dev);
    return hipGetLastError();
}

}  // namespace mxp
