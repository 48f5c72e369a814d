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
// right-hand side with its own exchange buffers).  Work-group = one strip of
// TS rows; strips are processed as a dataflow: a strip of block j accumulates
// the products of its rows of the off-diagonal factor with every dependency
// block's solution as soon as that is there (`out`), publishes its rows of the
// block right-hand side (`tbuf`), applies its rows of the FP32 inverse of the
// diagonal block once the rows they take are there (the inverse is triangular:
// the strips above it in the block for L, below it for U), and publishes its
// rows of the solution.  Forward (L): dependencies are the blocks before j,
// strips run in increasing order; backward (U): the blocks after j, strips in
// decreasing order.
//
// A work-group takes its position (right-hand side, strip) from a counter
// of the launch when it starts, not from its index, and every wait is on
// strips of earlier positions, so every wait is on work-groups that have
// started: the earliest unfinished one waits on none and runs to its end.
// The launch then always drains, whatever else holds the device: the
// hardware deals the indices out to the XCDs, each dispatching its share in
// order, and with other launches on other streams it can hold back a
// launch's remaining work-groups while that launch's resident ones spin.
// Each wait is still bounded; on expiry it sets *err and the work-group goes
// through its remaining steps without waiting.  All sums are taken in a fixed
// order (deterministic results).
constexpr int TS = 64;

// Values exchanged between work-groups (block solutions, block right-hand
// sides) are written and read with device-scope atomic accesses, which go to
// the device's coherence point instead of an XCD's L2.
MXP_DEV double get_shared(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// v, treated as written at this point: arithmetic on prefetched registers
// cannot move above it (the compiler would otherwise unpack a load's result
// right after issuing it, which waits for the load)
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
MXP_DEV void pin4(u32x4v& v) { asm volatile("" : "+v"(v)); }

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

// A step of the substitution is a chain of exchanges between work-groups: the
// block's solution to every strip of the next block, and the strips' right-hand
// side rows among each other.  A value is its own flag: the exchange buffers
// hold UNSET (a NaN no computation gives, put_value) until the value is
// written, so an exchange is one store and one load that sees it, not a store,
// its acknowledgement, a flag, the flag's load and the value's load.
constexpr unsigned long long UNSET = 0x7FF8D15EA5EDF1A6ull;
MXP_DEV void put_value(double* p, double v) {
    unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    if (u == UNSET) u ^= 1ull;
    __hip_atomic_store((unsigned long long*)p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
MXP_DEV void put_unset(double* p) {
    __hip_atomic_store((unsigned long long*)p, UNSET, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
MXP_DEV bool is_set(double v) { return __builtin_bit_cast(unsigned long long, v) != UNSET; }

// Bounded waits of one wave for the values p[c], p[c + 64] of its lanes (those
// below cnt; the others are given 0).  far: a value several steps away is
// looked for with one address per wave (the last) before all are.  False:
// expired here or anywhere (*err is looked at every 64 polls).
MXP_DEV bool wait_values(const double* p, int cnt, bool far, double& v0, double& v1, int* err) {
    const int l = threadIdx.x & 63;
    v0 = v1 = 0.0;
    if (cnt <= 0) return true;
    for (unsigned it = 0;; ++it) {
        bool up = true;
        if (far) {
            up = is_set(get_shared(p + cnt - 1));
            if (__all(up)) { far = false; continue; }
        } else {
            if (l < cnt) v0 = get_shared(p + l);
            if (l + 64 < cnt) v1 = get_shared(p + l + 64);
            up = is_set(v0) && is_set(v1);
            if (__all(up)) return true;
        }
        if ((it & 63) == 63 &&
            (it > (1u << 24) || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
            if (l == 0) atomicOr(err, 1);
            return false;
        }
        if (far) __builtin_amdgcn_s_sleep(4);
        else __builtin_amdgcn_s_sleep(1);
    }
}

// a wave's LDS stores before its lanes' loads (LDS operations of a wave are in order)
MXP_DEV void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// x, y of every lane -> lanes below 32: x + x of lane + 32, lanes above: y + y
// of lane - 32 (fold32); the same between the 16-lane rows of each half
// (fold16) and the 8-lane halves of each row (fold8): log2 steps of a sum over
// lanes in which each lane ends with the sums of its own rows
MXP_DEV double join(unsigned lo, unsigned hi) { return __hiloint2double((int)hi, (int)lo); }
MXP_DEV double fold32(double x, double y) {
    const auto a = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return join(a[0], b[0]) + join(a[1], b[1]);
}
MXP_DEV double fold16(double x, double y) {
    const auto a = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto b = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return join(a[0], b[0]) + join(a[1], b[1]);
}
MXP_DEV double fold8(double x, double y) {
    const bool up = threadIdx.x & 8;
    const double keep = up ? y : x, give = up ? x : y;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(give), 0x128, 0xF, 0xF, true);   // row_ror:8
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(give), 0x128, 0xF, 0xF, true);
    return keep + __hiloint2double(hi, lo);
}

// What bounds a solve: the chain of exchanges, about 7 us per block of 1024
// columns at n = 8192; at n = 32768 also the panels' bytes (one factor half,
// 1.07 GB, in 318 us: 3.4 TB/s).  Eight waves per strip
// and at most 128 registers: two waves per SIMD also where a CU holds one
// strip (one wave issues an instruction every 8 cycles at most, two nearly
// twice as many) and four where it holds two.
//   a block's panel: each wave an eighth of the columns, in registers before the
//   block's solution is there (with FP32 storage half of it), taken in one pass;
//   the next block's loads, at the last block the inverse's, take their place.
//   A wave waits only for the solution values of its own columns.
// The loads that fill a set of registers are issued as one group with the
// panel's scale factor first: a later load in the chain would wait for them all
// (loads return in order).
// Per solve, against four waves per strip with a flag per exchange: n = 32768
// FP16 610 -> 318 us, n = 20001 FP16 312 -> 173, n = 8192 BF16 with eight
// right-hand sides 219 -> 122, n = 600 BF16 23.5 -> 14.2.
template <int ST, bool LOWER, bool VEC>
__global__ __launch_bounds__(512, 4) void k_trsv(int64_t n, int nb, int db, const typename Store<ST>::T* __restrict__ A,
                                                 int64_t lda, const float* __restrict__ inv_all,
                                                 const float* __restrict__ lsc, int64_t nstrips32,
                                                 const double* __restrict__ scale, const double* rhs, int64_t ld_rhs,
                                                 double* tbuf, double* out, double* other_tbuf, double* other_out,
                                                 double* zout, int64_t ld_z, unsigned* ticket, unsigned* other_ticket,
                                                 int* err) {
    typedef typename Store<ST>::T T;
    constexpr int RPL = 16 / (int)sizeof(T);   // rows per lane: one 16-byte load
    constexpr int RG = TS / RPL;               // lanes per column
    constexpr int CPI = 64 / RG;               // columns per wave and load
    constexpr int RQ = TS / 4, CS = 64 / RQ;   // the inverse (FP32): lanes per column, columns per wave and load
    constexpr int NW = 8, WC = 128;            // waves; columns of a wave at most (blocks have at most 1024)
    constexpr int PF = 16;                     // loads of one group
    constexpr int PH = WC / (CPI * PF);        // groups of a panel
    static_assert(TS == 64 && (RPL == 4 || RPL == 8), "a wave holds one value per row of a strip");
    __shared__ double zs[NW][WC];              // each wave's weights
    __shared__ double part[2][NW][TS];
    __shared__ double own[TS];
    __shared__ unsigned s_pos;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // position in start order: strip pos % S of right-hand side pos / S (the
    // grid is S x nrhs work-groups)
    if (tid == 0) s_pos = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int64_t S = (n + TS - 1) / TS;
    const int64_t pos = __builtin_amdgcn_readfirstlane((int)s_pos);
    const int64_t py = __builtin_amdgcn_readfirstlane((int)((unsigned)pos / (unsigned)S)), px = pos - py * S;
    // right-hand side py: its own vectors and exchange buffers
    rhs += py * ld_rhs;
    out += py * n;
    tbuf += py * n;
    // the substitution's diagonal blocks (size db, a multiple of nb) are the
    // dataflow's steps
    const int64_t sidx = LOWER ? px : S - 1 - px;
    const int64_t j = __builtin_amdgcn_readfirstlane((int)((unsigned)sidx / (unsigned)(db / TS)));
    const int64_t Jd = (n + db - 1) / db, r0 = sidx * TS;
    const int rows = (int)(n - r0 < TS ? n - r0 : TS);
    auto cols_of = [&](int64_t b) -> int { return (int)(n - b * db < db ? n - b * db : db); };
    // wave 0: the strip's rows, one per lane (the forward solve starts from S v).
    // The buffers of the other triangular solve, which is not running, are
    // cleared for its next launch (the backward solve's right-hand side is the
    // forward solve's `out`: read first).
    double w = 0.0;
    if (tid < rows) {
        w = LOWER ? scale[r0 + tid] * rhs[r0 + tid] : rhs[r0 + tid];
        asm volatile("" : "+v"(w) : : "memory");
        put_unset(other_tbuf + py * n + r0 + tid);
        put_unset(other_out + py * n + r0 + tid);
    }
    if (pos == 0 && tid == 0) __hip_atomic_store(other_ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // The ragged last strip takes the same 16-byte loads: with 16-byte aligned
    // columns the rows up to lda may be read (its panel columns lie before the
    // last one), the lanes past lda re-read the strip's first rows, and the
    // sums of rows past n are dropped.  (Element loads, waited for one by one,
    // made that one strip the end of the forward solve: n = 20001 FP16 846 us
    // per solve against 312 us.)
    const int rg = lane % RG, cl = lane / RG;
    const int64_t rl = r0 + RPL * rg < lda ? r0 + RPL * rg : r0;   // first row this lane reads
    const int rsub = lane % RQ, csub = lane / RQ;
    // the rows whose sums the lane ends with (reduce below)
    const int prow = RPL == 8 ? 8 * rg + (lane >> 3 & 1) + 2 * (lane >> 4 & 1) + 4 * (lane >> 5)
                              : 4 * rg + (lane >> 4 & 1) + 2 * (lane >> 5);
    const int irow = 4 * rsub + (lane >> 4 & 1) + 2 * (lane >> 5);
    // a wave's columns [cb, cb + cnt) of block b / of the strip's rows of the
    // diagonal block's inverse (lower / upper triangular: a row takes the
    // columns up to / from itself)
    struct Cols {
        int cb, cnt;
    };
    auto share = [&](int lo, int hi) {
        const int q = (hi - lo + NW - 1) / NW, cb = lo + wv * q;
        Cols C;
        C.cb = cb < hi ? cb : lo;
        C.cnt = cb < hi ? (cb + q < hi ? q : hi - cb) : 0;
        return C;
    };
    const int64_t cj = j * db;
    const int kbj = cols_of(j), ro = (int)(r0 - cj);      // the strip's first row in its block
    const Cols CI = LOWER ? share(0, ro + TS < kbj ? ro + TS : kbj) : share(ro, kbj);
    const float* blkinv = inv_all + j * (int64_t)db * db;
    // Loads carry no condition (a column past the range re-reads the first and
    // has the weight zero): a load under a branch ends in a wait for every load
    // in flight, which would serialise them.  A uniform base and 32-bit byte
    // offsets: VEC only where the 128 columns of a wave span at most 4 GB.
    u32x4v pre[PF];
    double acc[RPL] = {};
    float us = 1.0f;
    // (the weights of a whole group at once would not fit the registers either)
    auto pin_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < RPL; ++k) asm volatile("" : "+v"(acc[k]));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load_group = [&](const char* base, uint32_t ldb, uint32_t row, int c0, int cnt, int step) __attribute__((always_inline)) {
        // (opaque: the columns of all loads would otherwise be kept, which costs
        // more registers than there are; and not before acc is final)
#pragma unroll
        for (int k = 0; k < RPL; ++k) asm volatile("" : "+v"(c0) : "v"(acc[k]));
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const int c = c0 + m * step;
            pre[m] = *(const u32x4v*)(base + (uint32_t)(c < cnt ? c : 0) * ldb + row);
        }
    };
    auto load_inverse = [&](int c0) __attribute__((always_inline)) {
        load_group((const char*)(blkinv + (int64_t)CI.cb * db), (uint32_t)db * 4u, (uint32_t)(ro + 4 * rsub) * 4u,
                   csub + c0, CI.cnt, CS);
    };
    // group ph of block b's panel, or (on false) the first of the inverse:
    // chosen by value, since a branch around the loads would cost a copy of
    // their registers
    auto load_next = [&](int64_t b, bool on, int ph) __attribute__((always_inline)) {
        const Cols C = share(0, cols_of(on ? b : 0));
        if (LOWER && ph == 0) {
            // stored strips carry a power of two per factor block and 32 rows; a
            // dependency of the forward solve is a whole block, so a wave's
            // columns lie in one factor block
            const int64_t i = (on ? b : 0) * (db / nb) + (int64_t)C.cb / nb;
            us = lsc[i * nstrips32 + (r0 + prow < n ? r0 + prow : r0) / 32];
        }
        const bool pan = VEC && on;
        const int64_t off = pan ? (int64_t)(uintptr_t)(A + (b * db + C.cb) * lda)
                                : (int64_t)(uintptr_t)(blkinv + (int64_t)CI.cb * db);
        load_group((const char*)(uintptr_t)off, pan ? (uint32_t)(lda * sizeof(T)) : (uint32_t)db * 4u,
                   pan ? (uint32_t)(rl * sizeof(T)) : (uint32_t)(ro + 4 * rsub) * 4u,
                   (pan ? cl : csub) + ph * PF * CPI, pan ? C.cnt : CI.cnt, pan ? CPI : CS);
    };
    const int64_t bstep = LOWER ? 1 : -1;
    auto in_range = [&](int64_t b) { return LOWER ? b < j : b > j; };
    // a wave whose wait has expired (*err is set) waits no more and goes
    // through its steps: a way out of the loop would cost the registers that
    // hold the loads
    bool ok = true;
    int pb = 0;
    int64_t b = LOWER ? 0 : Jd - 1;
    load_next(b, in_range(b), 0);
    for (; in_range(b); b += bstep) {
        const Cols C = share(0, cols_of(b));
        const bool more = in_range(b + bstep);
        double v0 = 0.0, v1 = 0.0;
        if (ok) ok = wait_values(out + b * db + C.cb, C.cnt, more, v0, v1, err);
        zs[wv][lane] = v0;
        zs[wv][lane + 64] = v1;
        wave_sync();
        if (!more) __builtin_amdgcn_s_setprio(2);
        const float usb = us;
#pragma unroll
        for (int k = 0; k < RPL; ++k) acc[k] = 0.0;
        if (VEC) {
#pragma unroll
            for (int ph = 0; ph < PH; ++ph) {
#pragma unroll
                for (int m = 0; m < PF; ++m) {
                    pin4(pre[m]);
                    const double zc = zs[wv][cl + (ph * PF + m) * CPI];
#pragma unroll
                    for (int k = 0; k < RPL; ++k) acc[k] += (double)u4_elem<ST>(pre[m], k) * zc;
                    if (m % 4 == 3) pin_sums();
                }
                if (ph + 1 < PH) load_next(b, true, ph + 1);
            }
        } else {
            const T* base = A + rl + (b * db + C.cb) * lda;
            for (int c = cl; c < C.cnt; c += CPI) {
                const double zc = zs[wv][c];
#pragma unroll
                for (int k = 0; k < RPL; ++k)
                    if (RPL * rg + k < rows) acc[k] += (double)Store<ST>::load(base, (int64_t)c * lda + k) * zc;
            }
        }
        load_next(b + bstep, more, 0);
        __builtin_amdgcn_sched_barrier(0);
        double r;
        if constexpr (RPL == 8)
            r = fold8(fold16(fold32(acc[0], acc[4]), fold32(acc[2], acc[6])),
                      fold16(fold32(acc[1], acc[5]), fold32(acc[3], acc[7])));
        else
            r = fold16(fold32(acc[0], acc[2]), fold32(acc[1], acc[3]));
        part[pb][wv][prow] = LOWER ? r * (1.0 / (double)usb) : r;
        __syncthreads();
        if (wv == 0) {
            double t[NW];
#pragma unroll
            for (int u = 0; u < NW; ++u) t[u] = part[pb][u][lane];
            w -= ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        }
        pb ^= 1;
    }
    __builtin_amdgcn_s_setprio(2);
    // this strip's rows of the block right-hand side are final (wave 0)
    if (wv == 0) {
        if (tid < rows) put_value(tbuf + r0 + tid, w);
        own[tid] = w;
    }
    // Its rows of the inverse: each wave waits for the rows of its columns (its
    // own strip's come from wave 0)
    {
        const int lim = LOWER ? ro : ro + rows;           // others' rows: below lim (L), from lim (U)
        const int lo = LOWER ? CI.cb : (CI.cb > lim ? CI.cb : lim);
        const int hi = LOWER ? (CI.cb + CI.cnt < lim ? CI.cb + CI.cnt : lim) : CI.cb + CI.cnt;
        const int off = lo - CI.cb;                       // of the awaited range in the wave's columns
        double v0 = 0.0, v1 = 0.0;
        if (ok) ok = wait_values(tbuf + cj + lo, hi - lo, false, v0, v1, err);
        __syncthreads();
        // first the columns of its own strip (and zeros), then the awaited ones
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = CI.cb + lane + 64 * u - ro;
            const bool mine = c >= 0 && c < rows && lane + 64 * u < CI.cnt;
            zs[wv][lane + 64 * u] = mine ? own[c < 0 ? 0 : (c < TS ? c : 0)] : 0.0;
        }
        wave_sync();
        if (lane < hi - lo) zs[wv][off + lane] = v0;
        if (lane + 64 < hi - lo) zs[wv][off + lane + 64] = v1;
        wave_sync();
    }
#pragma unroll
    for (int k = 0; k < RPL; ++k) acc[k] = 0.0;
    for (int t0 = 0;;) {
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            pin4(pre[m]);
            const double zc = zs[wv][csub + t0 + CS * m];
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] += (double)__uint_as_float(pre[m][k]) * zc;
            if (m % 4 == 3) pin_sums();
        }
        t0 += PF * CS;
        if (t0 >= CI.cnt) break;                          // wave-uniform
        load_inverse(t0);
    }
    part[pb][wv][irow] = fold16(fold32(acc[0], acc[2]), fold32(acc[1], acc[3]));
    __syncthreads();
    if (wv == 0 && tid < rows) {
        double t[NW];
#pragma unroll
        for (int u = 0; u < NW; ++u) t[u] = part[pb][u][lane];
        const double z = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        put_value(out + r0 + tid, z);
        if (!LOWER) zout[py * ld_z + r0 + tid] = z;
    }
}

__global__ void k_prec_reset(double* buf, int64_t count, unsigned* words) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) put_unset(buf + i);
    if (i < 3) words[i] = 0u;
}

// forward solution and its block right-hand sides, the backward solve's two
// (n x nr each); the two solves' start-order counters and the error word
size_t prec_work_bytes(int64_t n, int nr) { return (size_t)(4 * n * nr) * 8 + 256; }

static unsigned* prec_words(double* W, int64_t n, int nr) { return (unsigned*)(W + 4 * n * nr); }

// the forward solve's buffers, the counters and the error word: once before the
// applies with this n, nr (each solve then clears the other's)
hipError_t prec_reset(double* W, int64_t n, int nr, hipStream_t s) {
    const int64_t count = 2 * n * nr;
    k_prec_reset<<<(unsigned)((count + 255) / 256), 256, 0, s>>>(W, count, prec_words(W, n, nr));
    return hipGetLastError();
}

hipError_t prec_err_read(double* W, int64_t n, int nr, int* err, hipStream_t s) {
    hipError_t e = hipMemcpyAsync(err, prec_words(W, n, nr) + 2, sizeof(int), hipMemcpyDeviceToHost, s);
    if (!e) e = hipStreamSynchronize(s);
    return e;
}

template <int ST>
static hipError_t prec_typed(const PrecPlan& p, const double* V, int64_t ldv, double* Z, int64_t ldz, int nr,
                             double* W, hipStream_t s) {
    typedef typename Store<ST>::T T;
    const int64_t n = p.n, nb = p.nb;
    const int64_t nstrips32 = (n + 31) / 32;
    const int64_t S = (n + TS - 1) / TS;
    double *Y = W, *Tf = Y + n * nr, *Xb = Tf + n * nr, *Tb = Xb + n * nr;
    unsigned* tk = prec_words(W, n, nr);
    int* err = (int*)(tk + 2);
    // 16-byte loads: aligned columns, and a wave's 128 of them within 32-bit offsets
    const int64_t colb = p.lda * (int64_t)sizeof(T);
    const bool vec = colb % 16 == 0 && ((uintptr_t)p.A) % 16 == 0 && colb <= (1ll << 32) / 128;
    const int db = (int)prec_block(nb);
    const dim3 grid((unsigned)S, (unsigned)nr);
    hipEvent_t pt = prof::begin(prof::PREC, s);
    auto solves = [&](auto VEC) {
        constexpr bool V16 = decltype(VEC)::value;
        k_trsv<ST, true, V16><<<grid, 512, 0, s>>>(n, (int)nb, db, (const T*)p.A, p.lda, p.linv_full, p.lsc, nstrips32,
                                                   p.rowscale, V, ldv, Tf, Y, Tb, Xb, nullptr, 0, tk, tk + 1, err);
        k_trsv<ST, false, V16><<<grid, 512, 0, s>>>(n, (int)nb, db, (const T*)p.A, p.lda, p.uinv_full, nullptr,
                                                    nstrips32, nullptr, Y, n, Tb, Xb, Tf, Y, Z, ldz, tk + 1, tk, err);
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
