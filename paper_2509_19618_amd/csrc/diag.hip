// diag.hip -- FP32 LU without pivoting of one diagonal block (the panel
// factorisation of the right-looking blocked LU; paper: "Algorithmic
// Framework" and its Figure 1: the panel is factored in 32-bit arithmetic
// before the 16-bit trailing update).
//
// The block is at most 1024 x 1024, P x P tiles of 32 x 32.  It is factored as
// a dataflow of tiles, every tile formed by one wave in registers: the
// products of the tiles left of and above it are accumulated as those are
// published, then the tile is solved against its diagonal tile and published.
//
// Layout.  A tile of L or U is exchanged "K-major": L(i,s) by rows (row-major
// copy Trm), U(s,j) by columns (column-major T), so that both are 32 runs of
// 32 consecutive floats over the inner index.  A wave holds a tile as 2 x 2
// blocks of the 16 x 16 MFMA: lane l = 16 g + c has, in register 8 J + 4 I + q,
// run 16 J + c at inner index 16 I + 4 g + q.  That is at once the A and the B
// operand order of v_mfma_f32_16x16x4f32 (any order of K serves if both
// operands share it; in that of K itself, which takes 4-byte loads, the
// factorisation at n = 12013 took 6.75 against 6.10 ms for the same error on
// dominant and sqrt(n) matrices; on uniform entries, where a small pivot's terms
// cancel in the next one, |LU - A| / |L||U| was 0.12 against 0.20 units of 2^-24,
// rms) and the order of its result registers, so that a tile
// goes from accumulation through the solve to the next product without moving
// between lanes.  Tiles of L are kept transposed, which makes L (solve with
// U^T) and U (solve with L) one code path: side 0 = L(o,d), side 1 = U(d,o),
// with outer index o and step d < o.
//
// The solve against a 32 x 32 triangle runs in eight blocks of four rows: the
// four rows stand in four registers of one 16-lane row of the wave, so the
// 4 x 4 substitution is six FMAs on broadcast multipliers; three lane-row
// swaps turn them into an operand, and the rows below take a rank-4 update by
// one MFMA per 16 x 16 block, the block of the next four rows first.  The LU
// of a diagonal tile (the leaf) does the same on the tile and on its
// transpose at once: one supplies the rows of U, the other the columns of L,
// each the operand the other's update needs.  (With 32 x 32 x 2 MFMAs, whose
// results take twice as long, the leaf took 3.1 us.)
//
// One work-group carries the chain that bounds the block: wave 0 the diagonal
// tiles, four waves the tiles at distance one and two from the diagonal (both
// sides), exchanging through LDS; two waves publish their tiles.  A chain tile
// of step t only takes its last update (by step t - 1; the diagonal tile its
// last two) there.  All other
// tiles, the earlier updates of the chain's tiles, the copies of its tiles that
// later kernels read and the inverses of the 64 x 64 diagonal sub-blocks are
// tasks taken in order from a device counter by the remaining waves (one of the
// chain's work-group, so that one resident work-group suffices, and all of the
// others).  A task only waits for tiles of earlier tasks and of the chain's
// earlier steps.  The chain's work-group is the first of the block to start, by a
// device counter, not one index: the hardware deals the indices out to the XCDs,
// each dispatching its share in order, and the helpers of several launches on
// several streams could hold the places that the work-groups they wait for need.
// So every wait is for work-groups that have started.  Tiles between work-groups go through device-scope accesses
// with one flag per tile; a flag is raised after the tile's stores are
// acknowledged (sync_release in common.hpp).  Every wait is bounded: on expiry
// it records an error in *info and the wave exits.
//
// What bounds it: the chain, about 6.5 us per tile step (leaf 2.5, solve 1.5,
// last update 0.9, the rest hand-overs and the round through the helpers: a
// tile at distance three is back 5.7 us after its leaf).  With one phase per
// kind of task, opened and closed through device counters, a step took 15 us.
// Measured with rocprofv3 inside factorisations (BF16): nb = 512 252 -> 148 us
// per block (n = 12013, in part beside other strips' solves; 131 alone), nb = 256
// 122 -> 65 us, nb = 128 71 -> 35 us.
#include "common.hpp"
#include "kernels.hpp"

namespace mxp {

namespace {

typedef float f4v_t __attribute__((ext_vector_type(4)));

// eight waves of at most 128 registers and 80 KB of LDS: a work-group takes
// the place of one work-group of the concurrent trailing update on a CU
constexpr int DW = 8;
constexpr int DT = DW * 64;
constexpr int SP = 36;              // LDS pitch of a tile
constexpr int TILE_F = 32 * SP;     // floats of a tile in LDS
constexpr int FAC_F = TILE_F + 32;  // a triangle and its diagonal's reciprocals
constexpr int NR = 2;               // ring slots per side and distance
// LDS of the chain's work-group (floats): two leaf slots (L, U with reciprocals), the
// rings of distance one and two, and the triangle of its task wave; the other
// work-groups: one triangle per wave
constexpr int O_FAC = 0;                            // [slot][L, U]
constexpr int O_RING = 4 * FAC_F;                   // [distance - 1][side][slot]
constexpr int O_TASK = O_RING + 4 * NR * TILE_F;
constexpr int O_END = O_TASK + FAC_F;
constexpr unsigned LIMIT_G = 1u << 26;              // polls of a device flag
constexpr unsigned LIMIT_L = 1u << 29;              // polls of an LDS word

MXP_DEV float rl(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
MXP_DEV int ild(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// v, hidden from the optimiser
MXP_DEV int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// element of register r = 8 J + 4 I + q in lane 16 g + c: inner index, run
MXP_DEV int kin(int r, int g) { return 16 * ((r >> 2) & 1) + 4 * g + (r & 3); }
MXP_DEV int krun(int r, int c) { return 16 * (r >> 3) + c; }

// the four values y0..y3 of lane row GB as one MFMA operand: lane row k gets
// y_k of lane row GB
template <int GB> MXP_DEV float gather4(float y0, float y1, float y2, float y3) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(y0), __float_as_int(y1), false, false);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(y2), __float_as_int(y3), false, false);
    const auto o = __builtin_amdgcn_permlane32_swap(p[GB & 1], r[GB & 1], false, false);
    return __int_as_float(o[GB >> 1]);
}
MXP_DEV f4v_t mma16(float a, float b, f4v_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// a tile in registers: x[2 J + I] = the block of runs 16 J.., inner 16 I..
struct Tile {
    f4v_t x[4];
};
MXP_DEV Tile neg(Tile t) {
#pragma unroll
    for (int b = 0; b < 4; ++b) t.x[b] = -t.x[b];
    return t;
}
// a published tile: device scope, 8 bytes per access
MXP_DEV Tile ld_tile(const float* base, int ld, int c, int g) {
    Tile t;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const uint64_t* p = (const uint64_t*)(base + (16 * (b >> 1) + c) * ld + 16 * (b & 1) + 4 * g);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint64_t v = __hip_atomic_load(p + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            t.x[b][2 * h] = __uint_as_float((uint32_t)v);
            t.x[b][2 * h + 1] = __uint_as_float((uint32_t)(v >> 32));
        }
    }
    return t;
}
MXP_DEV void st_tile(const Tile& t, float* base, int ld, int c, int g) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        uint64_t* p = (uint64_t*)(base + (16 * (b >> 1) + c) * ld + 16 * (b & 1) + 4 * g);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint64_t v = (uint64_t)__float_as_uint(t.x[b][2 * h]) |
                               ((uint64_t)__float_as_uint(t.x[b][2 * h + 1]) << 32);
            __hip_atomic_store(p + h, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}
MXP_DEV Tile lds_ld_tile(const float* s, int c, int g) {
    Tile t;
#pragma unroll
    for (int b = 0; b < 4; ++b) t.x[b] = *(const f4v_t*)(s + (16 * (b >> 1) + c) * SP + 16 * (b & 1) + 4 * g);
    return t;
}
MXP_DEV void lds_st_tile(const Tile& t, float* s, int c, int g) {
#pragma unroll
    for (int b = 0; b < 4; ++b) *(f4v_t*)(s + (16 * (b >> 1) + c) * SP + 16 * (b & 1) + 4 * g) = t.x[b];
}

// t + the product of two tiles (runs of a: the inner index of the result),
// the product summed on its own (32 terms) and added with one rounding
MXP_DEV Tile mma_tile(const Tile& a, const Tile& b, Tile t) {
    f4v_t acc[4] = {};
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int o = 0; o < 4; ++o)
            acc[o] = mma16(a.x[2 * (o & 1) + (k >> 2)][k & 3], b.x[2 * (o >> 1) + (k >> 2)][k & 3], acc[o]);
#pragma unroll
    for (int o = 0; o < 4; ++o) t.x[o] += acc[o];
    return t;
}

// x <- M^-1 x for a lower triangle in LDS: F[r * SP + k] = M[r][k] (k < r),
// DIV: its diagonal's reciprocals at F[TILE_F + k] (else unit)
template <bool DIV, int B> MXP_DEV void solve_step(Tile& t, const float* F, int c, int g) {
    if constexpr (B < 8) {
        constexpr int I = B >> 2, gb = B & 3;
        const float m10 = F[(4 * B + 1) * SP + 4 * B];
        const f4v_t m2 = *(const f4v_t*)(F + (4 * B + 2) * SP + 4 * B);
        const f4v_t m3 = *(const f4v_t*)(F + (4 * B + 3) * SP + 4 * B);
        // the operand's rows at or above the block are left out
        float a0 = 0.0f, a1 = 0.0f;
        if constexpr (gb < 3) {
            a0 = F[(16 * I + c) * SP + 4 * B + g];
            a0 = c >= 4 * gb + 4 ? -a0 : 0.0f;
        }
        if constexpr (I == 0) a1 = -F[(16 + c) * SP + 4 * B + g];
        f4v_t d = {1.0f, 1.0f, 1.0f, 1.0f};
        if constexpr (DIV) d = *(const f4v_t*)(F + TILE_F + 4 * B);
        const bool own = g == gb;
        float op[2];
#pragma unroll
        for (int J = 0; J < 2; ++J) {
            f4v_t& x = t.x[2 * J + I];
            float y0 = x[0], y1 = x[1], y2 = x[2], y3 = x[3];
            if constexpr (DIV) y0 *= d[0];
            y1 = fmaf(-m10, y0, y1);
            y2 = fmaf(-m2[0], y0, y2);
            y3 = fmaf(-m3[0], y0, y3);
            if constexpr (DIV) y1 *= d[1];
            y2 = fmaf(-m2[1], y1, y2);
            y3 = fmaf(-m3[1], y1, y3);
            if constexpr (DIV) y2 *= d[2];
            y3 = fmaf(-m3[2], y2, y3);
            if constexpr (DIV) y3 *= d[3];
            x[0] = own ? y0 : x[0];
            x[1] = own ? y1 : x[1];
            x[2] = own ? y2 : x[2];
            x[3] = own ? y3 : x[3];
            if constexpr (B < 7) op[J] = gather4<gb>(y0, y1, y2, y3);
        }
        if constexpr (gb < 3) {
            t.x[I] = mma16(a0, op[0], t.x[I]);
            t.x[2 + I] = mma16(a0, op[1], t.x[2 + I]);
        }
        if constexpr (I == 0) {
            t.x[1] = mma16(a1, op[0], t.x[1]);
            t.x[3] = mma16(a1, op[1], t.x[3]);
        }
        solve_step<DIV, B + 1>(t, F, c, g);
    }
}
MXP_DEV void solve_tile(Tile& t, const float* F, bool div, int c, int g) {
    if (div) solve_step<true, 0>(t, F, c, g);
    else solve_step<false, 0>(t, F, c, g);
}

// Four columns of the leaf.  T: blocks of the tile by rows (lane = column):
// [0] (rows 0.., columns 0..), [1] (rows 0.., columns 16..), [2] (rows 16..,
// columns 16..); W the same of its transpose (lane = row).  The rows of U go
// to FU[column * SP + row], the columns of L to FL[row * SP + column], the
// pivots' reciprocals to FU[TILE_F + ..].  The update of the block with the
// next pivots is issued first.
template <int B> MXP_DEV void leaf_step(f4v_t (&T)[3], f4v_t (&W)[3], float* FL, float* FU, int c, int g) {
    if constexpr (B < 8) {
        constexpr int I = B >> 2, gb = B & 3, l0 = 20 * gb;        // lane 16 gb + 4 gb
        constexpr int NJ = I == 0 ? 2 : 1, b0 = I == 0 ? 0 : 2;
        f4v_t r[NJ], w[NJ];
#pragma unroll
        for (int J = 0; J < NJ; ++J) { r[J] = T[b0 + J]; w[J] = W[b0 + J]; }
        const float p0 = rl(r[0][0], l0), i0 = __builtin_amdgcn_rcpf(p0);    // v_rcp_f32 (1 ulp)
        const float l10 = -(rl(r[0][1], l0) * i0);
        r[0][1] = fmaf(l10, r[0][0], r[0][1]);
        const float p1 = rl(r[0][1], l0 + 1), i1 = __builtin_amdgcn_rcpf(p1);
        const float l20 = -(rl(r[0][2], l0) * i0), l30 = -(rl(r[0][3], l0) * i0);
        r[0][2] = fmaf(l20, r[0][0], r[0][2]);
        r[0][3] = fmaf(l30, r[0][0], r[0][3]);
        const float l21 = -(rl(r[0][2], l0 + 1) * i1), l31 = -(rl(r[0][3], l0 + 1) * i1);
        r[0][2] = fmaf(l21, r[0][1], r[0][2]);
        const float p2 = rl(r[0][2], l0 + 2), i2 = __builtin_amdgcn_rcpf(p2);
        r[0][3] = fmaf(l31, r[0][1], r[0][3]);
        const float l32 = -(rl(r[0][3], l0 + 2) * i2);
        r[0][3] = fmaf(l32, r[0][2], r[0][3]);
        const float p3 = rl(r[0][3], l0 + 3), i3 = __builtin_amdgcn_rcpf(p3);
        const float u01 = rl(r[0][0], l0 + 1), u02 = rl(r[0][0], l0 + 2), u03 = rl(r[0][0], l0 + 3);
        const float u12 = rl(r[0][1], l0 + 2), u13 = rl(r[0][1], l0 + 3), u23 = rl(r[0][2], l0 + 3);
        if constexpr (NJ == 2) {
            r[1][1] = fmaf(l10, r[1][0], r[1][1]);
            r[1][2] = fmaf(l20, r[1][0], r[1][2]);
            r[1][3] = fmaf(l30, r[1][0], r[1][3]);
            r[1][2] = fmaf(l21, r[1][1], r[1][2]);
            r[1][3] = fmaf(l31, r[1][1], r[1][3]);
            r[1][3] = fmaf(l32, r[1][2], r[1][3]);
        }
#pragma unroll
        for (int J = 0; J < NJ; ++J) {
            w[J][0] *= i0;
            w[J][1] = fmaf(-w[J][0], u01, w[J][1]) * i1;
            w[J][2] = fmaf(-w[J][1], u12, fmaf(-w[J][0], u02, w[J][2])) * i2;
            w[J][3] = fmaf(-w[J][2], u23, fmaf(-w[J][1], u13, fmaf(-w[J][0], u03, w[J][3]))) * i3;
        }
        const bool below = c >= 4 * gb + 4;
        if (g == gb) {
#pragma unroll
            for (int J = 0; J < NJ; ++J) {
                const int o = (I == 0 ? 16 * J : 16) + c;
                *(f4v_t*)(FU + o * SP + 4 * B) = r[J];
                *(f4v_t*)(FL + o * SP + 4 * B) = w[J];
            }
            const f4v_t iv = {i0, i1, i2, i3};
            *(f4v_t*)(FU + TILE_F + 4 * B) = iv;
        }
        float ou[NJ], ol[NJ];
        if constexpr (B < 7) {
#pragma unroll
            for (int J = 0; J < NJ; ++J) {
                ol[J] = gather4<gb>(w[J][0], w[J][1], w[J][2], w[J][3]);
                ou[J] = gather4<gb>(r[J][0], r[J][1], r[J][2], r[J][3]);
            }
        }
        if constexpr (gb < 3) {
            const float al = below ? -ol[0] : 0.0f, au = below ? -ou[0] : 0.0f;
            T[b0] = mma16(al, ou[0], T[b0]);
            W[b0] = mma16(au, ol[0], W[b0]);
            if constexpr (NJ == 2) {
                T[1] = mma16(al, ou[1], T[1]);
                W[1] = mma16(au, ol[1], W[1]);
            }
        }
        if constexpr (NJ == 2) {
            T[2] = mma16(-ol[1], ou[1], T[2]);
            W[2] = mma16(-ou[1], ol[1], W[2]);
        }
        leaf_step<B + 1>(T, W, FL, FU, c, g);
    }
}

}  // namespace

struct DiagOne {
    void* A;
    int64_t lda, k;
    int kb, kbp, ldt, wgs;
    float *T, *Trm, *linv, *uinv;
    int* sync;
    unsigned long long* info;
};
struct DiagGroup {
    DiagOne g[GEMM_GROUP_MAX];
    int count;
};

// device words of one block: the task counter, the count of work-groups that have
// started, then (from SYNC_FLAGS on) a flag per side and tile:
// 1 = the early part of a chain tile is stored, 2 = the tile is final; the
// diagonal tile's final flag is side 0's, its early flag side 1's
constexpr int SYNC_FLAGS = 16;
size_t diag_sync_words(int64_t nb) {
    const int64_t P = (nb + 31) / 32;
    return (size_t)(SYNC_FLAGS + 2 * P * P);
}

// the tasks of step t, in order: the tiles at distance three and more, the
// early updates (all but the last) of the chain tiles of step t + 2, the
// copies of the chain tiles of step t, the inverses of the 64 x 64 sub-block
// that ends with tile t
MXP_DEV int tasks_tiles(int t, int P) { return P - 3 - t > 0 ? 2 * (P - 3 - t) : 0; }
MXP_DEV int tasks_chain(int t, int P) { return t >= P ? 0 : 1 + (t + 1 < P ? 2 : 0) + (t + 2 < P ? 2 : 0); }
MXP_DEV int tasks_inv(int t) { return (t & 1) ? 2 : 0; }

// One launch factors the diagonal blocks of a group of factorisations (one
// per request of the solve server, or a single one): blockIdx.y picks the
// block, each with its own counters; work-groups beyond a block's count leave
// at once.
template <int ST>
__global__ __launch_bounds__(DT, 4) void k_diag_lu(const DiagGroup grp) {
    typedef typename Store<ST>::T STT;
    extern __shared__ __attribute__((aligned(16))) float dsm[];
    __shared__ int s_w[16];            // progress of the chain, in steps (see W_*)
    __shared__ int s_order;            // work-groups of the block that started before
    const DiagOne& G = grp.g[blockIdx.y];
    if ((int)blockIdx.x >= G.wgs) return;
    STT* A = (STT*)G.A;
    const int64_t lda = G.lda, k0 = G.k;
    const int kb = G.kb, ldt = G.ldt, P = G.kbp / 32;
    float *const Trm = G.Trm, *const T0 = G.T;
    auto Kbase = [&](int side) -> float* { return side ? T0 : Trm; };
    int* const flags = G.sync + SYNC_FLAGS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // remade through opaque() before every task and chain step: what is derived
    // from them then stays inside it instead of being held throughout
    int c = lane & 15, g = lane >> 4;
    auto refresh = [&]() {
        c = opaque(lane & 15);
        g = opaque(lane >> 4);
    };
    const bool vec = (lda & 3) == 0 && ((uintptr_t)A & (4 * sizeof(STT) - 1)) == 0;

    auto Ktile = [&](int side, int o, int s) -> float* { return Kbase(side) + (int64_t)(32 * o) * ldt + 32 * s; };
    auto flag = [&](int side, int o, int s) -> int* { return flags + (side * P + o) * P + s; };
    auto fail = [&]() {
        if (lane == 0) atomicMin(G.info, 1ull << 62);
    };
    auto raise = [&](int side, int o, int s, int v) {
        sync_release();
        if (lane == 0) __hip_atomic_store(flag(side, o, s), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // bounded wait until a flag is at least v
    auto wait_flag = [&](const int* f, int v) -> bool {
        for (unsigned it = 0; ild(f) < v; ++it) {
            if (it > LIMIT_G) { fail(); return false; }
            __builtin_amdgcn_s_sleep(1);
        }
        sync_acquire();
        asm volatile("" ::: "memory");
        return true;
    };
    auto lds_get = [&](int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    // after this wave's LDS reads and writes so far
    auto lds_set = [&](int* p, int v) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
    };
    auto wait_lds = [&](int* p, int v) -> bool {
        for (unsigned it = 0; lds_get(p) < v; ++it) {
            if (it > LIMIT_L) { fail(); return false; }
            __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");
        return true;
    };
    // element (i,j) of the block in FP32, the identity beyond kb
    auto a_el = [&](int i, int j) -> float {
        const bool in = i < kb && j < kb;
        const float v = Store<ST>::load(A, in ? (k0 + i) + (k0 + j) * lda : k0 + k0 * lda);
        return in ? v : ((i == j) ? 1.0f : 0.0f);
    };
    // minus tile (side, o, d) of A in the tile layout (side 1 with o = d: the
    // diagonal tile, lane = column)
    auto load_a = [&](int side, int o, int d) -> Tile {
        Tile t;
        if (side == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) t.x[r >> 2][r & 3] = -a_el(32 * o + krun(r, c), 32 * d + kin(r, g));
        } else if (vec && 32 * o + 32 <= kb && 32 * d + 32 <= kb) {
            typedef STT st4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const st4 x = *(const st4*)(A + (k0 + 32 * d + 16 * (b & 1) + 4 * g) +
                                            (k0 + 32 * o + 16 * (b >> 1) + c) * lda);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const STT e = x[i];
                    t.x[b][i] = -Store<ST>::load(&e, 0);
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) t.x[r >> 2][r & 3] = -a_el(32 * d + kin(r, g), 32 * o + krun(r, c));
        }
        return t;
    };
    // tile (side, o, d) to A in the storage format
    auto store_a = [&](int side, int o, int d, const Tile& t) {
        const bool full = 32 * o + 32 <= kb && 32 * d + 32 <= kb;
        if (side && full && vec) {
            typedef STT st4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                st4 x;
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = Store<ST>::from_f32(t.x[b][i]);
                *(st4*)(A + (k0 + 32 * d + 16 * (b & 1) + 4 * g) + (k0 + 32 * o + 16 * (b >> 1) + c) * lda) = x;
            }
            return;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ii = 32 * (side ? d : o) + (side ? kin(r, g) : krun(r, c));
            const int jj = 32 * (side ? o : d) + (side ? krun(r, c) : kin(r, g));
            if (full || (ii < kb && jj < kb)) A[(k0 + ii) + (k0 + jj) * lda] = Store<ST>::from_f32(t.x[r >> 2][r & 3]);
        }
    };
    // the copies of a final tile that only later kernels read: the other
    // orientation in FP32 and A
    auto store_copies = [&](int side, int o, int d, const Tile& t) {
        float* p = Kbase(1 - side) + (int64_t)(32 * d) * ldt + 32 * o;
#pragma unroll
        for (int r = 0; r < 16; ++r) p[(int64_t)kin(r, g) * ldt + krun(r, c)] = t.x[r >> 2][r & 3];
        store_a(side, o, d, t);
    };
    // t += products of the published tiles (1 - side, d, s) and (side, o, s),
    // s in [0, s1), the next pair's loads in flight while one is multiplied
    auto accumulate = [&](Tile& t, int side, int o, int d, int s1) -> bool {
        const int* fa = flag(1 - side, d, 0);
        const int* fb = flag(side, o, 0);
        const float* pa = Ktile(1 - side, d, 0);
        const float* pb = Ktile(side, o, 0);
        const int ls = lane & 31;
        const int* fl = (lane < 32 ? fa : fb) + (ls < s1 ? ls : 0);
        // leading steps with both tiles final
        auto ready = [&]() -> int {
            const unsigned long long m = __ballot(ild(fl) >= 2);
            const unsigned both = (unsigned)m & (unsigned)(m >> 32);
            const int r = both == 0xFFFFFFFFu ? 32 : __ffs(~both) - 1;
            sync_acquire();
            asm volatile("" ::: "memory");
            return r < s1 ? r : s1;
        };
        int r = 0;
        auto need = [&](int s) -> bool {
            for (unsigned it = 0; r <= s; ++it) {
                if (it > LIMIT_G) { fail(); return false; }
                r = ready();
                if (r <= s) __builtin_amdgcn_s_sleep(1);
            }
            return true;
        };
        if (s1 <= 0) return true;
        if (!need(0)) return false;
        Tile a0 = ld_tile(pa, ldt, c, g), b0 = ld_tile(pb, ldt, c, g), a1, b1;
        for (int s = 0; s < s1; s += 2) {
            const bool more = s + 1 < s1;
            bool have = more && s + 1 < r;
            if (have) {
                a1 = ld_tile(pa + 32 * (s + 1), ldt, c, g);
                b1 = ld_tile(pb + 32 * (s + 1), ldt, c, g);
            }
            t = mma_tile(a0, b0, t);
            if (!more) break;
            if (!have) {
                if (!need(s + 1)) return false;
                a1 = ld_tile(pa + 32 * (s + 1), ldt, c, g);
                b1 = ld_tile(pb + 32 * (s + 1), ldt, c, g);
            }
            const bool more2 = s + 2 < s1;
            have = more2 && s + 2 < r;
            if (have) {
                a0 = ld_tile(pa + 32 * (s + 2), ldt, c, g);
                b0 = ld_tile(pb + 32 * (s + 2), ldt, c, g);
            }
            t = mma_tile(a1, b1, t);
            if (more2 && !have) {
                if (!need(s + 2)) return false;
                a0 = ld_tile(pa + 32 * (s + 2), ldt, c, g);
                b0 = ld_tile(pb + 32 * (s + 2), ldt, c, g);
            }
        }
        return true;
    };
    // the published diagonal tile t's triangle of a side (0: L, 1: U) into F
    auto stage_tri = [&](int side, int t, float* F) {
        const Tile v = ld_tile(Ktile(side, t, t), ldt, c, g);
        lds_st_tile(v, F, c, g);
        if (side)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kin(r, g) == krun(r, c)) F[TILE_F + krun(r, c)] = __builtin_amdgcn_rcpf(v.x[r >> 2][r & 3]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };

    // ---- a task (wave-uniform indices); false: a wait expired
    auto run_task = [&](int t, int u, float* F) -> bool {
        const int nt = tasks_tiles(t, P), ne = tasks_chain(t + 2, P), nc = tasks_chain(t, P);
        if (u < nt) {
            const int side = u & 1, o = t + 3 + (u >> 1);
            Tile x = load_a(side, o, t);
            if (!accumulate(x, side, o, t, t)) return false;
            x = neg(x);
            if (!wait_flag(flag(0, t, t), 2)) return false;
            stage_tri(1 - side, t, F);
            solve_tile(x, F, side == 0, c, g);
            st_tile(x, Ktile(side, o, t), ldt, c, g);
            raise(side, o, t, 2);
            store_copies(side, o, t, x);
            return true;
        }
        u -= nt;
        if (u < ne) {
            // all updates but the last (two, the diagonal tile) of a chain
            // tile of step e
            const int e = t + 2;
            const int side = u == 0 ? 1 : (u - 1) & 1, o = u == 0 ? e : e + 1 + ((u - 1) >> 1);
            Tile x = load_a(side, o, e);
            if (!accumulate(x, side, o, e, u == 0 ? e - 2 : e - 1)) return false;
            st_tile(x, Ktile(side, o, e), ldt, c, g);
            raise(side, o, e, 1);
            return true;
        }
        u -= ne;
        if (u < nc) {
            // the copies of a chain tile of step t (the diagonal tile: A alone)
            const int side = u == 0 ? 1 : (u - 1) & 1, o = u == 0 ? t : t + 1 + ((u - 1) >> 1);
            if (!wait_flag(flag(u == 0 ? 0 : side, o, t), 2)) return false;
            const Tile x = ld_tile(Ktile(side, o, t), ldt, c, g);
            if (u == 0) store_a(1, t, t, x);
            else store_copies(side, o, t, x);
            return true;
        }
        u -= nc;
        // the inverse of the 64 x 64 sub-block of tiles (t - 1, t): L (u = 0,
        // column-major) or U (u = 1, row-major), both as lower triangles:
        // [M11 0; M21 M22]^-1 = [Y11 0; -M22^-1 M21 Y11  Y22]
        const int side = u;
        float* I = (side ? G.uinv : G.linv) + (t >> 1) * 4096;
        if (!wait_flag(flag(0, t - 1, t - 1), 2) || !wait_flag(flag(side, t, t - 1), 2) ||
            !wait_flag(flag(0, t, t), 2))
            return false;
        Tile id;
#pragma unroll
        for (int r = 0; r < 16; ++r) id.x[r >> 2][r & 3] = kin(r, g) == krun(r, c) ? 1.0f : 0.0f;
        auto put = [&](const Tile& x, int co, int ro) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *(f4v_t*)(I + (co + 16 * (b >> 1) + c) * 64 + ro + 16 * (b & 1) + 4 * g) = x.x[b];
        };
        const Tile a = ld_tile(Ktile(side, t, t - 1), ldt, c, g);
        Tile x = id;
        stage_tri(side, t - 1, F);
        solve_tile(x, F, side == 1, c, g);
        put(x, 0, 0);
        const Tile zero = {};
        const Tile z = neg(mma_tile(a, x, zero));
        stage_tri(side, t, F);
        x = id;
        solve_tile(x, F, side == 1, c, g);
        put(x, 32, 32);
        // Y21 = Y22 z as a product (a solve rounds its 32 terms at the result's
        // magnitude: the inverses were off by 0.61 instead of 0.51 units of 2^-24,
        // rms of |L Y - I| / |L||Y|), Y22 by its rows through F
        lds_st_tile(x, F, c, g);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int r = 0; r < 16; ++r) x.x[r >> 2][r & 3] = F[kin(r, g) * SP + krun(r, c)];
        put(mma_tile(x, z, zero), 0, 32);
        put(zero, 32, 0);
        return true;
    };
    auto task_loop = [&](float* F) {
        int t = 0, base = 0;
        for (;;) {
            int u = 0;
            if (lane == 0) u = atomicAdd(G.sync, 1);
            u = __builtin_amdgcn_readfirstlane(u);
            for (;;) {
                if (t >= P) return;
                const int nt = tasks_tiles(t, P) + tasks_chain(t + 2, P) + tasks_chain(t, P) + tasks_inv(t);
                if (u < base + nt) break;
                base += nt;
                ++t;
            }
            refresh();
            if (!run_task(t, u - base, F)) return;
        }
    };

    // progress words: steps whose updates the chain waves (0-4: diagonal,
    // distance one side 0, 1, distance two side 0, 1) have finished, steps
    // whose distance-one and -two tiles are published, leaves done, leaves
    // published, and steps solved per distance and side
    constexpr int W_UPD = 0, W_PUB = 5, W_LEAF = 7, W_PUBLEAF = 8, W_DONE = 9;
    if (tid < 16) s_w[tid] = 0;
    if (tid == 0) s_order = __hip_atomic_fetch_add(G.sync + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const bool helper = __builtin_amdgcn_readfirstlane(s_order) != 0;
    // roles of the waves of the first work-group: 0 the diagonal, 1 and 2 distance
    // one, 3 and 7 distance two, 4 and 5 publish (they run no MFMA beside waves 0
    // and 1 on their SIMDs), 6 takes tasks
    if (helper || wave == 6) {
        task_loop(dsm + (helper ? wave * FAC_F : O_TASK));
        return;
    }

    // ---- the chain (the block's first work-group)
    auto fac = [&](int t, int side) -> float* { return dsm + O_FAC + ((t & 1) * 2 + side) * FAC_F; };
    auto ring = [&](int dist, int side, int t) -> float* {
        return dsm + O_RING + (((dist - 1) * 2 + side) * NR + t % NR) * TILE_F;
    };
    // the chain tile (side, o, d) of step d with all updates but the last, then
    // the last (by step d - 1; the diagonal tile the last two): tile (1 - side,
    // d, d - 1) from its ring, tile (side, o, d - 1) from its ring or, at
    // distance three, from memory
    auto chain_tile = [&](Tile& t, int side, int o, int d) -> bool {
        if (d < 2) {
            t = load_a(side, o, d);
            if (d == 0) return true;
        }
        const int s = d - 1, db = o - s;
        Tile a, b;
        if (d >= 2) {
            // both flags in one access
            const int* f = db > 2 && lane == 1 ? flag(side, o, s) : flag(side, o, d);
            for (unsigned it = 0;; ++it) {
                if (!__ballot(ild(f) < (db > 2 && lane == 1 ? 2 : 1))) break;
                if (it > LIMIT_G) { fail(); return false; }
                __builtin_amdgcn_s_sleep(1);
            }
            sync_acquire();
            asm volatile("" ::: "memory");
            t = ld_tile(Ktile(side, o, d), ldt, c, g);
        } else if (db > 2) {
            if (!wait_flag(flag(side, o, s), 2)) return false;
        }
        if (o == d && d >= 2) {
            // the diagonal tile's update by step d - 2
            if (!wait_lds(&s_w[W_DONE + 2], s) || !wait_lds(&s_w[W_DONE + 3], s)) return false;
            const Tile a2 = lds_ld_tile(ring(2, 0, s - 1), c, g), b2 = lds_ld_tile(ring(2, 1, s - 1), c, g);
            t = mma_tile(a2, b2, t);
        }
        if (db > 2) {
            b = ld_tile(Ktile(side, o, s), ldt, c, g);
        } else {
            if (!wait_lds(&s_w[W_DONE + 2 * (db - 1) + side], s + 1)) return false;
            b = lds_ld_tile(ring(db, side, s), c, g);
        }
        if (!wait_lds(&s_w[W_DONE + 1 - side], s + 1)) return false;
        a = lds_ld_tile(ring(1, 1 - side, s), c, g);
        t = mma_tile(a, b, t);
        return true;
    };
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        for (int t = 0; t < P; ++t) {
            refresh();
            Tile x;
            if (!chain_tile(x, 1, t, t)) return;
            lds_set(&s_w[W_UPD], t + 1);
            // the leaf slot of step t - 2 has been published and its solves have ended
            if (t >= 2) {
                for (unsigned it = 0;; ++it) {
                    const int v = lds_get(&s_w[lane < 5 ? W_PUBLEAF + lane : 0]);
                    if (!__ballot(lane < 5 && v < t - 1)) break;
                    if (it > LIMIT_L) { fail(); return; }
                }
                asm volatile("" ::: "memory");
            }
            float* FL = fac(t, 0);
            float* FU = fac(t, 1);
            // the transpose through this slot
            x = neg(x);
            lds_st_tile(x, FU, c, g);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            f4v_t T[3] = {x.x[0], x.x[2], x.x[3]}, W[3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                W[0][q] = FU[(4 * g + q) * SP + c];
                W[1][q] = FU[(4 * g + q) * SP + 16 + c];
                W[2][q] = FU[(16 + 4 * g + q) * SP + 16 + c];
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            leaf_step<0>(T, W, FL, FU, c, g);
            lds_set(&s_w[W_LEAF], t + 1);
            // the first zero / non-finite pivot (the identity beyond kb has pivots 1)
            const float p = FU[(lane & 31) * (SP + 1)];
            const unsigned bad = (unsigned)__ballot(!(p != 0.0f && isfinite(p)));
            if (bad && 32 * t + __ffs(bad) - 1 < kb && lane == 0)
                atomicMin(G.info, (unsigned long long)(k0 + 32 * t + __ffs(bad)));
        }
    } else if (wave == 4) {
        // publishes the diagonal tiles, by columns and by rows
        __builtin_amdgcn_s_setprio(1);
        for (int t = 0; t < P; ++t) {
            refresh();
            if (!wait_lds(&s_w[W_LEAF], t + 1)) return;
            const float* FL = fac(t, 0);
            const float* FU = fac(t, 1);
            Tile cm = lds_ld_tile(FU, c, g), rm = lds_ld_tile(FL, c, g);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kk = kin(r, g), o = krun(r, c);
                const float l = FL[kk * SP + o], u = FU[kk * SP + o];
                cm.x[r >> 2][r & 3] = kk <= o ? cm.x[r >> 2][r & 3] : l;
                rm.x[r >> 2][r & 3] = kk < o ? rm.x[r >> 2][r & 3] : u;
            }
            st_tile(cm, Ktile(1, t, t), ldt, c, g);
            st_tile(rm, Ktile(0, t, t), ldt, c, g);
            lds_set(&s_w[W_PUBLEAF], t + 1);
            raise(0, t, t, 2);
        }
    } else if (wave == 5) {
        // publishes the tiles at distance one and two
        __builtin_amdgcn_s_setprio(1);
        for (int t = 0; t + 1 < P; ++t)
            for (int dist = 1; dist <= 2 && t + dist < P; ++dist) {
                refresh();
                for (int side = 0; side < 2; ++side) {
                    if (!wait_lds(&s_w[W_DONE + 2 * (dist - 1) + side], t + 1)) return;
                    st_tile(lds_ld_tile(ring(dist, side, t), c, g), Ktile(side, t + dist, t), ldt, c, g);
                }
                lds_set(&s_w[W_PUB + dist - 1], t + 1);
                raise(0, t + dist, t, 2);
                raise(1, t + dist, t, 2);
            }
    } else {
        __builtin_amdgcn_s_setprio(2);
        const int dist = wave <= 2 ? 1 : 2, side = dist == 1 ? wave - 1 : wave >> 2;
        const int me = W_UPD + 2 * dist - 1 + side;
        for (int t = 0; t + dist < P; ++t) {
            refresh();
            Tile x;
            if (!chain_tile(x, side, t + dist, t)) return;
            lds_set(&s_w[me], t + 1);
            x = neg(x);
            // the ring slot of step t - NR is no longer read: every chain wave
            // has finished the updates of step t - 1, its tile is published
            if (t >= NR) {
                for (unsigned it = 0;; ++it) {
                    const int v = lds_get(&s_w[lane < 7 ? lane : 0]);
                    if (!__ballot(lane < 5 ? v < t : lane == W_PUB + dist - 1 && v < t - NR + 1)) break;
                    if (it > LIMIT_L) { fail(); return; }
                }
                asm volatile("" ::: "memory");
            }
            if (!wait_lds(&s_w[W_LEAF], t + 1)) return;
            solve_tile(x, fac(t, 1 - side), side == 0, c, g);
            lds_st_tile(x, ring(dist, side, t), c, g);
            lds_set(&s_w[W_DONE + 2 * (dist - 1) + side], t + 1);
        }
        // past its last step a wave holds nobody up
        lds_set(&s_w[me], 1 << 20);
        lds_set(&s_w[W_DONE + 2 * (dist - 1) + side], 1 << 20);
    }
}

// (a CU each: a helper beside the chain's work-group takes issue slots from it, 133
// against 131 us per block at nb = 512)
size_t diag_lu_smem() {
    const size_t need = (size_t)(O_END > DW * FAC_F ? O_END : DW * FAC_F) * sizeof(float);
    return need < OWN_CU_LDS ? OWN_CU_LDS : need;
}

// most work-groups cooperating on one diagonal block
#ifndef MXP_DIAG_WGS
#define MXP_DIAG_WGS 32
#endif

template <int ST>
static hipError_t diag_lu_typed(const DiagCall* calls, int count, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_diag_lu<ST>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)diag_lu_smem());
    if (attr) return attr;
    DiagGroup grp;
    int wmax = 1;
    for (int i = 0; i < count; ++i) {
        const DiagCall& c = calls[i];
        DiagOne& g = grp.g[i];
        g.A = c.A; g.lda = c.lda; g.k = c.k; g.kb = c.kb; g.kbp = c.kbp; g.ldt = c.ldt;
        g.T = c.T; g.Trm = c.Trm; g.linv = c.linv; g.uinv = c.uinv; g.sync = c.sync; g.info = c.info;
        // task waves scale with the work: one work-group per tile column
        const int P = c.kbp / 32;
        g.wgs = P > MXP_DIAG_WGS ? MXP_DIAG_WGS : P;
        wmax = g.wgs > wmax ? g.wgs : wmax;
    }
    grp.count = count;
    k_diag_lu<ST><<<dim3(wmax, count), DT, diag_lu_smem(), s>>>(grp);
    return hipGetLastError();
}

hipError_t diag_lu_group(int store, const DiagCall* calls, int count, hipStream_t s) {
    if (count < 1 || count > GEMM_GROUP_MAX) return hipErrorInvalidValue;
    for (int i = 0; i < count; ++i) {
        const DiagCall& c = calls[i];
        if (c.kb < 1 || c.kbp % 64 || c.kbp > c.ldt || c.kb > c.kbp || c.kbp > 1024) return hipErrorInvalidValue;
    }
    switch (store) {
    case F32: return diag_lu_typed<F32>(calls, count, s);
    case F16: return diag_lu_typed<F16>(calls, count, s);
    case BF16: return diag_lu_typed<BF16>(calls, count, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t diag_lu(int store, void* A, int64_t lda, int64_t k, int kb, int kbp, float* T, float* Trm, int ldt,
                   float* linv, float* uinv, int* sync, unsigned long long* info, hipStream_t s) {
    DiagCall c{A, lda, k, kb, kbp, ldt, T, Trm, linv, uinv, sync, info};
    return diag_lu_group(store, &c, 1, s);
}

}  // namespace mxp
