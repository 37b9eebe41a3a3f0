// ftgemm_split.hpp -- FP32 online ABFT GEMM on the bf16 matrix instructions (gfx950).
//
// The FP32 matrix instruction takes 64 cycles for 32 x 32 x 2, the bf16 one 32
// cycles for 32 x 32 x 16: sixteen times the rate.  Every FP32 operand is split
// (Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence
// Datatype For Higher-Precision Computations", ARITH 2019) exactly into three
// bf16 parts, x = x0 + x1 + x2 (each the rest rounded to
// nearest: 8 + 8 + 8 bits), and a product is the six part products down to
// 2^-16 of the largest, x0 y0, x0 y1, x1 y0, x1 y1, x0 y2 and x2 y0, added to
// one FP32 accumulator; the dropped ones are below 2^-25 of |x y| and of either
// sign.  Against 64 bits the result is closer than the FP32 instruction's
// (2-norm of the error over K = 64 .. 8192 on normal, uniform, positive and
// heavy-tailed operands: 0.6 to 0.93 of it; positive operands, K = 4 .. 39: 0.39 to
// 0.95, the most at K = 17), because an accumulator is rounded
// once per 16 k and product instead of once per k.  (Cutting the leading part
// off instead of rounding it leaves remainders of one sign, and on positive
// data the small products are then lost to rounding all in one direction.)
//
// The fault tolerance is that of the FP32 kernels (ftgemm_fp32.hpp: encodings
// from the staging registers, references per line, the check of
// ftgemm_abft.hpp), in FP32 on the unsplit operands.  A thread keeps the four
// lines x 4 k it stages in registers until the panel's encodings are complete,
// one barrier later, and adds their products with the encodings to its own
// partial references, which are summed over the four threads of a line only at
// a check: the owners' reads of whole rows and columns from LDS are gone.
//
// What bounds it: at 256 x 256 and 8192^3 the matrix instructions take some 3 ms
// of 5.1 to 5.3 (six times the library's bf16 product of that size takes 5.8 ms).
// Vector instructions issue beside
// matrix instructions of either wavefront on the SIMD (measured: six between
// two MFMAs are 90-95% hidden; v_dot2 is the exception, it waits for the matrix
// pipe), so the split, the encodings and the reference updates of a panel,
// about 190 instructions per wavefront, are dealt out between its 48 MFMAs.
// 8192^3 online: 8.7 ms on the FP32 instructions, 5.13 to 5.29 ms here; 2048^3 (one
// 128 x 128 tile per compute unit, bound by the latency of a panel: LDS reads
// after the barrier, split and store before the next) 0.210 -> 0.131 ms.
//
// Every operand is multiplied by 2^16 as it is split, and the sums by 2^-32 at the
// end (both exact): a binary32 number, denormals included, is then a multiple of
// bf16's smallest denormal 2^-133, so none is too small for its three parts.
// Where the split does not hold: Inf, NaN and lines whose norm is 2^43 or more,
// whose scaled sums could overflow.  Those are seen before the first check that
// would cover them; the tile is then computed again by f32::tile, which is what
// the kernel's callers do on `false`.
#pragma once

#include "ftgemm_fp32.hpp"

namespace ftgemm_impl {
namespace f32s {

using namespace abft;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int KC = 16;      // k of one panel (one 32x32x16 MFMA deep)
constexpr int PARTS = 3;

// A panel in fragment order: [part][block of 32 rows][16-byte unit], 64 units
// of 8 k per block.  The unit of (row, lane half) is a permutation of the
// block, so a fragment read is 1 KB of consecutive LDS in some lane order.
template <int ROWS>
struct Panel {
    unsigned short p[PARTS][ROWS / 32][64][8];
};

// The encodings are kept as the partial sums of the wavefronts that stage a
// panel; their readers add them.  (LDS float atomics into one sum took 200
// LDS cycles per wavefront and panel at 256 x 256, more than every other LDS
// access of the step together.)
template <int BM, int BN, int NE>   // NE: wavefronts per role
struct alignas(16) OperandsSplit {
    Panel<BM> A[2];
    Panel<BN> B[2];
    float wsum[2][NE][KC];      // e^T A per k
    float vsum[2][NE][KC];      // B e per k
    float dummy[64];            // sink for the stores of lanes that own no value
};

template <int BM, int BN, int WM, int WN>
struct SmemSplit {
    OperandsSplit<BM, BN, WM * WN / 2> op;
    CheckLds<Geometry<BM, BN, WM, WN>> ck;
};

// Unit of (row % 32, lane half).  A's stores write rows 4 apart, B's
// consecutive columns, both for all four k-quads; with these permutations the
// 16 lanes of a store group fall into 16 distinct bank pairs.
__device__ __forceinline__ int unit_a(int row, int half) { return (row ^ ((row >> 3) & 3) ^ (half << 1)) + 32 * half; }
__device__ __forceinline__ int unit_b(int row, int half) { return (row ^ (half << 2)) + 32 * half; }

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float bf_lo(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf_hi(unsigned x) { return __uint_as_float(x & 0xffff0000u); }
__device__ __forceinline__ float uniform(float x) {   // a wave-uniform value, in a scalar register
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

constexpr float kScale = 65536.0f;                        // of an operand
constexpr float kUnit = 1.0f / (kScale * kScale);         // one unit of a scaled product
// Squares of scaled norms from here on leave the split: below, a product is less
// than 2^118 in size and a line's sum over 256 of them less than 2^126.
constexpr float kHugeNorm2 = 0x1p118f;

constexpr int kRsrcWord3 = 0x00020000;        // raw 32-bit data format
constexpr int kOutside = (int)0x80000000;     // offset past a resource's end: reads as zero
constexpr int kLines = 4;                     // floats of a load
// Offset of a load with `rem` floats of its line left: one that would straddle
// the end is moved back inside.
__device__ __forceinline__ int moved(int off, int rem) { return rem >= kLines ? off : rem > 0 ? off - 4 * (kLines - rem) : kOutside; }

// Whether the tile's operands can take the split path over all of K, multiplied
// by `scale`: asked before the tile does what must not be done twice.
//   * A tile with faults to inject asks first (they are logged as they are
//     applied).  Its accumulators are not scaled (a bit flip is one of the
//     accumulator as FP32 arithmetic has it), so no element may be too small for
//     its parts.  16-byte loads, 32 in flight per thread (DEEP): one fault adds
//     0.30 ms to a launch of 8192^3, 0.03 to 4096^3 and 0.016 to 2048^3 (one 4-byte
//     load after another: 1.29, 0.97 and 0.41 ms).
//   * Any other tile asks at its first flag, if k is left, with the few registers
//     that are free there.  If it leaves, what was flagged goes with the pass it
//     happened in: f32::tile starts from clean accumulators.
// What a thread reads of all lines has a sum of squares that keeps every line's
// norm below the one at which a check leaves.  (Quads at the last rows may look
// at the tile above too.)
template <class G, bool DEEP>
__device__ __forceinline__ bool splittable(const LaunchArgs& a, const Thread& th, int* flag, float scale) {
    constexpr int RQ = G::BM / kLines, PK = G::NT / RQ;     // row quads; k per pass over A
    constexpr int CK = 64, NQ = CK / kLines, CC = G::NT / NQ;   // k and k-quads of a chunk; columns per pass over B
    constexpr int P = CK / PK;                              // passes
    static_assert(P == G::BN / CC, "as many passes over A as over B");
    const int rq = th.tid % RQ, ka = th.tid / RQ, kq = th.tid % NQ, cb = th.tid / NQ;
    const float* const baseA = a.A + th.i0 - kLines;
    const float* const baseB = a.B + (int64_t)th.j0 * a.ldb - kLines;
    const int vA = moved((ka * (int)a.lda + kLines * rq + kLines) * 4, th.mI - kLines * rq);
    const int vB = (cb * (int)a.ldb + kLines * kq + kLines) * 4;
    // pass e of the chunk with `left` k to go
    auto load_a = [&](int left, int e) {
        const int64_t k = (int64_t)a.K - left + e * PK;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(baseA + k * a.lda), (short)0, 0x7fffffff, kRsrcWord3);
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, e * PK + ka < left ? vA : kOutside, 0, 0));
    };
    auto load_b = [&](int left, int e) {
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(baseB + ((int64_t)a.K - left)), (short)0, 0x7fffffff, kRsrcWord3);
        const int v = cb + CC * e < th.nJ ? moved(vB, left - kLines * kq) : kOutside;
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, v, e * CC * (int)a.ldb * 4, 0));
    };
    unsigned least = 0xffffffffu;   // smallest of 2 |x| - 1 as integers, where 0 is the largest
    float sq = 0.f;
    auto see = [&](const f32x4& x) {
#pragma unroll
        for (int q = 0; q < kLines; ++q) {
            least = min(least, (__float_as_uint(x[q]) << 1) - 1u);
            sq = fmaf(x[q], x[q], sq);
        }
    };
    if constexpr (DEEP) {
        f32x4 x[2][2 * P];
        auto load = [&](f32x4 (&y)[2 * P], int left) {
#pragma unroll
            for (int e = 0; e < P; ++e) y[e] = load_a(left, e);
#pragma unroll
            for (int e = 0; e < P; ++e) y[P + e] = load_b(left, e);
        };
        load(x[0], a.K);
        for (int left = a.K; left > 0; left -= 2 * CK) {
            load(x[1], left - CK);
#pragma unroll
            for (int e = 0; e < 2 * P; ++e) see(x[0][e]);
            load(x[0], left - 2 * CK);
#pragma unroll
            for (int e = 0; e < 2 * P; ++e) see(x[1][e]);
        }
    } else {
        for (int left = a.K; left > 0; left -= CK)
#pragma unroll 1
            for (int e = 0; e < P; ++e) {
                const f32x4 x = load_a(left, e), y = load_b(left, e);
                see(x);
                see(y);
            }
    }
    // 2^-100; a factor of two for the sums' own rounding
    const bool bad = (scale == 1.0f && least < 2 * 0x0d800000u - 1) || !(sq * (scale * scale) < kHugeNorm2 / (2 * G::NT));
    if (th.tid == 0) *flag = 0;
    __syncthreads();
    if (bad) *flag = 1;
    __syncthreads();
    const bool ok = __builtin_amdgcn_readfirstlane(*flag) == 0;
    __syncthreads();
    return ok;
}

// What a check asks the split tile: whether it leaves (see check in ftgemm_abft.hpp).
template <class F, class H>
struct Leave {
    F norms;    // a line's norm is too large, or not finite
    H flag;     // something is about to be logged
    __device__ __forceinline__ bool operator()() const { return norms(); }
    __device__ __forceinline__ bool flagged() const { return flag(); }
};
template <class F, class H>
__device__ Leave(F, H) -> Leave<F, H>;

// One BM x BN tile.  Returns false, with C untouched, when the tile's
// operands do not fit the split; the caller then runs f32::tile.
template <int BM, int BN, int WM, int WN, int FT, bool INJ>
__device__ __forceinline__ bool tile(const LaunchArgs& a, int tm, int tn, SmemSplit<BM, BN, WM, WN>& sm) {
    using G = Geometry<BM, BN, WM, WN>;
    constexpr int NT = G::NT, TM = G::TM, TN = G::TN, MI = G::MI, NI = G::NI;
    constexpr int BK = 32;              // k-step of the interface: two panels
    constexpr int NE = WM * WN / 2;     // wavefronts per role
    constexpr int LT = kLines;          // lines per thread
    constexpr int LQ = BM / LT;         // line groups per panel
    static_assert(BM == BN && NT == 2 * BM && LQ % 32 == 0 && NI == 2, "four lines x 4 k per thread");

    auto& op = sm.op;
    Thread th = make_thread<G, true>(a, tm, tn);
    const int tid = th.tid, lane = th.lane, wm = th.wm, wn = th.wn, l32 = th.l32, hh = th.hh;
    const int mI = th.mI;
    const int nk = (a.K + BK - 1) / BK;
    const bool row_role = __builtin_amdgcn_readfirstlane(tid >> 6) < NE;

    // offsets inside a panel have to fit in 31 bits
    if ((int64_t)(KC + 1) * a.lda * 4 >= (int64_t(1) << 31) || (int64_t)(BN + 1) * a.ldb * 4 >= (int64_t(1) << 31)) return false;
    if (a.M < LT || a.K < LT) return false;

    // ---- roles: the first half of the threads stages A, the other B; thread
    // st of a role holds k-quad kq = st % 4 of four lines, rows 4 lq + r of A or
    // columns lq + LQ r of B, and owns line r = kq of them
    const int st = row_role ? tid : tid - NT / 2;
    const int kq = st & 3, lq = st >> 2;
    th.my_row = row_role ? st : -1;
    th.my_col = row_role ? -1 : lq + LQ * kq;

    if constexpr (FT > 0) {
        clear_check(sm.ck, tid);
    }
    if (tid == 0) sm.ck.bail = 0;
    int fnext = 0, flogged = 0;
    bool faulty = false;
    if constexpr (INJ) {
        gather_faults<G>(sm.ck, a, th);
        __syncthreads();
        faulty = __builtin_amdgcn_readfirstlane(sm.ck.nf) > 0;   // (kept unscaled, see splittable)
        if (faulty && !splittable<G, true>(a, th, &sm.ck.bail, 1.0f)) return false;
    }
    __syncthreads();

    // ---- global -> registers: four 16-byte loads, x[e] = rows 4 lq .. + 3 of
    // k = 4 kq + e of A, or k 4 kq .. + 3 of column lq + LQ e of B.
    // The loads have no alignment beyond a float's; what lies outside the matrix
    // is given an offset past the resource's end and reads as zero.  (The loads
    // stay out of branches: with them in one, the waits for them were coarser.)  A load that would straddle the last row of the tile
    // or the last k is moved back inside, and fix() shifts what it got.
    constexpr int inset = LT;     // the base lies four floats early, so that a moved load's offset is not negative
    const int voff = row_role ? moved((4 * kq * (int)a.lda + LT * lq + inset) * 4, mI - LT * lq) : (lq * (int)a.ldb + 4 * kq + inset) * 4;
    const int pstride = row_role ? KC * (int)a.lda * 4 : KC * 4;
    const int estride = (row_role ? (int)a.lda : LQ * (int)a.ldb) * 4;
    const bool whole_n = th.nJ == BN;
    const char* const base0 = row_role ? reinterpret_cast<const char*>(a.A + th.i0 - inset)
                                       : reinterpret_cast<const char*>(a.B + (int64_t)th.j0 * a.ldb - inset);
    auto load = [&](f32x4 (&x)[4], int p) {
        const int k0 = p * KC;
        // the panel's origin in the resource, a load's line or k in a scalar
        // offset: no address arithmetic in the vector unit and little in the scalar one
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base0 + (int64_t)p * pstride), (short)0, 0x7fffffff, kRsrcWord3);
        int vo[4] = {voff, voff, voff, voff};
        if (!(k0 + KC <= a.K && (row_role || whole_n))) {   // past the last whole panel, or B's last column tile
            const int vk = row_role ? voff : moved(voff, a.K - (k0 + 4 * kq));
#pragma unroll
            for (int e = 0; e < 4; ++e) vo[e] = (row_role ? k0 + 4 * kq + e < a.K : lq + LQ * e < th.nJ) ? vk : kOutside;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo[e], e * estride, 0));
    };
    const int shift = (LT - (row_role ? mI : a.K) % LT) % LT;
    // The panels to fix are those p with (p & fix_mask) == fix_panel: every one of
    // rows that are cut, the one of columns in which K ends, or none.  (One test:
    // the three branches of the conditions written out cost every panel of a
    // ragged tile; 7040 x 128 x 910 online 63.4 -> 58.9 us.)
    const int fix_mask = shift != 0 && !row_role ? ~0 : 0, fix_panel = shift == 0 ? 1 : row_role ? 0 : a.K / KC;
    auto fix = [&](f32x4 (&x)[4], int p) {
        if ((p & fix_mask) != fix_panel) return;
        const int rem = row_role ? mI - LT * lq : a.K - (p * KC + 4 * kq);
        const bool cut = rem > 0 && rem < LT;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int by = 1; by < LT; by *= 2)
                if (shift & by) {
#pragma unroll
                    for (int q = 0; q < LT; ++q) {
                        const float from = q + by < LT ? x[e][q + by < LT ? q + by : 0] : 0.f;
                        x[e][q] = cut ? from : x[e][q];
                    }
                }
        }
    };

    // ---- registers -> LDS: y[r][q] = k 4 kq + q of line r, scaled
    const float scale = INJ ? uniform(faulty ? 1.0f : kScale) : kScale, unit = INJ ? uniform(faulty ? 1.0f : kUnit) : kUnit;
    float y[LT][4];
    // A's 4 x 4 elements are transposed in place, by the wavefronts that stage it
    // (copies, and a branch with all of it in both arms, left the matrix pipe idle
    // for some 60 cycles a panel).
    auto transpose = [&](f32x4 (&x)[4]) {
        if (row_role) {
            float a01 = x[0][1], a02 = x[0][2], a03 = x[0][3], a12 = x[1][2], a13 = x[1][3], a23 = x[2][3];
            float a10 = x[1][0], a20 = x[2][0], a30 = x[3][0], a21 = x[2][1], a31 = x[3][1], a32 = x[3][2];
            asm volatile("v_swap_b32 %0, %6\n\tv_swap_b32 %1, %7\n\tv_swap_b32 %2, %8\n\t"
                         "v_swap_b32 %3, %9\n\tv_swap_b32 %4, %10\n\tv_swap_b32 %5, %11"
                         : "+v"(a01), "+v"(a02), "+v"(a03), "+v"(a12), "+v"(a13), "+v"(a23),
                           "+v"(a10), "+v"(a20), "+v"(a30), "+v"(a21), "+v"(a31), "+v"(a32));
            x[0][1] = a01; x[0][2] = a02; x[0][3] = a03; x[1][2] = a12; x[1][3] = a13; x[2][3] = a23;
            x[1][0] = a10; x[2][0] = a20; x[3][0] = a30; x[2][1] = a21; x[3][1] = a31; x[3][2] = a32;
        }
    };
    auto scale_lines = [&](const f32x4 (&x)[4], int r0) {
#pragma unroll
        for (int r = r0; r < r0 + 2; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) y[r][q] = x[r][q] * scale;
    };
    constexpr int PS = BM / 32 * 64 * 8;   // halves per part
    constexpr int BUF = PARTS * PS;        // halves per panel
    const int ua = unit_a((LT * lq) & 31, kq >> 1);
    unsigned short* const dst0 = (row_role ? &op.A[0].p[0][LT * lq >> 5][ua][0] : &op.B[0].p[0][lq >> 5][unit_b(lq & 31, kq >> 1)][0]) +
                                 4 * (kq & 1);
    int doff[LT];   // A: row LT lq + r is unit ua ^ r; B: columns LQ apart are LQ / 32 blocks apart
#pragma unroll
    for (int r = 0; r < LT; ++r) doff[r] = row_role ? ((ua ^ r) - ua) * 8 : r * (LQ / 32) * 512;
    u32x2 part[PARTS];
    auto split_half = [&](int r, int h) {
        const float x0 = y[r][2 * h], x1 = y[r][2 * h + 1];
        part[0][h] = pack_bf16(x0, x1);
        const float e0 = x0 - bf_lo(part[0][h]), e1 = x1 - bf_hi(part[0][h]);
        part[1][h] = pack_bf16(e0, e1);
        part[2][h] = pack_bf16(e0 - bf_lo(part[1][h]), e1 - bf_hi(part[1][h]));
    };
    auto store_line = [&](int buf, int r) {
        unsigned short* d = dst0 + buf * BUF + doff[r];
#pragma unroll
        for (int s = 0; s < PARTS; ++s) *reinterpret_cast<u32x2*>(d + s * PS) = part[s];
    };
    // the lane's store of one encoding partial (lanes that own none: the sink) and its reads
    float* const enc_out = (lane & 12) == 0 ? (row_role ? &op.wsum[0][0][0] : &op.vsum[0][0][0]) +
                                                  (row_role ? th.wave : th.wave - NE) * KC + 4 * kq + ((lane >> 4) & 3)
                                            : &op.dummy[lane];
    const int enc_slot = (lane & 12) == 0 ? NE * KC : 0;
    const float* const enc_in = (row_role ? &op.vsum[0][0][0] : &op.wsum[0][0][0]) + 4 * kq;
    float es[4];
    auto encode_sum = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q) es[q] = (y[0][q] + y[1][q]) + (y[2][q] + y[3][q]);
    };
    auto encode_add = [&](int slot) {
        ReduceScatter<4, 5, 2>::run(es, lane);
        enc_out[slot * enc_slot] = es[0];
    };

    // ---- reference checksums: partial over the thread's k-quads
    float R[LT], n2[LT], rebase = 0.f;
#pragma unroll
    for (int r = 0; r < LT; ++r) R[r] = n2[r] = 0.f;
    auto ft_update = [&](f32x4 v, int r) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            R[r] = fmaf(y[r][q], v[q], R[r]);
            n2[r] = fmaf(y[r][q], y[r][q], n2[r]);
        }
        asm volatile("" : "+v"(R[r]), "+v"(n2[r]));   // keeps the update here (it would be sunk to the next step)
    };

    Acc<G> acc;
#pragma unroll
    for (int bi = 0; bi < MI; ++bi)
#pragma unroll
        for (int bj = 0; bj < NI; ++bj)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.0f;

    const unsigned short* const fa = &op.A[0].p[0][wm * (TM / 32)][unit_a(l32, hh)][0];
    const unsigned short* const fb = &op.B[0].p[0][wn * (TN / 32)][unit_b(l32, hh)][0];
    auto frag = [&](const unsigned short* p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p)); };

    constexpr int NX = BM == 128 ? 2 : 1;   // panels in flight from global memory
    f32x4 xs[NX][4];
    // panel p (LDS buffer `buf`) on the matrix cores, panel p + 1 to the other buffer
    auto step = [&](int p, auto parity) {
        constexpr int buf = decltype(parity)::value;
        auto& x = xs[NX == 2 ? buf ^ 1 : 0];
        f32x4 v;
        if constexpr (FT > 0) {
            v = *reinterpret_cast<const f32x4*>(enc_in + buf * NE * KC);
#pragma unroll
            for (int w = 1; w < NE; ++w) v += *reinterpret_cast<const f32x4*>(enc_in + (buf * NE + w) * KC);
        }
        // Fragments: both column blocks', and the row blocks' one at a time;
        // each register is reloaded for the next row block when its last
        // product of this one is issued, two or more slots before its next use.
        bf16x8 b[NI][PARTS], f[PARTS];
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};   // the small products first
        constexpr int FREED[6] = {2, -1, -1, 1, -1, 0};                         // part last used in slot s
#pragma unroll
        for (int s = 0; s < PARTS; ++s) {   // in the order of use
            f[PARTS - 1 - s] = frag(fa + buf * BUF + (PARTS - 1 - s) * PS);
#pragma unroll
            for (int bj = 0; bj < NI; ++bj) b[bj][s] = frag(fb + buf * BUF + s * PS + bj * 512);
        }
        __builtin_amdgcn_sched_barrier(0);
        // The vector work of the step in units, dealt out over the MFMAs
        constexpr int FTU = FT > 0 ? LT : 0, EU = FT > 0 ? 2 : 0, U = FTU + 4 + EU + 2 * LT;
        auto unit = [&](int u) {
            if (u < FTU) {
                ft_update(v, u);
            } else if (u == FTU) {
                fix(x, p + 1);
                transpose(x);
            } else if (u < FTU + 3) {
                scale_lines(x, 2 * (u - FTU - 1));
            } else if (u == FTU + 3) {
                load(x, p + 1 + NX);
            } else if (u < FTU + 4 + EU) {
                if (u == FTU + 4) encode_sum();
                else encode_add(buf ^ 1);
            } else {
                const int h = u - FTU - EU - 4;
                split_half(h >> 1, h & 1);
                if (h & 1) store_line(buf ^ 1, h >> 1);
            }
        };
        constexpr int S = 6 * MI;                 // slots of NI MFMAs
        constexpr int U0 = FT > 0 ? LT / 2 : 0;   // units that run while the fragments arrive
#pragma unroll
        for (int u = 0; u < U0; ++u) unit(u);
        if constexpr (U0 > 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int bi = s / 6, c = s % 6;
#pragma unroll
            for (int bj = 0; bj < NI; ++bj)
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[bj][PB[c]], f[PA[c]], acc[bi][bj], 0, 0, 0);
            if (FREED[c] >= 0 && bi + 1 < MI) f[FREED[c]] = frag(fa + buf * BUF + FREED[c] * PS + (bi + 1) * 512);
#pragma unroll
            for (int u = U0; u < U; ++u)
                if (u * S < (s + 1) * U && (u * S >= s * U || s == 0)) unit(u);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // What the k-loop stops for, after k-step t; true: the tile leaves the split.
    // A check (every check_interval k-steps and after the last; detect-only: after
    // the last), or without fault tolerance, where K has more than 16 k-steps, a
    // look at the accumulators after the first 8 and after the last: operands with
    // Inf, NaN or large elements throughout take little more than f32::tile's time,
    // not that and the whole split's (8192^3 with one element of 1000 Inf: 12.0 ->
    // 7.9 ms).  Detect-only has no such look, its stop would show on every call
    // (2048^3: 118 -> 121 us): 12.9 ms.  Ends with a barrier behind the step.
    bool stays = faulty;    // what the tile has logged holds: it will not leave any more
    auto stop = [&](int t) -> bool {
        if constexpr (FT > 0) {
            float rr[LT], nn[LT];
#pragma unroll
            for (int r = 0; r < LT; ++r) { rr[r] = R[r]; nn[r] = n2[r]; }
            ReduceScatter<LT, 1, 0>::run(rr, lane);
            ReduceScatter<LT, 1, 0>::run(nn, lane);
            if (!(nn[0] < kHugeNorm2)) sm.ck.bail = 1;
            const float r0 = rr[0] + rebase;
            float ref = r0;
            auto left = [&]() { return __builtin_amdgcn_readfirstlane(sm.ck.bail) != 0; };
            auto flagged = [&]() {
                if (!stays && t + 1 < nk && !splittable<G, false>(a, opaque_lanes(th), &sm.ck.bail, scale)) return true;
                stays = true;
                return false;
            };
            if (check<G, FT, INJ>(acc, sm.ck, a, th, t, min((t + 1) * BK, a.K), ref, nn[0], ref, nn[0], fnext, flogged,
                                  Leave{left, flagged}, unit))
                return true;
            rebase += ref - r0;
            return false;
        } else {
            float z = 0.f;   // stays 0 unless an accumulator is Inf or NaN
#pragma unroll
            for (int bi = 0; bi < MI; ++bi)
#pragma unroll
                for (int bj = 0; bj < NI; ++bj)
#pragma unroll
                    for (int r = 0; r < 16; ++r) z = fmaf(acc[bi][bj][r], 0.f, z);
            if (!(z == 0.f) && !faulty) sm.ck.bail = 1;
            __syncthreads();
            return __builtin_amdgcn_readfirstlane(sm.ck.bail) != 0;
        }
    };
    const int last = nk - 1;
    auto next_stop = [&](int t) {   // after the one behind k-step t (-1: the first)
        if constexpr (FT > 0) return last - t > a.check_interval ? t + a.check_interval : last;
        return t < 0 && last > 15 ? 7 : last;
    };

    load(xs[0], 0);
    if constexpr (NX == 2) load(xs[NX - 1], 1);
    fix(xs[0], 0);
    transpose(xs[0]);
    scale_lines(xs[0], 0);
    scale_lines(xs[0], 2);
    load(xs[0], NX);
#pragma unroll
    for (int r = 0; r < LT; ++r) {
        split_half(r, 0);
        split_half(r, 1);
        store_line(0, r);
    }
    if constexpr (FT > 0) {
        encode_sum();
        encode_add(0);
    }
    __syncthreads();
    for (int t = 0, at = next_stop(-1); t < nk; at = next_stop(t), ++t) {
        for (;; ++t) {
            step(2 * t, std::integral_constant<int, 0>{});
            __syncthreads();
            step(2 * t + 1, std::integral_constant<int, 1>{});
            if constexpr (INJ) inject<G>(acc, sm.ck, a, th, t, fnext);
            if (t == at) break;
            __syncthreads();
        }
        if (stop(t)) return false;
    }
    // back to the product's units with alpha, unless alpha is so small that
    // the factor would be denormal
    float factor = unit;
    if (fabsf(a.alpha) < 0x1p-94f) {
        factor = 1.0f;
#pragma unroll
        for (int bi = 0; bi < MI; ++bi)
#pragma unroll
            for (int bj = 0; bj < NI; ++bj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[bi][bj][r] *= unit;
    }
    finish_tile<G, FT>(acc, sm.ck, a, th, factor);
    return true;
}

}  // namespace f32s
}  // namespace ftgemm_impl
