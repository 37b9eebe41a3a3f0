// ftgemm_bf16m.hpp -- BF16-input online ABFT GEMM for gfx950: operands of any
// alignment, references on the matrix cores.
//
// The method and the layout of the result are those of ftgemm_bf16.hpp; what
// differs is how the fault tolerance is carried through the k-loop:
//   * a thread stages four rows x 8 k of A and four columns x 8 k of B, with all
//     rows of a k in one wavefront (512 contiguous bytes of a column per load),
//     so e^T A needs no sum across wavefronts; of B e every wavefront leaves
//     its part.  Both are put in LDS as matrix operands: FP32 values split
//     exactly into three bf16 parts, one operand row per part and wavefront;
//   * R = A (B e) and S = (e^T A) B are then one more MFMA per operand block and
//     16 k, with the block's fragment that the product reads anyway (each block
//     by one of the wavefronts that read it: blocks are rotated per wavefront,
//     see Geometry, so that it is block 0).  Exact products, FP32 sums;
//   * the squares for the norms come from the staging registers.
// Before, owners read whole rows and columns back from LDS, and the encodings
// were summed by LDS float atomics (two per wavefront and step, about 200 LDS
// cycles each, of the 6600 LDS cycles a 64-k step took) with v_dot2, which
// waits for the matrix pipe.
//
// What bounds it (256 x 256, a 64-k step): matrix instructions 2560 cycles per
// SIMD (2048 without the references), vector instructions about 330 per
// wavefront; with two wavefronts per SIMD every instruction of a wavefront takes
// about 8.8 cycles of issue, so the step takes about 5000 at level 2 and 3400
// without fault tolerance.  Unaligned operands took element loads before.
// 8192^3 online 2.02 -> 1.60 to 1.70 ms, plain 1.02 ms as before (the library's
// product without fault tolerance: 0.96 ms); 2048^3 with recompute 87 -> 68 us;
// 3001 x 1999 x 4097, detection only, 685 -> 150 us.
#pragma once

#include "ftgemm_bf16.hpp"

namespace ftgemm_impl {
namespace bf16m {

using namespace abft;
using bf16::bf16x8;
using bf16::bf16x2;
using bf16::u32x2;
using bf16::u32x4;
using bf16::bf_lo;
using bf16::bf_hi;
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int KC = 64;           // k of one panel, the k-step of the interface
constexpr int SUBS = KC / 16;    // MFMAs deep

// Operand panels in fragment order: 1 KB per (block of 32 lines, 16 k), in
// 16-byte units of 8 k, one per (line, lane half), so that a fragment read is
// 1 KB of consecutive LDS in some lane order.
// venc / wenc: B e and e^T A as matrix operands, three bf16 parts (exact) per
// k: rows 3 w .. 3 w + 2 of venc are wavefront w's part of B e, the first
// three rows of wenc are e^T A; the other rows of the fragments are read from
// `zero`.
template <int BM, int BN, int NW>
struct alignas(16) OperandsBF16M {
    unsigned short A[2][BM / 32][SUBS][64][8];
    unsigned short B[2][BN / 32][SUBS][64][8];
    unsigned short venc[2][SUBS][2][3 * NW + 1][8];   // (odd row count: a store's eight octets fall into eight bank groups)
    unsigned short wenc[2][SUBS][2][4][8];
    unsigned short zero[SUBS][2][3 * NW + 1][8];    // read in place of the rows a fragment does not have, at venc's offsets
    float nrow[8][BM];          // squares of the rows by k-octet, at a check
    float ncol[BN];
    float rref[BM], cref[BN];   // references at a check
};

template <int BM, int BN, int WM, int WN>
struct SmemBF16M {
    OperandsBF16M<BM, BN, WM * WN> op;
    CheckLds<Geometry<BM, BN, WM, WN, true>> ck;
};

// Unit of (line % 32, k-octet).  The eight lanes of a store group write one
// octet of eight rows 4 apart (A) or the eight octets of one column (B).
__device__ __forceinline__ int unit_a(int line, int oct) { return (line ^ ((line >> 3) & 3)) + 32 * (oct & 1); }
__device__ __forceinline__ int unit_b(int line, int oct) { return (line ^ (oct & 7)) + 32 * (oct & 1); }

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// One BM x BN tile.  Returns false, with C untouched, for shapes its loads do
// not cover (fewer than 4 rows or 8 k, offsets past 31 bits).
template <int BM, int BN, int WM, int WN, int FT, bool INJ>
__device__ __forceinline__ bool tile(const LaunchArgs& a, int tm, int tn, SmemBF16M<BM, BN, WM, WN>& sm) {
    using G = Geometry<BM, BN, WM, WN, true>;
    constexpr int NT = G::NT, TM = G::TM, TN = G::TN, MI = G::MI, NI = G::NI, NW = G::NW;
    constexpr int AL = BM / 4;          // lanes that hold one k-octet of the A panel
    constexpr int CQ = NT / 8;          // columns per B load
    static_assert(BM == BN && NT == 2 * BM && (AL == 64 || AL == 32) && 3 * NW <= 24, "four rows and four columns x 8 k per thread");
    static_assert(MI == WN && NI == WM, "one reference block of rows and one of columns per wavefront");

    auto& op = sm.op;
    Thread th = make_thread<G, true>(a, tm, tn);
    const int tid = th.tid, wm = th.wm, wn = th.wn, l32 = th.l32, hh = th.hh;
    const int mI = th.mI, nJ = th.nJ;
    const int nk = (a.K + KC - 1) / KC;
    if ((int64_t)(KC + 1) * a.lda * 2 >= (int64_t(1) << 31) || (int64_t)(BN + 1) * a.ldb * 2 >= (int64_t(1) << 31)) return false;
    if (a.M < 4 || a.K < 8) return false;

    // ---- staging: a thread holds rows 4 al .. 4 al + 3 of the eight k of
    // octet ao (all rows of an octet in one wavefront, so that e^T A needs no
    // sum across wavefronts), and octet bo of columns bc + CQ r.  These indices
    // and the LDS addresses made of them are derived from opaque_tid() where
    // they are used: kept over the k-loop they were spilled at 256 x 256, and
    // every reload waits for the loads in flight.
    constexpr int OW = 64 / AL;         // octets per wavefront
    const int wave = th.wave;
    struct Slot {
        int al, ao, bo, bc, lane;
    };
    auto slot_of = [&]() {
        const int t = opaque_tid(), l = t & 63;
        return Slot{l & (AL - 1), OW * wave + l / AL, l & 7, t >> 3, l};
    };

    if constexpr (FT > 0) {
        for (int x = tid; x < (int)sizeof(op.zero) / 4; x += NT) reinterpret_cast<unsigned*>(&op.zero[0][0][0][0])[x] = 0u;
        clear_check(sm.ck, tid);
    }
    int fnext = 0, flogged = 0;
    if constexpr (INJ) gather_faults<G>(sm.ck, a, th);
    __syncthreads();

    // Loads have no alignment beyond an element's.  Elements outside the matrix
    // are given an offset past the resource's end and read as zero; a load
    // that would straddle the last row of the tile or the last k is moved back
    // inside, and what it got is shifted (fix_a, fix_b).
    const unsigned short* const A = static_cast<const unsigned short*>(static_cast<const void*>(a.A));
    const unsigned short* const B = static_cast<const unsigned short*>(static_cast<const void*>(a.B));
    constexpr int kOutside = (int)0x80000000;
    constexpr int inset = 8;      // the bases lie eight elements early, so that a moved load's offset is not negative
    const int sA = (int)a.lda * 2, sB = CQ * (int)a.ldb * 2;
    const char* const baseA = reinterpret_cast<const char*>(A + th.i0 - inset) + (int64_t)(8 * OW * wave) * sA;
    const char* const baseB = reinterpret_cast<const char*>(B + (int64_t)th.j0 * a.ldb - inset);
    const int voffB = ((tid >> 3) * (int)a.ldb + 8 * (tid & 7) + inset) * 2;
    constexpr int kRsrcWord3 = 0x00020000;   // raw 32-bit data format
    u32x2 ra[8];
    u32x4 rb[4];
    auto load_a = [&](int p) {
        const int k0 = p * KC;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(baseA + (int64_t)k0 * sA), (short)0, 0x7fffffff, kRsrcWord3);
        const Slot q = slot_of();
        const int rem = mI - 4 * q.al;
        const int vo = rem > 0 ? (q.lane >= AL ? 8 * sA : 0) + (4 * q.al + inset - (rem < 4 ? 4 - rem : 0)) * 2 : kOutside;
        const int left = a.K - (k0 + 8 * (AL == 64 ? wave : q.ao));   // (uniform where a wavefront has one octet)
#pragma unroll
        for (int e = 0; e < 8; ++e) ra[e] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, e < left ? vo : kOutside, e * sA, 0));
    };
    auto load_b = [&](int p) {
        const int k0 = p * KC;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(baseB + (int64_t)k0 * 2), (short)0, 0x7fffffff, kRsrcWord3);
        int vo[4] = {voffB, voffB, voffB, voffB};
        if (!(k0 + KC <= a.K && nJ == BN)) {   // (no loads inside a branch: the waits for them were coarser)
            const Slot q = slot_of();
            const int rem = a.K - (k0 + 8 * q.bo);
            const int vk = rem > 0 ? voffB - (rem < 8 ? 8 - rem : 0) * 2 : kOutside;
#pragma unroll
            for (int r = 0; r < 4; ++r) vo[r] = q.bc + CQ * r < nJ ? vk : kOutside;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) rb[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo[r], r * sB, 0));
    };
    auto fix_a = [&]() {
        if ((mI & 3) != 0) {
            const int rem = mI - 4 * slot_of().al;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned long long v = __builtin_bit_cast(unsigned long long, ra[e]) >> (16 * (4 - (mI & 3)));
                ra[e] = rem > 0 && rem < 4 ? __builtin_bit_cast(u32x2, v) : ra[e];
            }
        }
    };
    auto fix_b = [&](int k0) {
        if ((a.K & 7) != 0 && k0 < a.K && k0 + KC > a.K) {
            const int rem = a.K - (k0 + 8 * slot_of().bo), s = 8 - (a.K & 7);
            const bool cut = rem > 0 && rem < 8;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                u32x4 v = rb[r];
                if (s & 1) v = u32x4{__builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16),
                                     __builtin_amdgcn_alignbit(v[3], v[2], 16), v[3] >> 16};
                if (s & 2) v = u32x4{v[1], v[2], v[3], 0u};
                if (s & 4) v = u32x4{v[2], v[3], 0u, 0u};
#pragma unroll
                for (int d = 0; d < 4; ++d) rb[r][d] = cut ? v[d] : rb[r][d];
            }
        }
    };

    // ---- registers -> LDS, squares and encodings (section 2.2, Eq. 1-2)
    constexpr int BLK = SUBS * 512;              // halves per block of 32 lines
    constexpr int BUF = BM / 32 * BLK;           // halves per panel
    // rows 4 al + r are units ua ^ r; columns CQ apart are CQ / 32 blocks apart
    unsigned short *pa = nullptr, *pb = nullptr;
    int ua = 0;
    auto address_a = [&](int buf) {
        const Slot q = slot_of();
        ua = unit_a((4 * q.al) & 31, q.ao);
        pa = &op.A[buf][q.al >> 3][q.ao >> 1][0][0];
    };
    auto address_b = [&](int buf) {
        const Slot q = slot_of();
        pb = &op.B[buf][q.bc >> 5][q.bo >> 1][unit_b(q.bc & 31, q.bo)][0];
    };
    float na[4] = {0.f, 0.f, 0.f, 0.f}, nb[4] = {0.f, 0.f, 0.f, 0.f};
    float ea[8], eb[8];
    auto row = [&](int r) {
        u32x4 y;
#pragma unroll
        for (int h = 0; h < 4; ++h)
            y[h] = __builtin_amdgcn_perm(ra[2 * h + 1][r >> 1], ra[2 * h][r >> 1], (r & 1) ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<u32x4*>(pa + 8 * (ua ^ r)) = y;
    };
    auto sum_a = [&](int quarter) {   // two of the eight k, from the row pairs as loaded
#pragma unroll
        for (int e = 2 * quarter; e < 2 * quarter + 2; ++e) {
            float x[4];
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                x[2 * d] = bf_lo(ra[e][d]);
                x[2 * d + 1] = bf_hi(ra[e][d]);
            }
            ea[e] = (x[0] + x[1]) + (x[2] + x[3]);
#pragma unroll
            for (int r = 0; r < 4; ++r) na[r] = fmaf(x[r], x[r], na[r]);
        }
        asm volatile("" : "+v"(na[0]), "+v"(na[1]), "+v"(na[2]), "+v"(na[3]));
    };
    auto column = [&](int r, int half) {
        if (half == 0) *reinterpret_cast<u32x4*>(pb + r * (CQ / 32) * BLK) = rb[r];
        if constexpr (FT > 0) {
#pragma unroll
            for (int h = 2 * half; h < 2 * half + 2; ++h) {
                const float lo = bf_lo(rb[r][h]), hi = bf_hi(rb[r][h]);
                eb[2 * h] = r == 0 ? lo : eb[2 * h] + lo;
                eb[2 * h + 1] = r == 0 ? hi : eb[2 * h + 1] + hi;
                nb[r] = fmaf(lo, lo, nb[r]);
                nb[r] = fmaf(hi, hi, nb[r]);
            }
            asm volatile("" : "+v"(nb[r]));
        }
    };
    // three bf16 parts of an encoding value
    auto parts = [&](float v, unsigned (&w)[3]) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            w[s] = pack_bf16(v, v);
            v -= bf_lo(w[s]);
        }
    };
    auto put_w = [&](int buf) {   // after the reduce-scatter over the octet's lanes: k = 8 ao + al / (AL / 8)
        const Slot q = slot_of();
        const int s = min(q.lane & (AL / 8 - 1), 2);   // each part by a lane of its own
        unsigned w[3];
        parts(ea[0], w);
        op.wenc[buf][q.ao >> 1][q.ao & 1][s][q.al / (AL / 8)] = (unsigned short)(s == 0 ? w[0] : s == 1 ? w[1] : w[2]);
    };
    auto put_v = [&](int buf) {   // k = 8 bo + (lane >> 3)
        const Slot q = slot_of();
        unsigned w[3];
        parts(eb[0], w);
#pragma unroll
        for (int s = 0; s < 3; ++s) op.venc[buf][q.bo >> 1][q.bo & 1][3 * wave + s][q.lane >> 3] = (unsigned short)w[s];
    };

    Acc<G> acc;
#pragma unroll
    for (int bi = 0; bi < MI; ++bi)
#pragma unroll
        for (int bj = 0; bj < NI; ++bj)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.0f;
    // References (Eq. 4) of row block wn and column block wm of the wave tile,
    // its blocks 0: the MFMA of an encoding fragment with the block's operand
    // fragment leaves line l % 32 in lane l and, over the registers and lane
    // halves, one partial sum per encoding row: rows 0-23 (registers 0-11) for
    // the rows of A, rows 24-26 (registers 12-15) for the columns of B.
    f32x16 E;
#pragma unroll
    for (int r = 0; r < 16; ++r) E[r] = 0.f;
    float rebase = 0.f;

    const unsigned short* const fa = &op.A[0][wm * (TM / 32)][0][0][0];
    const unsigned short* const fb = &op.B[0][wn * (TN / 32)][0][0][0];
    auto frag = [&](const unsigned short* p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p)); };

    auto step = [&](int p, auto parity) {
        constexpr int buf = decltype(parity)::value, nxt = buf ^ 1;
        // the vector work of the step in units, dealt out over the MFMAs
        constexpr int U = FT > 0 ? 22 : 12;
        auto unit = [&](int u) {
            if constexpr (FT > 0) {
                if (u < 4) { if (u == 0) fix_a(); sum_a(u); }
                else if (u < 8) { if (u == 4) address_a(nxt); row(u - 4); }
                else if (u == 8) load_a(p + 2);
                else if (u == 9) ReduceScatter<8, ilog2(AL) - 1, 0>::run(ea, opaque_tid() & 63);
                else if (u == 10) put_w(nxt);
                else if (u < 19) { if (u == 11) { fix_b((p + 1) * KC); address_b(nxt); } column((u - 11) >> 1, (u - 11) & 1); }
                else if (u == 19) load_b(p + 2);
                else if (u == 20) ReduceScatter<8, 5, 3>::run(eb, opaque_tid() & 63);
                else put_v(nxt);
            } else {
                if (u == 0) { fix_a(); address_a(nxt); }
                else if (u < 5) row(u - 1);
                else if (u == 5) load_a(p + 2);
                else if (u == 6) { fix_b((p + 1) * KC); address_b(nxt); }
                else if (u < 11) column(u - 7, 0);
                else load_b(p + 2);
            }
        };
        const int ln = opaque_tid() & 63, c32 = ln & 31, ch = ln >> 5;
        const int u = 8 * unit_a(c32, ch);
        const unsigned short* const pv = c32 < 3 * NW ? &op.venc[buf][0][ch][c32][0] : &op.zero[0][0][0][0];
        const unsigned short* const pw = c32 >= 24 && c32 < 27 ? &op.wenc[buf][0][ch][c32 - 24][0] : &op.zero[0][0][0][0];
        constexpr int S1 = MI + (FT > 0 ? 1 : 0), S = SUBS * S1;   // slots of two MFMAs
        constexpr int SU = S - 2;                                      // the last ones without vector work
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
            const int ub = 8 * unit_b(c32, 2 * s + ch);
            bf16x8 b[NI], f[2], ve = {}, we = {};
            auto row_frag = [&](int pos) { return frag(fa + buf * BUF + G::row_block(pos, wn) * BLK + s * 512 + u); };
            f[0] = row_frag(0);
            if constexpr (FT > 0) ve = frag(pv + s * (2 * (3 * NW + 1) * 8));
#pragma unroll
            for (int bj = 0; bj < NI; ++bj) b[bj] = frag(fb + buf * BUF + G::col_block(bj, wm) * BLK + s * 512 + ub);
            if constexpr (FT > 0) we = frag(pw + s * (2 * 4 * 8));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < S1; ++q) {
                const int bi = q - (S1 - MI);
                if (bi + 1 > 0 && bi + 1 < MI) f[(bi + 1) & 1] = row_frag(bi + 1);
                if (bi < 0) {
                    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ve, f[0], E, 0, 0, 0);
                    E = __builtin_amdgcn_mfma_f32_32x32x16_bf16(we, b[0], E, 0, 0, 0);
                } else {
#pragma unroll
                    for (int bj = 0; bj < NI; ++bj)
                        acc[bi < 0 ? 0 : bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[bj], f[bi & 1], acc[bi < 0 ? 0 : bi][bj], 0, 0, 0);
                }
                const int slot = s * S1 + q;
#pragma unroll
                for (int v = 0; v < U; ++v)
                    if (v * SU >= slot * U && v * SU < (slot + 1) * U) unit(v);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // the next step with a check (a counter: the remainder of t by a run-time
    // interval is some forty instructions)
    int next_check = a.check_interval >= nk ? nk - 1 : a.check_interval - 1;
    auto due = [&](int t) { return FT > 0 && t == next_check; };
    // the squares over the k prefix of step t, before the step stages the next panel
    auto put_norms = [&]() {
        const int t = opaque_tid();
        *reinterpret_cast<f32x4*>(&op.nrow[t / AL][4 * (t & (AL - 1))]) = f32x4{na[0], na[1], na[2], na[3]};
        float nn[4] = {nb[0], nb[1], nb[2], nb[3]};
        ReduceScatter<4, 2, 0>::run(nn, t & 63);
        op.ncol[(t >> 3) + CQ * ((t >> 1) & 3)] = nn[0];
    };
    auto post = [&](int t) -> bool {
        if constexpr (INJ) inject<G>(acc, sm.ck, a, th, t, fnext);
        if constexpr (FT > 0) {
            if (due(t)) {
                float r = ((E[0] + E[1]) + (E[2] + E[3])) + ((E[4] + E[5]) + (E[6] + E[7])) + ((E[8] + E[9]) + (E[10] + E[11]));
                float c = (E[12] + E[13]) + (E[14] + E[15]);
                r = swap_add<5>(r, r);
                c = swap_add<5>(c, c);
                if (hh == 0) {
                    op.rref[wm * TM + 32 * wn + l32] = r;
                    op.cref[wn * TN + 32 * wm + l32] = c;
                }
                __syncthreads();
                float n = 0.f, r0;
                if (th.row_role) {   // threads 0 .. BM - 1 own the rows, the others the columns
#pragma unroll
                    for (int o = 0; o < 8; ++o) n += op.nrow[o][tid];
                    r0 = op.rref[tid] + rebase;
                } else {
                    n = op.ncol[tid - BM];
                    r0 = op.cref[tid - BM] + rebase;
                }
                float ref = r0;
                check<G, FT, INJ>(acc, sm.ck, a, th, t, min((t + 1) * KC, a.K), ref, n, ref, n, fnext, flogged);
                rebase += ref - r0;
                next_check = nk - 1 - next_check > a.check_interval ? next_check + a.check_interval : nk - 1;
                return true;
            }
        }
        return false;
    };

    load_a(0);
    load_b(0);
    fix_a();
    fix_b(0);
    if constexpr (FT > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sum_a(q);
    }
    address_a(0);
    address_b(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        row(r);
        column(r, 0);
        column(r, 1);
    }
    load_a(1);
    load_b(1);
    if constexpr (FT > 0) {
        ReduceScatter<8, ilog2(AL) - 1, 0>::run(ea, opaque_tid() & 63);
        put_w(0);
        ReduceScatter<8, 5, 3>::run(eb, opaque_tid() & 63);
        put_v(0);
    }
    __syncthreads();
    auto advance = [&](int t, auto parity) {
        if (due(t)) put_norms();
        step(t, parity);
        if (!post(t)) __syncthreads();
    };
    for (int t = 0; t < nk; t += 2) {
        advance(t, std::integral_constant<int, 0>{});
        if (t + 1 < nk) advance(t + 1, std::integral_constant<int, 1>{});
    }
    finish_tile<G, FT>(acc, sm.ck, a, th, a.scale);
    return true;
}

}  // namespace bf16m
}  // namespace ftgemm_impl
