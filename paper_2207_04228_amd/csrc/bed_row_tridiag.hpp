// Load, power-of-two pre-scaling and Householder tridiagonalisation (Sec. 3.1) of a symmetric matrix of at most 32 rows in one
// wavefront, a row per lane: lanes 0..31 hold the working matrix, lanes 32..63 the accumulated reflector product P (Eq. (8)), or the
// same rows once more where P is not wanted.  One instruction stream serves both: the dot product with u gives
// p = 2Au/|u|^2 below and w = 2Pu/|u|^2 above, and x <- x - q u^T is one half of the rank-2 update of A (q = p - 2K u) and the
// whole rank-1 update of P (q = w); the other half, x <- x - u p^T, runs with u = 0 above.
//
// What bounds it is the number of instructions: one wavefront issues one every 4.3 to 5 cycles whether the chip is full or not.  The
// entries of u and p are operands that the multiply-adds take from another lane of their row of 16 (DPP row_newbcast): 3 m
// instructions for m remaining columns and about 50 beside them; with a v_readlane for each entry, sums that ended in a scalar register and
// T stored column by column, as before, 5 m and 70.  The load takes a column per lane and constant address steps: 480 instructions at 32
// rows, 1130 with a division by n for each entry and the mirroring on the way back.  us per launch before / now: divide and conquer 512 x 32x32
// 33.3 / 29.9, 16384 x 32x32 261 / 243, 512 x 16x16 16.7 / 15.5, eigenvalues of 1000 x 23x23 23.3 / 22.0; rotations 512 x 8x8 13.8 / 13.4.
#ifndef BED_ROW_TRIDIAG_HPP
#define BED_ROW_TRIDIAG_HPP
#include "bed_wave_common.hpp"

namespace bed {

namespace {

// A vector whose entry r is in lane r of each half: lo, hi hold entries 0..15 and 16..31 in every row of 16 lanes.
template <int N>
struct Spread {
    float lo, hi;
    __device__ __forceinline__ explicit Spread(float v) {
        lo = hi = v;
        if constexpr (N > 16) {
            const unsigned b = __float_as_uint(v);
            const auto s = __builtin_amdgcn_permlane16_swap(b, b, false, false);
            lo = __uint_as_float(s[0]);
            hi = __uint_as_float(s[1]);
        }
    }
};

// The multiply-adds with an entry of a Spread for one factor, columns FIRST .. N-1, as assembly: the compiler folds no DPP move into a
// multiply-add.  FIRST selects the columns while the text is assembled.  The s_nop is the wait between a write of lo or hi and its
// use by another lane, which the compiler cannot see to here.  Nor can it see how far in front of the block's end an x[c] was written, and what
// another lane reads next is x[FIRST] (a move between halves, a v_readlane: two waits at most): the columns behind it stand in between, and the
// last block, which has one, ends with the wait.
#define BED_COL(c, insn) ".if %c[first] <= " #c "\n\t" insn " row_newbcast:" #c "-16*(" #c "/16) row_mask:0xf bank_mask:0xf\n\t.endif\n\t"
#define BED_AXPY(c, half) BED_COL(c, "v_fmac_f32_dpp %[x" #c "], %[" #half "], %[f]")
#define BED_DOT(c, half, p)                                                       \
    ".if %c[first] <= " #c " && " #c " < %c[first]+4 && %c[first]+4 <= %c[n]\n\t" \
    "v_mul_f32_dpp %[p" #p "], %[" #half "], %[x" #c "] row_newbcast:" #c "-16*(" #c "/16) row_mask:0xf bank_mask:0xf\n\t.else\n\t" \
    BED_COL(c, "v_fmac_f32_dpp %[p" #p "], %[" #half "], %[x" #c "]") ".endif\n\t"
#define BED_LAST ".if %c[first]+2 == %c[n]\n\ts_nop 1\n\t.endif\n\t"
#define BED_FOUR(op_, a, b, c, d) op_(a) op_(b) op_(c) op_(d)
#define BED_AL(c) BED_AXPY(c, lo)
#define BED_AH(c) BED_AXPY(c, hi)
#define BED_DOT4(half, a, b, c, d) BED_DOT(a, half, 0) BED_DOT(b, half, 1) BED_DOT(c, half, 2) BED_DOT(d, half, 3)
#define BED_XS(o_, a, b, c, d) [x##a] o_(x[a]), [x##b] o_(x[b]), [x##c] o_(x[c]), [x##d] o_(x[d])
#define BED_AXPY4 BED_FOUR(BED_AL, 0, 1, 2, 3)
#define BED_AXPY8 BED_AXPY4 BED_FOUR(BED_AL, 4, 5, 6, 7)
#define BED_AXPY12 BED_AXPY8 BED_FOUR(BED_AL, 8, 9, 10, 11)
#define BED_AXPY16 BED_AXPY12 BED_FOUR(BED_AL, 12, 13, 14, 15)
#define BED_AXPY20 BED_AXPY16 BED_FOUR(BED_AH, 16, 17, 18, 19)
#define BED_AXPY24 BED_AXPY20 BED_FOUR(BED_AH, 20, 21, 22, 23)
#define BED_AXPY28 BED_AXPY24 BED_FOUR(BED_AH, 24, 25, 26, 27)
#define BED_AXPY32 BED_AXPY28 BED_FOUR(BED_AH, 28, 29, 30, 31)
#define BED_DOT_4 BED_DOT4(lo, 0, 1, 2, 3)
#define BED_DOT_8 BED_DOT_4 BED_DOT4(lo, 4, 5, 6, 7)
#define BED_DOT_12 BED_DOT_8 BED_DOT4(lo, 8, 9, 10, 11)
#define BED_DOT_16 BED_DOT_12 BED_DOT4(lo, 12, 13, 14, 15)
#define BED_DOT_20 BED_DOT_16 BED_DOT4(hi, 16, 17, 18, 19)
#define BED_DOT_24 BED_DOT_20 BED_DOT4(hi, 20, 21, 22, 23)
#define BED_DOT_28 BED_DOT_24 BED_DOT4(hi, 24, 25, 26, 27)
#define BED_DOT_32 BED_DOT_28 BED_DOT4(hi, 28, 29, 30, 31)
#define BED_X4(o_) BED_XS(o_, 0, 1, 2, 3)
#define BED_X8(o_) BED_X4(o_), BED_XS(o_, 4, 5, 6, 7)
#define BED_X12(o_) BED_X8(o_), BED_XS(o_, 8, 9, 10, 11)
#define BED_X16(o_) BED_X12(o_), BED_XS(o_, 12, 13, 14, 15)
#define BED_X20(o_) BED_X16(o_), BED_XS(o_, 16, 17, 18, 19)
#define BED_X24(o_) BED_X20(o_), BED_XS(o_, 20, 21, 22, 23)
#define BED_X28(o_) BED_X24(o_), BED_XS(o_, 24, 25, 26, 27)
#define BED_X32(o_) BED_X28(o_), BED_XS(o_, 28, 29, 30, 31)
#define BED_ROW_OPS(N_)                                                                                                          \
    template <int FIRST>                                                                                                         \
    __device__ __forceinline__ void row_axpy(float (&x)[N_], const Spread<N_>& s, float f) {                                     \
        static_assert(FIRST + 2 <= N_, "");                                                                                      \
        asm("s_nop 1\n\t" BED_AXPY##N_ BED_LAST                                                                                  \
            : BED_X##N_("+v")                                                                                                    \
            : [lo] "v"(s.lo), [hi] "v"(s.hi), [f] "v"(f), [first] "n"(FIRST), [n] "n"(N_));                                      \
    }                                                                                                                            \
    template <int FIRST>                                                                                                         \
    __device__ __forceinline__ float row_dot(const float (&x)[N_], const Spread<N_>& s) {                                        \
        float p0 = 0.f, p1 = 0.f, p2 = 0.f, p3 = 0.f;                                                                            \
        if constexpr (FIRST + 4 <= N_)                                                                                           \
            asm("s_nop 1\n\t" BED_DOT_##N_                                                                                       \
                : [p0] "=&v"(p0), [p1] "=&v"(p1), [p2] "=&v"(p2), [p3] "=&v"(p3)                                                 \
                : BED_X##N_("v"), [lo] "v"(s.lo), [hi] "v"(s.hi), [first] "n"(FIRST), [n] "n"(N_));                              \
        else                                                                                                                     \
            asm("s_nop 1\n\t" BED_DOT_##N_                                                                                       \
                : [p0] "+&v"(p0), [p1] "+&v"(p1), [p2] "+&v"(p2), [p3] "+&v"(p3)                                                 \
                : BED_X##N_("v"), [lo] "v"(s.lo), [hi] "v"(s.hi), [first] "n"(FIRST), [n] "n"(N_));                              \
        return (p0 + p1) + (p2 + p3);                                                                                            \
    }
// x[c] += entry c of s * f, and the sum of x[c] * entry c of s, for c >= FIRST
BED_ROW_OPS(4)
BED_ROW_OPS(8)
BED_ROW_OPS(12)
BED_ROW_OPS(16)
BED_ROW_OPS(20)
BED_ROW_OPS(24)
BED_ROW_OPS(28)
BED_ROW_OPS(32)
#undef BED_ROW_OPS

// a . b over the rows of each half, in all of its lanes (its first 16 up to 16 rows)
template <int N>
__device__ __forceinline__ float half_dot(float a, float b) {
#pragma clang fp contract(off)
    float s = a * b;             // not contracted with the first sum: each step is one instruction
    s = s + dpp_full<kQuadXor1>(s);
    s = s + dpp_full<kQuadXor2>(s);
    s = s + dpp_full<kRowHalfMirror>(s);
    if constexpr (N > 8) s = s + dpp_full<kRowMirror>(s);
    if constexpr (N > 16) {
        const Spread<N> t(s);
        s = t.lo + t.hi;
    }
    return s;
}

}  // namespace

// sP[k] = (e[k-1], d[k]) on return (entries 0..N), x the lane's row of P; inv_scale undoes the scaling.  stage: N * LD floats.
template <int N, int LD, bool WANT_P>
__device__ __forceinline__ void tridiag_rows(const float* __restrict__ Ab, const int n, const int lane, float* const stage,
                                             float2* const sP, float& inv_scale, float (&x)[N], PhaseClock& clk) {
    static_assert(N <= 32 && LD > N, "rows in half a wavefront, a spare column");
    const int row = lane & 31;
    const bool upper = lane >= 32;
    // ---- lane j + CW h takes column j of the rows RW k + h, all in flight, and leaves it in its place and, below the diagonal, in the mirrored
    // one: a later instruction than the one that leaves what stands above the diagonal.  Only constants are added to the addresses.
    constexpr int CW = N == 8 ? 8 : N <= 16 ? 16 : 32, RW = 64 / CW;
    static_assert(N % RW == 0, "the rows of the last load exist");
    {
        const int col = lane % CW, h = lane / CW;
        float t[N / RW];
#pragma unroll
        for (int k = 0; k < N / RW; ++k) t[k] = Ab[min((RW * k + h) * n + col, n * n - 1)];
        if (n < CW) {                                           // the same in all lanes
#pragma unroll
            for (int k = 0; k < N / RW; ++k) t[k] = col < n && RW * k + h < n ? t[k] : 0.f;
        }
        float* const place = stage + h * LD + col;
        float* const mirror = stage + min(col, N - 1) * LD + h;
        float* const spare = reinterpret_cast<float*>(sP) + h;  // N floats, for what has no mirrored place
#pragma unroll
        for (int k = 0; k < N / RW; ++k) {
            place[RW * k * LD] = t[k];
            (col <= RW * k + h ? mirror : spare)[RW * k] = t[k];
        }
    }
    wave_sync();
    const float* const mine = stage + min(row, N - 1) * LD;
    float amax = 0.f;
    static_for<0, N>([&](auto c_) {
        constexpr int c = decltype(c_)::value;
        x[c] = mine[c];
        amax = fmaxf(amax, fabsf(x[c]));        // drops NaNs; they still reach T through the arithmetic
    });
    float scale;
    pow2_scale(wave_max_nonneg<32>(amax), scale, inv_scale);
    const float s = row < N && !(WANT_P && upper) ? scale : 0.f;
    static_for<0, N>([&](auto c_) {
        constexpr int c = decltype(c_)::value;
        x[c] *= s;
        if (WANT_P) x[c] = lane == 32 + c ? 1.f : x[c];
    });
    wave_sync();
    clk.lap(kPhLoad);

    // ---- column J reduced at step J; a column that is reduced already runs with beta = 0
    float dv = 0.f, ev = 0.f;            // T: d[row], e[row]
    static_for<0, N>([&](auto J_) {
        constexpr int J = decltype(J_)::value;
        // row J of A, by lane (symmetric), in both halves
        float a = x[J];
        if constexpr (WANT_P) a = lower_to_both(a);
        const bool here = row == J;
        dv = here ? a : dv;
        if constexpr (J < N - 1) {
            const float x0 = read_lane(x[J], J + 1);            // A[J+1][J]
            float eJ = x0;
            if constexpr (J < N - 2) {
                const float xc = row > J ? a : 0.f;
                const float alpha = half_dot<N>(xc, xc);
                const bool active = J < n - 2 && alpha > kTinyAlpha;
                const float nrm = __builtin_amdgcn_sqrtf(alpha);
                const float sigma = x0 < 0.f ? -nrm : nrm;  // sign chosen to avoid cancellation
                const float u = row == J + 1 ? x0 + sigma : xc;
                const float beta = active ? __builtin_amdgcn_rcpf(fmaf(fabsf(x0), nrm, alpha)) : 0.f;       // 2/|u|^2
                eJ = active ? -sigma : x0;
                const Spread<N> us(u);
                const float p = beta * row_dot<J + 1>(x, us);              // above w
                // A - q u^T - u q^T with q = p - K u, K = u^T p / |u|^2, regrouped as A - u p^T - (p - 2K u) u^T: the first product does
                // not wait for K
                const float un = WANT_P && upper ? 0.f : -u;
                const Spread<N> ps(p);
                const float K2 = -beta * half_dot<N>(un, p);                            // 2K
                row_axpy<J + 1>(x, ps, un);
                row_axpy<J + 1>(x, us, fmaf(-K2, un, -p));                              // -(p - 2K u), above -w
                __builtin_amdgcn_sched_barrier(0);
            }
            ev = here ? eJ : ev;
        }
    });
    if constexpr (WANT_P) {
        // a matrix with a NaN or an infinity, which is in T by now, has no P
        if (__ballot(!(fabsf(dv) < __builtin_inff() && fabsf(ev) < __builtin_inff()))) {
            static_for<0, N>([&](auto c_) { x[decltype(c_)::value] = __builtin_nanf(""); });
        }
    }
    if (lane < N) {
        sP[lane].y = dv;
        sP[lane + 1].x = lane < n - 1 ? ev : 0.f;
    }
    if (lane == 0) sP[0].x = 0.f;
    wave_sync();
}

}  // namespace bed
#endif
