// What the kernels of one wavefront (or several) per matrix share: phase clocks, constants, movement of values between lanes.
#ifndef BED_WAVE_COMMON_HPP
#define BED_WAVE_COMMON_HPP
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bed_kernel.h"

namespace bed {

// Cycle counts per phase of one wavefront's work, for the phase-resolved profile
// (paper_2207_04228_amd/phase_profile.py builds a separate library with BED_PHASE_CLOCKS defined).
// In the product build every member is an empty inline function and the object holds nothing.
enum Phase { kPhLoad = 0, kPhTridiag, kPhBoundary, kPhFill, kPhSteady, kPhDrain, kPhStore, kPhIterations, kPhCount };
struct PhaseClock {
#ifdef BED_PHASE_CLOCKS
    unsigned long long last;
    unsigned long long acc[kPhCount];
    __device__ __forceinline__ void start() {
        for (int i = 0; i < kPhCount; ++i) acc[i] = 0;
        last = __builtin_readcyclecounter();
    }
    __device__ __forceinline__ void lap(int phase) {
        const unsigned long long t = __builtin_readcyclecounter();
        acc[phase] += t - last;
        last = t;
    }
    __device__ __forceinline__ void count(int phase) { acc[phase] += 1; }
    __device__ __forceinline__ void write(unsigned long long* out, int b, int lane) const {
        if (out && lane == 0)
            for (int i = 0; i < kPhCount; ++i) out[(size_t)b * kPhCount + i] = acc[i];
    }
#else
    __device__ __forceinline__ void start() {}
    __device__ __forceinline__ void lap(int) {}
    __device__ __forceinline__ void count(int) {}
    __device__ __forceinline__ void write(unsigned long long*, int, int) const {}
#endif
};

namespace {

// Relative deflation tolerance: |e_k| <= kEps (|d_k| + |d_k+1|), kEps = 4 * 2^-23.  Inside a
// cluster of (nearly) equal eigenvalues the recurrence leaves off-diagonals at the rounding
// level of the diagonal, one to two units in the last place of d; a tolerance of 2^-23 is only
// two such units when d is just above a power of two, and windows of repeated eigenvalues then
// hover around it without ever deflating.
constexpr float kEps = 4.7683716e-7f;
// The pair of sweeps with both eigenvalues of the trailing block has fixed points (the 3x3
// matrix with diagonal 1, 0, 1 and off-diagonals 1 is mapped onto itself up to signs), as the
// double-shift QR step has in general.  After this many iterations without any deflation both
// sweeps use the eigenvalue closer to the last diagonal entry, which leaves such a point.
constexpr uint32_t kExceptionalAfter = 5;
constexpr uint32_t kStallIterations = 12;   // iterations without any deflation before the absolute threshold applies
constexpr float kAbsTol1 = 2.3841858e-7f;   // 2^-22 of the pre-scaled matrix
constexpr float kAbsTol2 = 9.5367432e-7f;   // 2^-20
constexpr float kTinyE = 1.0e-18f;      // absolute floor for |e| (matrix is pre-scaled to max|a| in [0.5,1))
constexpr float kTinyG = 1.0e-18f;      // floor for |g| in a rotation (keeps f^2+g^2 a normal number)
constexpr float kTinyAlpha = 1.0e-35f;  // |x|^2 below this: column already reduced, reflector skipped

// ---- cross-lane helpers ---------------------------------------------------

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp0(float x) {
    // lanes not selected by ROW_MASK (or reading out of range) receive 0
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xF, false));
}

constexpr int kQuadXor1 = 0xB1;       // quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;       // quad_perm [2,3,0,1]
constexpr int kRowHalfMirror = 0x141;
constexpr int kRowMirror = 0x140;
constexpr int kRowBcast15 = 0x142;    // lane 15 of each row -> every lane of the next row
constexpr int kRowBcast31 = 0x143;    // lane 31 -> every lane of rows 2 and 3

// A workgroup is one wavefront, and a wavefront's LDS operations complete in
// program order, so data written to LDS by one lane is visible to a later read
// by another lane without a hardware barrier.  This only stops the compiler
// from moving memory operations across the point.
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

__device__ __forceinline__ float read_lane(float x, int lane_uniform) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane_uniform));
}

// Lanes 0..31 keep `keep`; lane 32 + i receives the value lane i holds in `src`
// (v_permlane32_swap exchanges the upper half of its first operand with the lower half of
// its second; the first result is the first operand after the exchange).
__device__ __forceinline__ float upper_from_lower(float keep, float src) {
    return __uint_as_float(
        __builtin_amdgcn_permlane32_swap(__float_as_uint(keep), __float_as_uint(src), false, false)[0]);
}

// Every lane receives the value lane 32 + (i & 31) holds: the second result of the same
// exchange applied to two copies of x is x with its upper half copied over its lower half.
__device__ __forceinline__ float from_upper_half(float x) {
    const unsigned u = __float_as_uint(x);
    return __uint_as_float(__builtin_amdgcn_permlane32_swap(u, u, false, false)[1]);
}

// Lanes 0..31 keep `keep`; lanes 32..63 receive the value lane 31 holds in `src`
// (DPP row_bcast31 restricted to rows 2 and 3): one instruction hands a value that is
// uniform over the lower half to the upper half.
__device__ __forceinline__ float upper_from_lane31(float keep, float src) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(keep), __float_as_int(src), kRowBcast31, 0xC, 0xF, false));
}

// Sum over lanes [0, W) of the wave (W = 8, 16, 32 or 64, lanes outside must
// hold 0 or are ignored), returned as a wave-uniform value.  Quad butterflies,
// then mirrors (which act as xor 4 / xor 8 on quad-uniform values), then row
// broadcasts; no LDS traffic.
template <int W>
__device__ __forceinline__ float wave_sum(float x) {
    x += dpp0<kQuadXor1>(x);
    x += dpp0<kQuadXor2>(x);
    x += dpp0<kRowHalfMirror>(x);
    if (W >= 16) x += dpp0<kRowMirror>(x);
    if (W <= 16) return read_lane(x, 0);
    x += dpp0<kRowBcast15, 0xA>(x);
    if (W == 32) return read_lane(x, 31);
    x += dpp0<kRowBcast31, 0xC>(x);
    return read_lane(x, 63);
}

// Same for max of non-negative values.
template <int W>
__device__ __forceinline__ float wave_max_nonneg(float x) {
    x = fmaxf(x, dpp0<kQuadXor1>(x));
    x = fmaxf(x, dpp0<kQuadXor2>(x));
    x = fmaxf(x, dpp0<kRowHalfMirror>(x));
    if (W >= 16) x = fmaxf(x, dpp0<kRowMirror>(x));
    if (W <= 16) return read_lane(x, 0);
    x = fmaxf(x, dpp0<kRowBcast15, 0xA>(x));
    if (W == 32) return read_lane(x, 31);
    x = fmaxf(x, dpp0<kRowBcast31, 0xC>(x));
    return read_lane(x, 63);
}

constexpr int lanes_for(int n) { return n <= 8 ? 8 : (n <= 16 ? 16 : (n <= 32 ? 32 : 64)); }

// Every lane takes part, so nothing is kept of the destination and the move folds into the instruction that uses it.
template <int CTRL>
__device__ __forceinline__ float dpp_full(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Every lane receives the value lane (i & 31) holds.
__device__ __forceinline__ float lower_to_both(float x) {
    const unsigned u = __float_as_uint(x);
    return __uint_as_float(__builtin_amdgcn_permlane32_swap(u, u, false, false)[0]);
}

// f(std::integral_constant<int, I>) for I in [A, B): indices that are constants of the instruction
template <int A, int B, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}

// Monotone map float -> uint32 (total order; NaNs land at the ends).
__device__ __forceinline__ uint32_t sort_key(float x) {
    uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// exact power-of-two scale bringing amax into [0.5, 1); 1 for 0 / non-finite
__device__ __forceinline__ void pow2_scale(float amax, float& scale, float& inv_scale) {
    int ex = 0;
    if (amax > 0.f && amax < __builtin_inff()) ex = __builtin_amdgcn_frexp_expf(amax);
    ex = min(max(ex, -125), 126);
    scale = ldexpf(1.0f, -ex);
    inv_scale = ldexpf(1.0f, ex);
}

}  // namespace

}  // namespace bed
#endif
