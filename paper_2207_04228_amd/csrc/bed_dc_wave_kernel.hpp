// n <= 32: tridiagonalisation in registers (shared with wave_kernel), divide and conquer on the
// tridiagonal, one wavefront per matrix; two threads per eigenvalue (four for n <= 16).
#ifndef BED_DC_WAVE_KERNEL_HPP
#define BED_DC_WAVE_KERNEL_HPP
#include "bed_dc.hpp"

namespace bed {

template <int N, bool WANT_V, int STAGE>
__global__ __launch_bounds__(64) void dc_wave_kernel(KernelArgs args) {
    static_assert(N <= 32, "one 32 x 32 tile");
    constexpr int R = N <= 16 ? 16 : 32;             // rows covered by the tile
    using Shared = DcShared<R, 64 / R, WANT_V>;
    using Acc = typename DcTile<R>::acc;
    constexpr int LD = Shared::LD;
    constexpr int SLD = 33;                          // stride of the tridiagonalisation's buffer
    constexpr int KT = 64 / R;                       // columns per matrix instruction
    constexpr int KS = (N + KT - 1) / KT;            // steps of a product over N columns
    constexpr int AR = R * R / 64;
    __shared__ Shared S;
    __shared__ float2 sP[N + 2];
    // staging of A, then P (column-major); the eigenvector arrays serve where they are large enough
    constexpr bool OWN = !WANT_V || R < 32;
    __shared__ float stage_own[OWN ? N * SLD : 1];
    float* const stage = OWN ? stage_own : S.V;

    const int lane = threadIdx.x;
    const int lo = lane & (R - 1), hi = lane / R;
    const int b = blockIdx.x;
    const int n = args.n;
    float inv_scale = 1.f;
    PhaseClock clk;
    auto sync = []() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    // P stays in registers as the left operand of the last product: pa[s] = P[lane % R][KT s + lane / R].  The columns from n on meet
    // rows of V that are zero.
    float pa[WANT_V ? KS : 1];
    {
        float x[N];
        tridiag_rows<N, SLD, WANT_V>(args.A + (size_t)b * n * n, n, lane, stage, sP, inv_scale, x, clk);
        if constexpr (WANT_V) {
            // row r of P is in lane 32 + r
            auto upper = [](float a, float c) {          // of a below, of c above
                return __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(c), false, false)[1];
            };
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if constexpr (KT == 2) {
                    pa[s] = __uint_as_float(upper(x[2 * s], x[2 * s + 1]));
                } else {
                    const unsigned even = upper(x[4 * s], x[4 * s + 2]), odd = upper(x[4 * s + 1], x[4 * s + 3]);
                    pa[s] = __uint_as_float(__builtin_amdgcn_permlane16_swap(even, odd, false, false)[0]);
                }
            }
        }
    }
    sync();

    const int unresolved = dc_solve<R, 64, WANT_V>(
        S, n, lane, [&](int k) { return sP[k].y; }, [&](int k) { return sP[k + 1].x; });

    // column `lo` of the result, in every group of R lanes
    const float lam = S.D[lo] * inv_scale;
    const int odd = dc_non_finite(S, n, lane);
    {
        const int e = lane / KT, part = lane % KT;
        const int at = dc_rank(S, n, e, part, odd != 0);
        if (part == 0) {
            S.perm[e] = at;
            if (args.evals && e < n) args.evals[(size_t)b * n + at] = S.D[e] * inv_scale;
        }
    }
    sync();
    const int rank = S.perm[lo];
    if (lane == 0 && args.info) args.info[b] = odd + unresolved;

    if constexpr (WANT_V) {
        // V = P V_T
        Acc acc{};
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = dc_mfma(pa[s], S.V[(KT * s + hi) * LD + lo], acc);
        if (STAGE == kFull || args.evecs) {
            float* __restrict__ Vb = args.evecs + (size_t)b * n * n;
#pragma unroll
            for (int v = 0; v < AR; ++v) {
                const int r = dc_row<R>(v, lane);
                if (r < n && lo < n) Vb[r * n + rank] = acc[v];
            }
        }
        if (STAGE == kSpectral) {
            // F = (V f(max(Lambda, floor))) V^T (Sec. 4.2-4.4): both operands are the same entry of V
#pragma unroll
            for (int v = 0; v < AR; ++v) S.U[dc_row<R>(v, lane) * LD + lo] = acc[v];
            const float x = fmaxf(lam, args.fn_floor);
            const float f = (args.fn == kFnInvSqrt) ? __builtin_amdgcn_rsqf(x) : __builtin_amdgcn_sqrtf(x);
            S.rn[lo] = lo < n ? f : 0.f;
            sync();
            Acc out{};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const float vk = S.U[lo * LD + KT * s + hi];
                out = dc_mfma(vk * S.rn[KT * s + hi], vk, out);
            }
            float* __restrict__ Fb = args.fn_out + (size_t)b * n * n;
#pragma unroll
            for (int v = 0; v < AR; ++v) {
                const int r = dc_row<R>(v, lane);
                if (r < n && lo < n) Fb[r * n + lo] = out[v];
            }
        }
    }
}

template <int N>
static hipError_t launch_dc_n(const KernelArgs& args, int stage, bool want_v, hipStream_t stream) {
    if (stage == kSpectral) return enqueue(dc_wave_kernel<N, true, kSpectral>, dim3(args.batch), dim3(64), stream, args);
    return want_v ? enqueue(dc_wave_kernel<N, true, kFull>, dim3(args.batch), dim3(64), stream, args)
                  : enqueue(dc_wave_kernel<N, false, kFull>, dim3(args.batch), dim3(64), stream, args);
}

}  // namespace bed
#endif
