// 32 < n <= 128: tridiagonalisation in the accumulators of the matrix cores and divide and conquer on
// the tridiagonal, one workgroup per matrix: four wavefronts for n <= 64, eight beyond.
//
// P leaves LDS before the divide and conquer and waits in registers as the left operand of the last
// product V = P V_T (a strip of 32 rows per wavefront, N / 2 registers), so that V_T and the
// eigenvectors of the merges have the two matrix-sized areas of LDS to themselves.  Beside the poles of the
// root finder that is the limit at 128 rows: 256 registers and 14 to 16 spilled (none at 64, 168 registers).
// 256 matrices: 64x64 282 us with the rotations, 90 now; 128x128 1195, 239.
#include "bed_tile_tridiag.hpp"

namespace bed {

namespace {

template <int N, bool WANT_V, int STAGE>
__global__ __launch_bounds__(4 * N, N == 64 ? 3 : 2) void dc_block_kernel(KernelArgs args) {
    constexpr int DT = 4 * N;                        // threads per matrix
    using Shared = DcShared<N, DT / N, WANT_V>;
    constexpr int LD = Shared::LD;
    constexpr int KS = N / 2;                        // steps of a product over N columns
    constexpr int NTILE = N / 32, JSTEP = (DT / 64) / NTILE, TJ = NTILE / JSTEP;
    __shared__ Shared S;
    __shared__ TileShared<N> tiles;
    __shared__ float sd[N], se[N];
    __shared__ float stage_own[WANT_V ? 1 : N * LD];
    float* const stage = WANT_V ? S.V : stage_own;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int lo = lane & 31, hi = lane >> 5;
    const int I = wv % NTILE, J0 = wv / NTILE;       // this wavefront's tile row, its first tile column
    const int b = blockIdx.x;
    const int n = args.n;
    float inv_scale = 1.f;

    tridiag_tiles<N, WANT_V>(args.A + (size_t)b * n * n, n, tid, tiles, stage, sd, se, inv_scale);
    float pa[WANT_V ? KS : 1];                       // pa[s] = P[32 I + lane % 32][2 s + lane / 32]
    if constexpr (WANT_V) {
#pragma unroll
        for (int s = 0; s < KS; ++s) pa[s] = stage[(32 * I + lo) * LD + 2 * s + hi];
    }
    __syncthreads();

    const int unresolved = dc_solve<N, DT, WANT_V>(
        S, n, tid, [&](int k) { return sd[k]; }, [&](int k) { return se[k]; });

    const int odd = dc_non_finite(S, n, lane);
    if (tid == 0 && args.info) args.info[b] = odd + unresolved;
    if (tid < n) {
        const int rank = dc_rank(S, n, tid, odd != 0);
        S.perm[tid] = rank;
        if (args.evals) args.evals[(size_t)b * n + rank] = S.D[tid] * inv_scale;
    }
    if constexpr (WANT_V) {
        dc_acc32 acc[TJ];
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) acc[tj] = dc_acc32{};
        // V = P V_T
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (2 * s < n) {
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj)
                    acc[tj] = dc_mfma(pa[s], S.V[(2 * s + hi) * LD + 32 * (J0 + tj * JSTEP) + lo], acc[tj]);
            }
        }
        if (STAGE == kFull || args.evecs) {          // the same in all threads
            __syncthreads();                         // ranks
            float* __restrict__ Vb = args.evecs + (size_t)b * n * n;
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                const int c = 32 * (J0 + tj * JSTEP) + lo;
                const int rank = S.perm[c];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 32 * I + dc_row<32>(v, lane);
                    if (r < n && c < n) Vb[r * n + rank] = acc[tj][v];
                }
            }
        }
        if (STAGE == kSpectral) {
            // F = (V f(max(Lambda, floor))) V^T (Sec. 4.2-4.4): both operands are rows of V
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int v = 0; v < 16; ++v) S.U[(32 * I + dc_row<32>(v, lane)) * LD + 32 * (J0 + tj * JSTEP) + lo] = acc[tj][v];
            if (tid < N) {
                const float x = fmaxf(S.D[tid] * inv_scale, args.fn_floor);
                const float f = (args.fn == kFnInvSqrt) ? __builtin_amdgcn_rsqf(x) : __builtin_amdgcn_sqrtf(x);
                S.rn[tid] = tid < n ? f : 0.f;
            }
            __syncthreads();
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[tj] = dc_acc32{};
#pragma unroll 4
            for (int k = 0; k < n; k += 2) {
                const float a = S.U[(32 * I + lo) * LD + k + hi] * S.rn[k + hi];
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) acc[tj] = dc_mfma(a, S.U[(32 * (J0 + tj * JSTEP) + lo) * LD + k + hi], acc[tj]);
            }
            float* __restrict__ Fb = args.fn_out + (size_t)b * n * n;
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                const int c = 32 * (J0 + tj * JSTEP) + lo;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 32 * I + dc_row<32>(v, lane);
                    if (r < n && c < n) Fb[r * n + c] = acc[tj][v];
                }
            }
        }
    }
}

template <int N>
hipError_t launch_size(const KernelArgs& args, int stage, bool want_v, hipStream_t stream) {
    if (stage == kSpectral) return enqueue(dc_block_kernel<N, true, kSpectral>, dim3(args.batch), dim3(4 * N), stream, args);
    return want_v ? enqueue(dc_block_kernel<N, true, kFull>, dim3(args.batch), dim3(4 * N), stream, args)
                  : enqueue(dc_block_kernel<N, false, kFull>, dim3(args.batch), dim3(4 * N), stream, args);
}

}  // namespace

hipError_t launch_dc_block(const KernelArgs& args, int stage, bool want_v, hipStream_t stream) {
    return args.n <= 64 ? launch_size<64>(args, stage, want_v, stream) : launch_size<128>(args, stage, want_v, stream);
}

}  // namespace bed
