// 32 < n <= 128: tridiagonalisation in the accumulators of the matrix cores and divide and conquer on
// the tridiagonal, one workgroup per matrix: four wavefronts for n <= 64, eight beyond.
//
// The reflectors of the tridiagonalisation leave LDS before the divide and conquer and wait in registers (N / 4 of
// them), so that the eigenvectors of T and of the merges have the two matrix-sized areas of LDS to themselves.  Then
// they come back and are applied to V, sixteen columns per wavefront.  256 matrices, us per launch: 64x64 96 with P accumulated and leaves of
// two rows, 60 now; 128x128 245, 148.
#include "bed_tile_tridiag.hpp"

namespace bed {

namespace {

// Up to 64 rows the first 32 columns of the reduction, by four wavefronts up to this batch, by one beyond: as many matrices as this chip
// has compute units (a number measured here, not asked of the device).  Then each SIMD has one of the four to itself; with more workgroups on
// a compute unit what all four repeat competes with the other matrices.  The two add the tiles' shares of A u in different orders: other last bits.  us per launch, one wavefront / four: 256 x 64x64 64.2 / 60.0, eigenvalues 52.6 / 48.1, 256 x 36x36 eigenvalues
// 41.1 / 36.5; 384 x 64x64 71.0 / 72.0, 512 x 36x36 55.6 / 56.7, 768 x 36x36 61.6 / 71.4, 768 x 64x64 79.1 / 89.7.
constexpr int kTilesUpToBatch = 256;

template <int N, bool WANT_V, int STAGE>
__global__ __launch_bounds__(4 * N, N == 64 ? 3 : 2) void dc_block_kernel(KernelArgs args) {
    constexpr int DT = 4 * N;                        // threads per matrix
    using Shared = DcShared<N, DT / N, WANT_V>;
    constexpr int LD = Shared::LD, LR = kReflectorStride<N>;
    constexpr int NTILE = N / 32, JSTEP = (DT / 64) / NTILE, TJ = NTILE / JSTEP;
    __shared__ Shared S;
    __shared__ float sd[N], se[N];
    __shared__ alignas(16) float stage_own[WANT_V ? 4 : N * LR];
    // R takes V and the first rows of U, the blocks of T rows of U behind it
    float* const R = WANT_V ? S.V : stage_own;
    dc_acc16* const Tb = reinterpret_cast<dc_acc16*>(S.V + N * LR);
    static_assert(!WANT_V || N * LR + 16 * N <= (int)(sizeof(S.V) + sizeof(S.U)) / 4, "R and T in the matrix areas");
    // not in use before the divide and conquer
    ReflectorFactors<N>& factors = *reinterpret_cast<ReflectorFactors<N>*>(S.dz);
    StripExchange& strips = *reinterpret_cast<StripExchange*>(S.om);
    TileExchange& tiles = *reinterpret_cast<TileExchange*>(S.om);
    float (&tile_rows)[2][64] = *reinterpret_cast<float (*)[2][64]>(S.zs);
    static_assert(sizeof(tiles) <= sizeof(S.om) && sizeof(tile_rows) <= sizeof(S.zs), "");
    static_assert(sizeof(factors) <= sizeof(S.dz) && (N == 64 || sizeof(strips) <= sizeof(S.om)), "");

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int b = blockIdx.x;
    const int n = args.n;
    float inv_scale = 1.f;

    {
        const float seen = load_symmetric<DT>(args.A + (size_t)b * n * n, n, tid, R, LD);
        if (lane == 0) S.rn[wv] = seen;
        __syncthreads();
        float scale, top = S.rn[0];
#pragma unroll
        for (int w = 1; w < DT / 64; ++w) top = fmaxf(top, S.rn[w]);
        pow2_scale(top, scale, inv_scale);
        if constexpr (N == 64) {
            const bool tiled = args.batch <= kTilesUpToBatch;
            TileState state;
            if (tiled) tridiag_tiles<LD>(R, R, tiles, tile_rows, state, n, lane, __builtin_amdgcn_readfirstlane(wv), scale);
            if (wv == (tiled ? 3 : 0)) tridiag_wave<LD>(R, R, factors, n, lane, scale, sd, se, tiled, state);
        } else {
            if (n <= 96)
                tridiag_strips<LD, 3>(R, R, factors, strips, n, tid, scale, sd, se);
            else
                tridiag_strips<LD, 4>(R, R, factors, strips, n, tid, scale, sd, se);
        }
        __syncthreads();
    }
    Reflectors<N> H;
    if constexpr (WANT_V) take_reflectors<N>(H, factors, R, n, tid);
    __syncthreads();

    const int unresolved = dc_solve<N, DT, WANT_V>(
        S, n, tid, [&](int k) { return sd[k]; }, [&](int k) { return se[k]; });

    const int odd = dc_non_finite(S, n, lane);
    if (tid == 0 && args.info) args.info[b] = odd + unresolved;
    {
        const int e = tid / 4, part = tid % 4;
        const int rank = dc_rank(S, n, e, part, odd != 0);
        if (e < n && part == 0) {
            S.perm[rank] = e;
            if (args.evals) args.evals[(size_t)b * n + rank] = S.D[e] * inv_scale;
        }
    }
    if constexpr (WANT_V) {
        // V = H_0 H_1 ... V_T; this wavefront's columns 16 wv ..
        const int i = lane & 15, g = lane >> 4;
        dc_acc16 x[N / 16];
#pragma unroll
        for (int t = 0; t < N / 16; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[t][v] = S.V[(16 * t + 4 * g + v) * LD + 16 * wv + i];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < Reflectors<N>::kShare; ++k) {
            const int at = tid + k * DT;
            *reinterpret_cast<dc_acc16*>(R + (at / (N / 4)) * LR + 4 * (at % (N / 4))) = H.rows[k];
        }
        Tb[tid] = H.t;
        __syncthreads();
        if (16 * wv < n) apply_reflectors<N>(x, R, Tb, n, lane);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < N / 16; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) S.V[(16 * t + 4 * g + v) * LD + 16 * wv + i] = x[t][v];
        if (STAGE == kSpectral && tid < N) {
            const float y = fmaxf(S.D[tid] * inv_scale, args.fn_floor);
            const float f = (args.fn == kFnInvSqrt) ? __builtin_amdgcn_rsqf(y) : __builtin_amdgcn_sqrtf(y);
            S.rn[tid] = tid < n ? f : 0.f;
        }
        __syncthreads();
        if (STAGE == kFull || args.evecs) {          // the same in all threads
            // ascending order; the columns of V change places on the way to memory
            float* __restrict__ Vb = args.evecs + (size_t)b * n * n;
            const float rcp_n = 1.0f / (float)n;
            for (int base = tid; base < n * n; base += 8 * DT) {
                float t[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int idx = min(base + k * DT, n * n - 1);
                    const int r = (int)(((float)idx + 0.5f) * rcp_n);
                    t[k] = S.V[r * LD + S.perm[idx - r * n]];
                }
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (base + k * DT < n * n) Vb[base + k * DT] = t[k];
            }
        }
        if (STAGE == kSpectral) {
            // F = (V f(max(Lambda, floor))) V^T (Sec. 4.2-4.4): both operands are rows of V
            const int lo = lane & 31, hi = lane >> 5;
            const int I = wv % NTILE, J0 = wv / NTILE;       // this wavefront's tile row, its first tile column
            dc_acc32 acc[TJ];
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[tj] = dc_acc32{};
#pragma unroll 4
            for (int k = 0; k < n; k += 2) {
                const float a = S.V[(32 * I + lo) * LD + k + hi] * S.rn[k + hi];
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) acc[tj] = dc_mfma(a, S.V[(32 * (J0 + tj * JSTEP) + lo) * LD + k + hi], acc[tj]);
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
