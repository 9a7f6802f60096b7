// Load, power-of-two pre-scaling and Householder tridiagonalisation (Sec. 3.1) of one matrix,
// 32 < n <= 128, with the working matrix and P^T in the accumulators of the matrix cores.
//
// Each wavefront owns a strip of 32 columns of A or of P^T (N / 32 tiles of 32 x 32, 16 registers
// each).  Both are updated by outer products with the reflector u,
//   A   <- A   - u p^T - (p - 2K u) u^T      (rank 2: one v_mfma_f32_32x32x2_f32 per tile),
//   P^T <- P^T - u w^T                       (rank 1: the same instruction with a zero column),
// and both products p = A u and w = P u are column sums of the strips (A is symmetric), so a lane
// adds up its own registers and only the two halves of the wavefront have to be combined.  Column J
// is read off as row J.  Rows up to J are finished: their tiles drop out.
// The earlier form of this phase, matrix and P in LDS, read and wrote every entry twice per step: 391 us
// for 256 matrices of 128x128 where the LDS traffic alone took most of it.  Around the same divide and conquer the call
// took 495 us with it and 260 with this.
#ifndef BED_TILE_TRIDIAG_HPP
#define BED_TILE_TRIDIAG_HPP
#include "bed_dc.hpp"

namespace bed {

template <int N>
struct TileShared {
    alignas(16) float u[N];      // row J right of the diagonal, zero up to J
    float p[N];
    float k[N / 32];             // partial sums of u^T p, one per strip
    float amax[N / 16];
};

// stage: N rows of stride N + 1, left with P[r][c] at stage[r * (N + 1) + c] when it is wanted.
// sd, se: T.  Threads: 4 N (N / 32 wavefronts for A, as many for P).  Ends with a barrier.
template <int N, bool WANT_P>
__device__ __forceinline__ void tridiag_tiles(const float* __restrict__ Ab, const int n, const int tid,
                                              TileShared<N>& S, float* const stage, float* const sd, float* const se,
                                              float& inv_scale) {
    constexpr int T = 4 * N, NS = N / 32, LD = N + 1;
    const int lane = tid & 63, wv = tid >> 6;
    const int lo = lane & 31, hi = lane >> 5;
    const bool isA = wv < NS;
    const int c = 32 * (isA ? wv : wv - NS) + lo;      // this lane's column
    const bool works = isA || WANT_P;

    // ---- lower triangle mirrored into LDS; pre-scaling from its largest entry ----
    {
        const float rcp_n = 1.0f / (float)n;
        float amax = 0.f;
        for (int base = tid; base < n * n; base += 8 * T) {
            float t[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) t[k] = base + k * T < n * n ? Ab[base + k * T] : 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int idx = base + k * T;
                const int i = (int)(((float)idx + 0.5f) * rcp_n);
                const int j = idx - i * n;
                if (idx < n * n && j <= i) {
                    amax = fmaxf(amax, fabsf(t[k]));   // drops NaNs; they reach T through the norm of their column
                    stage[i * LD + j] = t[k];
                    stage[j * LD + i] = t[k];
                }
            }
        }
        amax = wave_max_nonneg<64>(amax);
        if (lane == 0) S.amax[wv] = amax;
    }
    __syncthreads();
    float scale, top = S.amax[0];
#pragma unroll
    for (int w = 1; w < T / 64; ++w) top = fmaxf(top, S.amax[w]);
    pow2_scale(top, scale, inv_scale);

    dc_acc32 x[NS];                                    // x[t][v]: row 32 t + dc_row<32>(v, lane), column c
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = 32 * t + dc_row<32>(v, lane);
            const float a = (isA && r < n && c < n) ? stage[r * LD + c] * scale : 0.f;
            x[t][v] = isA ? a : ((r == c && c < n) ? 1.f : 0.f);
        }
    if (tid < N) S.p[tid] = 0.f;

    // entry of row `row` in this lane's column (one half of the wavefront holds it): registers are
    // indexed by compile-time constants, so `sub` = row % 4 comes from an unrolled loop
    auto pick = [&](int row, int sub) {
        const int tile = row >> 5, group = (row >> 3) & 3;
        float val = 0.f;
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) val = (t == tile && g == group) ? x[t][4 * g + sub] : val;
        return val;
    };

    for (int J0 = 0; J0 < n; J0 += 4) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int J = J0 + s;
            if (J < n) {                               // the same in all threads
                const int first = J >> 5;              // tiles above are finished
                if (isA) {
                    const float row = pick(J, s);
                    if (hi == ((J >> 2) & 1)) {
                        S.u[c] = c > J ? row : 0.f;
                        if (c == J) sd[J] = row;
                    }
                }
                __syncthreads();
                const float x0 = J + 1 < n ? S.u[J + 1 < N ? J + 1 : 0] : 0.f;
                float sq = S.u[lane] * S.u[lane];
                if (N > 64) sq = fmaf(S.u[(lane + 64) & (N - 1)], S.u[(lane + 64) & (N - 1)], sq);
                const float alpha = wave_sum<64>(sq);
                // a NaN in the column counts as active and goes into T: an inactive step touches nothing, and
                // no later step reads the column again
                const bool active = J < n - 2 && !(alpha <= kTinyAlpha);
                if (tid == 0) {
                    const float nrm = __builtin_amdgcn_sqrtf(alpha);
                    se[J] = active ? (x0 < 0.f ? nrm : -nrm) : x0;
                }
                if (active) {                          // the same in all threads
                    const float nrm = __builtin_amdgcn_sqrtf(alpha);
                    const float sigma = (x0 < 0.f) ? -nrm : nrm;       // sign chosen to avoid cancellation
                    const float beta = __builtin_amdgcn_rcpf(fmaf(fabsf(x0), nrm, alpha));    // 2/|u|^2
                    // u is the row in LDS with sigma added to entry J + 1
                    float pc = 0.f;
                    // entries of u that this lane needs after the second barrier: by then a wavefront that is
                    // ahead may write the next row over it
                    float ur[NS];
#pragma unroll
                    for (int t = 0; t < NS; ++t) ur[t] = S.u[32 * t + lo] + (32 * t + lo == J + 1 ? sigma : 0.f);
                    if (works) {
                        float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int t = 0; t < NS; ++t) {
                            if (t >= first && 32 * t < n) {
#pragma unroll
                                for (int g = 0; g < 4; ++g) {
                                    const float4 w = *reinterpret_cast<const float4*>(S.u + 32 * t + 8 * g + 4 * hi);
                                    part[0] = fmaf(x[t][4 * g + 0], w.x, part[0]);
                                    part[1] = fmaf(x[t][4 * g + 1], w.y, part[1]);
                                    part[2] = fmaf(x[t][4 * g + 2], w.z, part[2]);
                                    part[3] = fmaf(x[t][4 * g + 3], w.w, part[3]);
                                }
                            }
                        }
                        const float next = hi == (((J + 1) >> 2) & 1) ? pick(J + 1, (s + 1) & 3) : 0.f;
                        float sum = fmaf(sigma, next, (part[0] + part[1]) + (part[2] + part[3]));
                        const unsigned bits = __float_as_uint(sum);
                        const auto both = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
                        pc = beta * (__uint_as_float(both[0]) + __uint_as_float(both[1]));
                    }
                    const float uc = S.u[c] + (c == J + 1 ? sigma : 0.f);
                    if (isA) {
                        if (hi == 0) S.p[c] = pc;
                        const float dot = wave_sum<32>(uc * pc);
                        if (lane == 0) S.k[wv] = dot;
                    }
                    __syncthreads();
                    if (works) {
                        float K2 = S.k[0];
#pragma unroll
                        for (int w = 1; w < NS; ++w) K2 += S.k[w];
                        K2 *= beta;                                    // 2K
                        const float right = hi == 0 ? pc : (isA ? uc : 0.f);
#pragma unroll
                        for (int t = 0; t < NS; ++t) {
                            if (t >= first && 32 * t < n) {
                                const float left = hi == 0 ? ur[t] : fmaf(-K2, ur[t], S.p[32 * t + lo]);
                                x[t] = dc_mfma(-left, right, x[t]);
                            }
                        }
                    }
                } else {
                    __syncthreads();                   // all have read the row
                }
            }
        }
    }
    __syncthreads();
    if (WANT_P && !isA) {
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) stage[c * LD + 32 * t + dc_row<32>(v, lane)] = x[t][v];
    }
    __syncthreads();
}

}  // namespace bed
#endif
