// Householder tridiagonalisation (Sec. 3.1) of a symmetric matrix, 32 < n <= 128, held in the accumulators of the matrix cores,
// and the product with its reflectors.
//
// The matrix is cut into tiles of 32 x 32.  Step J applies reflector J - 1 (one matrix instruction per
// tile, rank 2: A <- A - u p^T - (p - 2K u) u^T) and forms its own p = A u as column sums of the tiles (A is
// symmetric): a lane adds up its own registers, then the lanes that share a column.  What bounds it is the
// serial chain of a column, so the chain is cut short: row J + 1 is taken from the tiles BEFORE the update and
// brought up to date beside the matrix instructions (a - u_J p - (p_J - 2K u_J) u, one or two entries per lane).  Up to 64
// rows one wavefront does all of it, with one LDS round trip a column (u in the order of the tiles' rows) and no barrier, or, where the chip
// has room, four wavefronts a tile each until one tile is left; beyond 64 rows three or four wavefronts own a strip of 32 columns each.  They exchange
// p and the next row, with ONE barrier a column: u^T p, the row and its norm are formed by each of them, the same bits.
// Matrix instructions in fp32 and multiply-adds of a wavefront do not overlap (64 cycles of a tile's update and 64 of its share of A u add up:
// with the update one step late and off the chain, 64x64 took as long), so what shortens a column is fewer of both in a wavefront.
// Finished rows and columns take part in the updates: what is left of them is T and rounding.
// The reflectors stay behind as the rows of R and are applied to the eigenvectors of T after the divide and conquer,
// sixteen at a time (compact WY form I - Y T Y^T, Schreiber and Van Loan 1989).
// The form before this one updated P beside A, in half of the wavefronts, with two barriers a column.
// Cycles from load to the end of the reduction, one matrix per compute unit: 64x64 130 k, 128x128 364 k; now 62 k (four wavefronts; one alone,
// two matrices per compute unit: 75 k) and 171 k, and 5 k and 8 k for the blocks of T.  A column costs 850 cycles with one tile left, 1270 with four (n <= 64) or in strips (128): 130 to 170
// instructions at 7.4 cycles, two sums over the wavefront, one LDS round trip and the matrix instructions in a chain.
#ifndef BED_TILE_TRIDIAG_HPP
#define BED_TILE_TRIDIAG_HPP
#include "bed_dc.hpp"

namespace bed {

// Row stride of R: rows start on 128 bits, and 16 rows at the same four columns lie in 64 different banks.
template <int N>
constexpr int kReflectorStride = N + 4;

// Reflector J: 2/|u|^2, and what is added to entry J + 1 of row J of R to make it u.
template <int N>
struct ReflectorFactors {
    float beta[N], sigma[N];
};

// The lower triangle of the matrix mirrored into `stage` (stride LD), T threads; returns the largest magnitude that this
// wavefront has seen (NaNs drop out; they reach T through the norm of their column).  CH loads per thread are in flight.
template <int T, int CH = 8>
__device__ __forceinline__ float load_symmetric(const float* __restrict__ Ab, const int n, const int tid, float* const stage,
                                                const int LD) {
    const float rcp_n = 1.0f / (float)n;
    float amax = 0.f;
    for (int base = tid; base < n * n; base += CH * T) {
        float t[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k) t[k] = base + k * T < n * n ? Ab[base + k * T] : 0.f;
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int idx = base + k * T;
            const int i = (int)(((float)idx + 0.5f) * rcp_n);
            const int j = idx - i * n;
            if (idx < n * n && j <= i) {
                amax = fmaxf(amax, fabsf(t[k]));
                stage[i * LD + j] = t[k];
                stage[j * LD + i] = t[k];
            }
        }
    }
    return wave_max_nonneg<64>(amax);
}

// Reflector of a column x with |x|^2 = alpha and first entry x0; left out (beta = 0: then p and all that follows from it are
// zero, whatever u is) where alpha is not above `limit`.  A NaN in the column counts as active and goes into T: an inactive step
// touches nothing, and no later step reads the column again.
struct Reflector {
    float sigma, beta, first;                          // added to the first entry of x, 2/|u|^2, first entry of u
    bool active;
    __device__ __forceinline__ Reflector(float alpha, float x0, float limit) {
        active = !(alpha <= limit);
        const float nrm = __builtin_amdgcn_sqrtf(alpha);
        sigma = copysignf(nrm, x0);                    // no cancellation
        // |u|^2/2 for the square root that was taken, and its reciprocal to the last bit: I - beta u u^T is then as
        // orthogonal as |x|^2 is accurate
        const float half = fmaf(fabsf(x0), nrm, 0.5f * fmaf(nrm, nrm, alpha));
        const float r = __builtin_amdgcn_rcpf(half);
        beta = active ? fmaf(fmaf(-half, r, 1.f), r, r) : 0.f;
        first = x0 + sigma;
    }
    static __device__ __forceinline__ float limit(int J, int n) { return J < n - 2 ? kTinyAlpha : __builtin_inff(); }
};

// What the loops leave per column, by index l: T, and the reflector.
template <int N>
__device__ __forceinline__ void finish_column(const float* const R, ReflectorFactors<N>& F, const int n, const int l,
                                              const float diagonal, const float alpha, float* const sd, float* const se) {
    const float x0 = l + 1 < n ? R[l * kReflectorStride<N> + l + 1] : 0.f;
    const Reflector H(alpha, x0, Reflector::limit(l, n));      // the same bits as in the loop
    sd[l] = diagonal;
    se[l] = H.active ? -H.sigma : x0;
    F.beta[l] = H.beta;
    F.sigma[l] = H.active ? H.sigma : 0.f;
}

// 32 < n <= 64, the first 32 columns by four wavefronts, a tile each (tile row wv / 2, tile column wv % 2); lanes hold the entry `lane` of a
// vector.  All four form u^T p, the row and its norm, the same bits, and exchange column sums and the next row, with one barrier a column.
struct TileExchange {
    float p[2][2][64];           // [step parity][tile row]: its share of A u by column
};
struct TileState {
    dc_acc32 x{};                // the last tile
    float a = 0.f, p = 0.f, un = 0.f, beta = 0.f, uJ = 0.f, dv = 0.f, av = 0.f;      // as in tridiag_wave
};
template <int LD>
__device__ __forceinline__ void tridiag_tiles(const float* const stage, float* const R, TileExchange& S, float (&rows)[2][64],
                                              TileState& out, const int n, const int lane, const int wv, const float scale) {
    constexpr int LR = kReflectorStride<64>;
    const int lo = lane & 31, hi = lane >> 5;
    const int t = wv >> 1, j = wv & 1, c = 32 * j + lo;
    dc_acc32 x;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = 32 * t + dc_row<32>(v, lane);
        const float entry = stage[r * LD + c];                  // within the buffer also from n on
        x[v] = (r < n && c < n) ? entry * scale : 0.f;
    }
    if (hi == 0) {
        S.p[0][t][c] = 0.f;
        if (t == 0) rows[0][c] = x[0];
    }
    __syncthreads();                                   // R may take the place of the matrix
    float p = 0.f, a = 0.f, un = 0.f, beta = 0.f, uJ = 0.f;     // as in tridiag_wave
    float dv = 0.f, av = 0.f;
    for (int J0 = 0; J0 < 32; J0 += 8) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int J = J0 + s, par = s & 1;
            p = beta * (S.p[par][0][lane] + S.p[par][1][lane]);
            a = rows[par][lane];
            const float K2 = -beta * wave_sum<64>(un * p);
            const float wJ = fmaf(-K2, uJ, read_lane(p, J));
            const float w = fmaf(K2, un, p);
            const float r = fmaf(wJ, un, fmaf(-uJ, p, a));
            const float row = lane > J ? r : 0.f;
            // every wavefront writes the row, the same bits, and reads back what it wrote itself
            R[J * LR + lane] = row;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const auto left = __builtin_amdgcn_permlane32_swap(__float_as_uint(un), __float_as_uint(w), false, false);
            const auto right = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(un), false, false);
            x = dc_mfma(__uint_as_float(t ? left[1] : left[0]), __uint_as_float(j ? right[1] : right[0]), x);
            const float alpha = wave_sum<64>(row * row);
            const Reflector H(alpha, read_lane(row, J + 1), Reflector::limit(J, n));
            dv = lane == J ? r : dv;
            av = lane == J ? alpha : av;
            un = lane == J + 1 ? -H.first : -row;
            beta = H.beta;
            uJ = H.first;
            const int sub = (s + 1) & 3, group = ((J + 1) >> 3) & 3;
            float part[4] = {0.f, 0.f, 0.f, 0.f}, next = x[sub];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const dc_acc16 u = *reinterpret_cast<const dc_acc16*>(R + J * LR + 32 * t + 8 * q + 4 * hi);
#pragma unroll
                for (int v = 0; v < 4; ++v) part[v] = fmaf(x[4 * q + v], u[v], part[v]);
                next = q == group ? x[4 * q + sub] : next;
            }
            const unsigned bits = __float_as_uint(next);
            const auto y = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
            const float up = __uint_as_float(y[((s + 1) >> 2) & 1]);
            const unsigned half = __float_as_uint((part[0] + part[1]) + (part[2] + part[3]));
            const auto z = __builtin_amdgcn_permlane32_swap(half, half, false, false);
            const float sum = __uint_as_float(z[0]) + __uint_as_float(z[1]);
            const bool here = ((J + 1) >> 5) == t;     // row J + 1 is one of this tile's
            if (hi == 0) {
                S.p[par ^ 1][t][c] = here ? fmaf(H.sigma, up, sum) : sum;    // u is row J of R with sigma added to entry J + 1
                if (here) rows[par ^ 1][c] = up;
            }
            __syncthreads();
        }
    }
    out.x = x;
    out.p = beta * (S.p[0][0][lane] + S.p[0][1][lane]);
    out.a = rows[0][lane];
    out.un = un;
    out.beta = beta;
    out.uJ = uJ;
    out.dv = dv;
    out.av = av;
}

// One wavefront, n <= 64, a vector entry per lane.  stage: the symmetric matrix, stride LD; R may be the same memory and is
// left with row J of R in row J (columns up to J zero).  sd, se: T.  tiled: columns 32 and up only, from the state
// that tridiag_tiles has left in the wavefront of the last tile.
template <int LD>
__device__ __forceinline__ void tridiag_wave(const float* const stage, float* const R, ReflectorFactors<64>& F, const int n,
                                             const int lane, const float scale, float* const sd, float* const se,
                                             const bool tiled, const TileState& state) {
    constexpr int NS = 2, LR = kReflectorStride<64>;
    const int lo = lane & 31, hi = lane >> 5;
    auto sync = []() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    dc_acc32 x[NS][NS];                                // x[t][j][v]: row 32 t + dc_row<32>(v, lane), column 32 j + lo
    float a = 0.f;                                     // row J before reflector J - 1
    float p = 0.f, un = 0.f, beta = 0.f, uJ = 0.f;     // p, -u and 2/|u|^2 of reflector J - 1, u_J
    float dv = 0.f, av = 0.f;                          // diagonal of T, |x|^2 of the columns
    if (tiled) {
        x[1][1] = state.x;
        a = state.a, p = state.p, un = state.un, beta = state.beta, uJ = state.uJ, dv = state.dv, av = state.av;
    } else {
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int j = 0; j < NS; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 32 * t + dc_row<32>(v, lane), c = 32 * j + lo;
                    const float entry = stage[r * LD + c];      // within the buffer also from n on
                    x[t][j][v] = (r < n && c < n) ? entry * scale : 0.f;
                }
        const float top = stage[lane];
        a = lane < n ? top * scale : 0.f;
        sync();                                        // R may take the place of the matrix
    }

    // columns 32 t0 and up are not finished; s, the step's place in the unrolled loop, names registers
    auto column = [&](const int J, const int s, const int t0) {
        const float K2 = -beta * wave_sum<64>(un * p);                              // 2K
        const float wJ = fmaf(-K2, uJ, read_lane(p, J));
        const float w = fmaf(K2, un, p);                                            // p - 2K u
        const float r = fmaf(wJ, un, fmaf(-uJ, p, a));                              // row J, all reflectors before it applied
        const float row = lane > J ? r : 0.f;
        R[J * LR + lane] = row;
        sync();
        // lanes 0..31 hold the operands of the first outer product, lanes 32..63 of the second
        const auto l = __builtin_amdgcn_permlane32_swap(__float_as_uint(un), __float_as_uint(w), false, false);
        const auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(un), false, false);
#pragma unroll
        for (int t = t0; t < NS; ++t)
#pragma unroll
            for (int j = t0; j < NS; ++j) x[t][j] = dc_mfma(__uint_as_float(l[t]), __uint_as_float(c[j]), x[t][j]);
        const float alpha = wave_sum<64>(row * row);
        const Reflector H(alpha, J < 63 ? read_lane(row, (J + 1) & 63) : 0.f, Reflector::limit(J, n));
        dv = lane == J ? r : dv;
        av = lane == J ? alpha : av;
        // column sums and row J + 1
        const int tile = (J + 1) >> 5, sub = (s + 1) & 3, group = ((J + 1) >> 3) & 3;
        float part[NS][4] = {}, next[NS] = {0.f, 0.f}, sum[NS];
#pragma unroll
        for (int t = t0; t < NS; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const dc_acc16 u = *reinterpret_cast<const dc_acc16*>(R + J * LR + 32 * t + 8 * q + 4 * hi);
#pragma unroll
                for (int j = t0; j < NS; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) part[j][v] = fmaf(x[t][j][4 * q + v], u[v], part[j][v]);
            }
#pragma unroll
        for (int j = t0; j < NS; ++j) {
            next[j] = x[t0][j][sub];
#pragma unroll
            for (int t = t0; t < NS; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) next[j] = (t == tile && q == group) ? x[t][j][4 * q + sub] : next[j];
        }
        un = lane == J + 1 ? -H.first : -row;
        beta = H.beta;
        uJ = H.first;
#pragma unroll
        for (int j = 0; j < NS; ++j) sum[j] = (part[j][0] + part[j][1]) + (part[j][2] + part[j][3]);
        // the halves of a column, and at the same time from strips to lanes
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(next[0]), __float_as_uint(next[1]), false, false);
        a = __uint_as_float(y[((s + 1) >> 2) & 1]);
        const auto z = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[0]), __float_as_uint(sum[1]), false, false);
        p = __uint_as_float(z[0]) + __uint_as_float(z[1]);
        p = beta * fmaf(H.sigma, a, p);                // u is row J of R with sigma added to entry J + 1
    };
    if (!tiled) {
        const int first = min(n, 32);
        for (int J0 = 0; J0 < first; J0 += 8) {
#pragma unroll
            for (int s = 0; s < 8; ++s)
                if (J0 + s < first) column(J0 + s, s, 0);
        }
    }
    for (int J0 = 32; J0 < n; J0 += 8) {
#pragma unroll
        for (int s = 0; s < 8; ++s)
            if (J0 + s < n) column(J0 + s, s, 1);
    }
    if (lane < n) finish_column<64>(R, F, n, lane, dv, av, sd, se);
    sync();
}

// 64 < n <= 32 NS: NS = 3 or 4 wavefronts, a strip of 32 columns each; lanes hold the entries `lane` and `lane + 64` of a vector.  Up to 96
// rows a fourth strip and tile row of zeros would cost 64 cycles of matrix instructions and 64 of multiply-adds a column: us per launch
// with four / three strips, 256 x 80x80 110.9 / 102.6, 256 x 96x96 125 / 115, eigenvalues of 256 x 80x80 87.5 / 77.5.
struct StripExchange {
    float p[2][128];             // [step parity]: A u by column
    float row[2][128];           // [step parity]: the next row
};
template <int LD, int NS>
__device__ __forceinline__ void tridiag_strips(const float* const stage, float* const R, ReflectorFactors<128>& F,
                                               StripExchange& S, const int n, const int tid, const float scale,
                                               float* const sd, float* const se) {
    constexpr int LR = kReflectorStride<128>;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lo = lane & 31, hi = lane >> 5;
    const int c = 32 * wv + lo;                        // this lane's column

    if (wv >= NS) {                                    // the same number of barriers
        if (wv == 3 && hi == 0) S.p[0][c] = S.p[1][c] = S.row[0][c] = S.row[1][c] = 0.f;       // the entries that nobody owns
        __syncthreads();
        for (int J = 0; J < n; ++J) __syncthreads();
        return;
    }
    dc_acc32 x[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = 32 * t + dc_row<32>(v, lane);
            const float entry = stage[r * LD + c];              // within the buffer also from n on
            x[t][v] = (r < n && c < n) ? entry * scale : 0.f;
        }
    if (hi == 0) {
        S.p[0][c] = 0.f;
        S.row[0][c] = x[0][0];
    }
    __syncthreads();                                   // R may take the place of the matrix

    float un[2] = {0.f, 0.f}, beta = 0.f, uJ = 0.f;    // -u and 2/|u|^2 of reflector J - 1, u_J
    float dv[2] = {0.f, 0.f}, av[2] = {0.f, 0.f};      // diagonal of T, |x|^2 of the columns
    const bool odd = wv & 1, upper = wv >> 1;

    // rows and columns 32 t0 and up are not finished
    auto column = [&](const int J, const int s, const int t0) {
        const int par = s & 1;
        float p[2], a[2], r[2], w[2], row[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            p[q] = beta * S.p[par][lane + 64 * q];
            a[q] = S.row[par][lane + 64 * q];
        }
        const float K2 = -beta * wave_sum<64>(fmaf(un[0], p[0], un[1] * p[1]));     // 2K
        const float wJ = fmaf(-K2, uJ, read_lane(t0 >= 2 ? p[1] : p[0], J & 63));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            w[q] = fmaf(K2, un[q], p[q]);
            r[q] = fmaf(wJ, un[q], fmaf(-uJ, p[q], a[q]));
            row[q] = lane + 64 * q > J ? r[q] : 0.f;
            // every wavefront writes the row, the same bits, and reads back what it wrote itself
            R[J * LR + lane + 64 * q] = row[q];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        {
            const auto cc = __builtin_amdgcn_permlane32_swap(__float_as_uint(upper ? p[1] : p[0]),
                                                             __float_as_uint(upper ? un[1] : un[0]), false, false);
            const float right = __uint_as_float(odd ? cc[1] : cc[0]);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (2 * q + 1 >= t0 && 2 * q < NS) {
                    const auto l = __builtin_amdgcn_permlane32_swap(__float_as_uint(un[q]), __float_as_uint(w[q]), false, false);
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (2 * q + k >= t0 && 2 * q + k < NS) x[2 * q + k] = dc_mfma(__uint_as_float(l[k]), right, x[2 * q + k]);
                }
            }
        }
        const int J1 = min(J + 1, 127);
        const float x0 = J + 1 < 128 ? read_lane(J1 >= 64 ? row[1] : row[0], J1 & 63) : 0.f;
        const float alpha = wave_sum<64>(fmaf(row[0], row[0], row[1] * row[1]));
        const Reflector H(alpha, x0, Reflector::limit(J, n));
        {
            constexpr int kBank[4] = {0, 0, 1, 1};
            const int q = kBank[t0];
            const bool here = lane == (J & 63);
            dv[q] = here ? r[q] : dv[q];
            av[q] = here ? alpha : av[q];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) un[q] = lane + 64 * q == J + 1 ? -H.first : -row[q];
        beta = H.beta;
        uJ = H.first;
        const int tile = (J + 1) >> 5, sub = (s + 1) & 3, group = ((J + 1) >> 3) & 3;
        float part[4] = {0.f, 0.f, 0.f, 0.f}, next = x[t0][sub];
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            if (t >= t0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const dc_acc16 u = *reinterpret_cast<const dc_acc16*>(R + J * LR + 32 * t + 8 * q + 4 * hi);
#pragma unroll
                    for (int v = 0; v < 4; ++v) part[v] = fmaf(x[t][4 * q + v], u[v], part[v]);
                    if (t <= t0 + 1) next = (t == tile && q == group) ? x[t][4 * q + sub] : next;
                }
            }
        }
        const unsigned bits = __float_as_uint(next);
        const auto y = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
        const float up = __uint_as_float(y[((s + 1) >> 2) & 1]);
        const unsigned half = __float_as_uint((part[0] + part[1]) + (part[2] + part[3]));
        const auto z = __builtin_amdgcn_permlane32_swap(half, half, false, false);
        const float sum = __uint_as_float(z[0]) + __uint_as_float(z[1]);
        if (hi == 0) {
            S.p[par ^ 1][c] = fmaf(H.sigma, up, sum);  // u is row J of R with sigma added to entry J + 1
            S.row[par ^ 1][c] = up;
        }
        __syncthreads();
    };
#pragma unroll
    for (int t0 = 0; t0 < NS; ++t0) {
        const int end = min(n, 32 * (t0 + 1));
        for (int J0 = 32 * t0; J0 < end; J0 += 8) {
#pragma unroll
            for (int s = 0; s < 8; ++s)
                if (J0 + s < end) column(J0 + s, s, t0);
        }
    }
    if (wv == 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int l = lane + 64 * q;
            if (l < n) finish_column<128>(R, F, n, l, dv[q], av[q], sd, se);
        }
    }
}

// The reflectors in the form in which they wait for the divide and conquer to end: T of this wavefront's block
// of sixteen as the left operand of X = T Z, and this thread's share of R.
template <int N>
struct Reflectors {
    static constexpr int kShare = N / 16;              // vectors of four entries of R per thread
    dc_acc16 rows[kShare];
    dc_acc16 t;
};

// R in LDS as the tridiagonalisation leaves it, visible to all threads.  Ends without a barrier.
template <int N>
__device__ __forceinline__ void take_reflectors(Reflectors<N>& H, const ReflectorFactors<N>& S, float* const R, const int n,
                                                const int tid) {
    constexpr int T = 4 * N, LR = kReflectorStride<N>;
    const int lane = tid & 63, wv = tid >> 6;
    const int i = lane & 15, g = lane >> 4;
    if (tid < n - 2) R[tid * LR + tid + 1] += S.sigma[tid];
    for (int k = n * N + tid; k < ((n + 13) & ~15) * N; k += T) R[(k / N) * LR + k % N] = 0.f;   // rows that fill the last block
    __syncthreads();
    const int J0 = 16 * wv;
    H.t = dc_acc16{};
    if (J0 < n - 2) {                                  // the same in all lanes of a wavefront
        // S = Y^T Y in 64 bits (both operands are the same entry of R, register v of the result is row 4 v + lane / 16):
        // the block is only as orthogonal as T fits Y.  With S in 32 bits V^T V - I was 10 % larger than
        // with P accumulated reflector by reflector, with this it is smaller.
        typedef double acc64 __attribute__((ext_vector_type(4)));
        acc64 s = acc64{};
        for (int k = J0; k < n; k += 16) {
            const dc_acc16 y = *reinterpret_cast<const dc_acc16*>(R + (J0 + i) * LR + k + 4 * g);
#pragma unroll
            for (int v = 0; v < 4; ++v) s = __builtin_amdgcn_mfma_f64_16x16x4f64((double)y[v], (double)y[v], s, 0, 0, 0);
        }
        // T = (diag(1/beta) + strictly upper part of S)^-1 with beta = 2 / S_jj; lane i has row i, from left to right
        const float f[4] = {(float)s[0], (float)s[1], (float)s[2], (float)s[3]};
        const float own_diag = i < 4 ? f[0] : i < 8 ? f[1] : i < 12 ? f[2] : f[3];      // S_ii where lane / 16 = i % 4
        const float b = S.beta[J0 + i] > 0.f ? 2.f / own_diag : 0.f;
        float t[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            float sum = i == j ? -1.f : 0.f;
#pragma unroll
            for (int k = 0; k < j; ++k) sum = fmaf(t[k], read_lane(f[k >> 2], 16 * (k & 3) + j), sum);
            t[j] = J0 + j < n - 2 ? -read_lane(b, 16 * (j & 3) + j) * sum : 0.f;
        }
        auto own = [&](int v) { return g == 0 ? t[v] : g == 1 ? t[4 + v] : g == 2 ? t[8 + v] : t[12 + v]; };
        H.t = dc_acc16{own(0), own(1), own(2), own(3)};
    }
#pragma unroll
    for (int k = 0; k < Reflectors<N>::kShare; ++k) {
        const int at = tid + k * T;
        H.rows[k] = *reinterpret_cast<const dc_acc16*>(R + (at / (N / 4)) * LR + 4 * (at % (N / 4)));
    }
}

// V <- H_0 H_1 ... V for this wavefront's columns 16 wv .. 16 wv + 15 of V, in accumulators: x[t][v] is row
// 16 t + 4 (lane / 16) + v.  R and the blocks of T (64 vectors each, by lane) in LDS.
template <int N>
__device__ __forceinline__ void apply_reflectors(dc_acc16 (&x)[N / 16], const float* const R, const dc_acc16* const T,
                                                 const int n, const int lane) {
    constexpr int LR = kReflectorStride<N>;
    const int i = lane & 15, g = lane >> 4;
    for (int blk = (n + 13) / 16 - 1; blk >= 0; --blk) {
        const dc_acc16 t = T[64 * blk + lane];
        dc_acc16 z[4] = {};                            // Z = Y^T V, four partial sums
#pragma unroll
        for (int k = 0; k < N / 16; ++k) {
            if (k >= blk && 16 * k < n) {
                const dc_acc16 y = *reinterpret_cast<const dc_acc16*>(R + (16 * blk + i) * LR + 16 * k + 4 * g);
#pragma unroll
                for (int v = 0; v < 4; ++v) z[v] = dc_mfma(y[v], x[k][v], z[v]);
            }
        }
        const dc_acc16 zz = (z[0] + z[1]) + (z[2] + z[3]);
        dc_acc16 w = dc_acc16{};                       // T Z
#pragma unroll
        for (int v = 0; v < 4; ++v) w = dc_mfma(t[v], zz[v], w);
#pragma unroll
        for (int k = 0; k < N / 16; ++k) {
            if (k >= blk && 16 * k < n) {
                // the sixteen products are summed before they meet V: one rounding at the size of V a block
                const float* const y = R + (16 * blk + 4 * g) * LR + 16 * k + i;
                dc_acc16 d = dc_acc16{};
#pragma unroll
                for (int v = 0; v < 4; ++v) d = dc_mfma(y[v * LR], w[v], d);
                x[k] -= d;
            }
        }
    }
}

}  // namespace bed
#endif
