// Gradients through the eigendecomposition on the matrix cores (gfx950, wave64).
//
// For A = V diag(lambda) V^T (Sec. 3.1 Eq. (1)) and a loss with upstream
// gradients g_lambda, g_V, first-order perturbation theory gives
//   g_A = V ( diag(g_lambda) + sym(K o (V^T g_V)) ) V^T,  K_ij = 1/(lambda_j - lambda_i),
// where the coupling K is either exact with a gap floor or replaced by its
// truncated geometric series (the Taylor polynomial the paper uses for the
// backward pass, App. B / App. B.1: degree 9).  For F = V f(max(Lambda, floor)) V^T
// (Sec. 4.2-4.4, App. B.1-B.3) the same structure holds with divided
// differences of f in place of K:
//   g_A = V ( Phi o (V^T sym(G) V) ) V^T.
//
// The three (four) n x n x n products are dense contractions and run on the fp32 matrix instructions (full fp32
// operands and accumulation).  Up to 32 rows one wavefront owns a matrix (or several) and every intermediate product
// stays in the accumulators (tile_grad_kernel); beyond, a wavefront owns 16 columns of every product and LDS holds the other
// operand (grad_kernel).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bed_kernel.h"

namespace bed {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// Register v of lane l of a result of v_mfma_f32_32x32x2_f32 is in row acc_row(v, l), column l % 32.
__device__ __forceinline__ int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

// 1 / x: the hardware reciprocal (one unit in the last place) and one Newton step; the division itself
// where one of the two would leave the normal range
__device__ __forceinline__ float reciprocal(float x) {
    if (!(fabsf(x) > 1e-37f && fabsf(x) < 1e37f)) return 1.0f / x;
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, r, 1.f), r, r);
}

// Couplings K of the pairs (a_v, b) = (lambda_i, lambda_j), i != j; ra, rb their reciprocals.  Exact with a gap floor, or the
// truncated series: with b the larger in magnitude, 1/(b - a) ~ (1/b) sum_{k<=degree} (a/b)^k; mirrored otherwise.  Equal
// magnitudes: the later index counts as the larger (later(v): is it j's?), which keeps K antisymmetric.  The
// recurrences of all V pairs run side by side: one after the other they took 2.3 us of a 10 us call (16 pairs a lane).
template <int V, typename Later>
__device__ __forceinline__ void couplings(float (&K)[V], const float (&a)[V], const float b, const float (&ra)[V], const float rb,
                                          Later&& later, int mode, int degree, float gap_floor) {
    if (mode == kGradExact) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float d = b - a[v];
            K[v] = (fabsf(d) >= gap_floor && d != 0.f) ? 1.0f / d : 0.f;
        }
        return;
    }
    float rho[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const bool big_b = fabsf(b) > fabsf(a[v]) || (fabsf(b) == fabsf(a[v]) && later(v));
        rho[v] = big_b ? a[v] * rb : b * ra[v];
        K[v] = 1.f;
    }
    for (int k = 0; k < degree; ++k)
#pragma unroll
        for (int v = 0; v < V; ++v) K[v] = fmaf(K[v], rho[v], 1.f);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const bool big_b = fabsf(b) > fabsf(a[v]) || (fabsf(b) == fabsf(a[v]) && later(v));
        const float kk = big_b ? K[v] * rb : -(K[v] * ra[v]);
        K[v] = (big_b ? b : a[v]) == 0.f ? 0.f : kk;
    }
}

// Divided difference of f~(x) = f(max(x, floor)) at (lambda_i, lambda_j); the derivative when they coincide.
__device__ __forceinline__ float divided_difference(float li, float lj, int mode, float floor) {
    const float ai = fmaxf(li, floor), aj = fmaxf(lj, floor);
    const float si = sqrtf(ai), sj = sqrtf(aj);
    // for unclamped arguments: (f(ai) - f(aj)) / (ai - aj) in a form without cancellation
    float phi = (mode == kGradSqrt) ? 1.0f / (si + sj) : -1.0f / (si * sj * (si + sj));
    if (li < floor || lj < floor) {
        // f~(li) - f~(lj) = (f(ai) - f(aj)); the denominator is the distance of the true eigenvalues
        phi = (ai == aj) ? 0.f : phi * ((ai - aj) / (li - lj));
    }
    return phi;
}

// ---- n <= 32: everything in registers ----
// Tiles of TS x TS on v_mfma_f32_32x32x2, 16x16x4 and 4x4x1 (16 blocks).  Lane l holds, in register v, the entry of row
// Tile::row(v, l) and column l % TS of a result; taken as it stands that is also a right operand (rows as the contracted
// index) and, for a symmetric matrix, a left one, as long as the other operand names its entries in the same
// order.  So with V by columns, vc[v] = V[row(v)][lo], and by rows, vr[v] = V[lo][row(v)],
//   C = V^T (sym(G) V):  T = mfma(gs, vc), C = mfma(vc, T);     C - C^T = V^T g_V - g_V^T V:  mfma(vc, gc), mfma(-gc, vc)
//   g_A = V (M V^T):     W = mfma(M, vr), g_A = mfma(vr, W)
// need no exchange at all; LDS only turns V (and G, for its symmetric part) once.
// Bound by the launch and one pass through the chain of products for small batches, by memory (three matrices) and the
// matrix cores for large ones.  us per launch of the spectral function's gradient, with every product through LDS (four and two
// matrices of up to 8 and 16 rows in a 32 x 32 tile) / this: 512 x 16x16 7.7 / 4.1 (4.0 is an empty launch), 512 x 32x32 8.8 / 5.7,
// 65536 x 4x4 33 / 4.6, 65536 x 16x16 120 / 36, 4096 x 24x24 16.6 / 13.2, 16384 x 32x32 70 / 49 (its bytes take 39 at the copy
// rate).  Four wavefronts on a SIMD are asked for: with three, 4096 x 27x27 took 19.8 instead of 15.6.
template <int TS>
struct Tile;
template <>
struct Tile<32> {
    using acc = floatx16;
    static constexpr int regs = 16;
    static __device__ __forceinline__ int row(int v, int lane) { return acc_row(v, lane); }
    static __device__ __forceinline__ acc mfma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <>
struct Tile<16> {
    using acc = floatx4;
    static constexpr int regs = 4;
    static __device__ __forceinline__ int row(int v, int lane) { return 4 * (lane >> 4) + v; }
    static __device__ __forceinline__ acc mfma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};
// sixteen matrices of 4 x 4: lanes 4 m .. 4 m + 3 hold the columns of matrix m
template <>
struct Tile<4> {
    using acc = floatx4;
    static constexpr int regs = 4;
    static __device__ __forceinline__ int row(int v, int) { return v; }
    static __device__ __forceinline__ acc mfma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0); }
};

// One wavefront's matrices.  PB = 8 (TS = 16): two matrices of n <= 8 as the diagonal blocks of one tile.  N < TS: registers
// that only hold rows from N on stay out (R of them are in use).
template <int TS, int PB, int N = TS>
struct Lanes {
    using T = Tile<TS>;
    static constexpr int R = TS == 32 ? (N + 7) / 8 * 4 : T::regs;
    static constexpr int kMatrices = TS == 4 ? 16 : PB ? TS / PB : 1;
    static constexpr int kPositions = TS == 4 ? 64 : TS;       // columns of all tiles
    static constexpr int kStride = TS + 4;                      // of a row in LDS (128-bit reads of rows)
    int lane, lo, first, count, n;
    __device__ __forceinline__ Lanes(int batch, int n_)
        : lane(threadIdx.x), lo(threadIdx.x % TS), first(blockIdx.x * kMatrices), count(min(kMatrices, batch - first)), n(n_) {}
    __device__ __forceinline__ int matrix_of(int position) const { return PB ? position / (PB ? PB : 1) : 0; }
    __device__ __forceinline__ int index_of(int position) const { return PB ? position % (PB ? PB : 1) : position; }
    __device__ __forceinline__ int matrix() const { return TS == 4 ? lane / 4 : matrix_of(lo); }
    // is register v an entry of a diagonal block?  What a product leaves in the others is zero unless a value is not finite (0 x NaN);
    // as an operand it would take that to the other matrix of the tile.
    __device__ __forceinline__ bool in_block(int v) const { return PB == 0 || matrix_of(T::row(v, lane)) == matrix_of(lo); }
    // is register v an entry of a matrix?
    __device__ __forceinline__ bool inside(int v) const {
        const int r = T::row(v, lane);
        return (TS == 4 || matrix_of(r) == matrix_of(lo)) && matrix() < count && index_of(r) < n && index_of(lo) < n;
    }
    // every register of every lane is one (the same in all lanes)
    __device__ __forceinline__ bool full() const { return PB == 0 && N == TS && n == TS && count == kMatrices; }
    // its place in bytes, counted from this wavefront's first matrix (at most 64 KB on)
    __device__ __forceinline__ unsigned offset(int v) const {
        return 4u * (unsigned)(matrix() * n * n + index_of(T::row(v, lane)) * n + index_of(lo));
    }
    // this lane's entries of a matrix in memory, zero outside; all loads go out before the first is used
    __device__ __forceinline__ void load(float (&x)[R], const float* __restrict__ M) const {
        const char* const base = reinterpret_cast<const char*>(M + (size_t)first * n * n);
        if (full()) {
#pragma unroll
            for (int v = 0; v < R; ++v) x[v] = *reinterpret_cast<const float*>(base + 4u * (unsigned)(matrix() * TS * TS + T::row(v, lane) * TS + lo));
        } else {
            const unsigned last = 4u * (unsigned)(count * n * n - 1);
#pragma unroll
            for (int v = 0; v < R; ++v) x[v] = *reinterpret_cast<const float*>(base + min(offset(v), last));
#pragma unroll
            for (int v = 0; v < R; ++v) x[v] = inside(v) ? x[v] : 0.f;
        }
    }
    __device__ __forceinline__ void store(float* __restrict__ M, const typename T::acc& x) const {
        char* const base = reinterpret_cast<char*>(M + (size_t)first * n * n);
        if (full()) {
#pragma unroll
            for (int v = 0; v < R; ++v) *reinterpret_cast<float*>(base + 4u * (unsigned)(matrix() * TS * TS + T::row(v, lane) * TS + lo)) = x[v];
        } else {
#pragma unroll
            for (int v = 0; v < R; ++v)
                if (inside(v)) *reinterpret_cast<float*>(base + offset(v)) = x[v];
        }
    }
    // x[v] = X[row(v)][lo] -> y[v] = X[lo][row(v)]
    __device__ __forceinline__ void transpose(float (&y)[R], const float (&x)[R], float* const S) const {
        float* const own = S + (TS == 4 ? (lane / 4) * 20 : 0);
        constexpr int LD = TS == 4 ? 4 : kStride;
        wave_sync();
#pragma unroll
        for (int v = 0; v < R; ++v) own[T::row(v, lane) * LD + lo] = x[v];
        wave_sync();
#pragma unroll
        for (int q = 0; q < R; q += 4) {
            const floatx4 t = *reinterpret_cast<const floatx4*>(own + lo * LD + T::row(q, lane));
#pragma unroll
            for (int k = 0; k < 4; ++k) y[q + k] = t[k];
        }
    }
    static constexpr int kBuffer = TS == 4 ? 16 * 20 : TS * kStride;
    // entries of a vector in LDS (one per position) at the rows of this lane's registers
    __device__ __forceinline__ void rows_of(float (&y)[R], const float* const S) const {
        const float* const own = S + (TS == 4 ? 4 * (lane / 4) : 0);
#pragma unroll
        for (int q = 0; q < R; q += 4) {
            const floatx4 t = *reinterpret_cast<const floatx4*>(own + T::row(q, lane));
#pragma unroll
            for (int k = 0; k < 4; ++k) y[q + k] = t[k];
        }
    }
    // position of a vector entry (lane < kPositions) -> its place in memory, or not one
    __device__ __forceinline__ bool vector_inside() const {
        return lane < kPositions && (TS == 4 ? lane / 4 : matrix_of(lane)) < count && index_of(TS == 4 ? lane % 4 : lane) < n;
    }
    __device__ __forceinline__ size_t vector_offset() const {
        return (size_t)(first + (TS == 4 ? lane / 4 : matrix_of(lane))) * n + index_of(TS == 4 ? lane % 4 : lane);
    }
    __device__ __forceinline__ int own_position() const { return TS == 4 ? lane : lo; }
};

template <int TS, int PB, int N = TS>
__global__ __launch_bounds__(64, 4) void tile_grad_kernel(GradArgs args) {
    using L = Lanes<TS, PB, N>;
    using T = Tile<TS>;
    constexpr int R = L::R;
    __shared__ __align__(16) float buffer[L::kBuffer];
    __shared__ __align__(16) float sL[L::kPositions];     // eigenvalues
    __shared__ __align__(16) float sR[L::kPositions];     // their reciprocals; for a spectral function sqrt(max(lambda, floor))
    __shared__ __align__(16) float sGl[L::kPositions];    // upstream gradient of the eigenvalues
    const L own(args.batch, args.n);
    const bool ed = (args.mode == kGradExact || args.mode == kGradTaylor);

    float vc[R], gc[R];
    own.load(vc, args.evecs);
    if (args.g_mat) own.load(gc, args.g_mat);             // the same in all lanes
    bool low = false;                                      // an eigenvalue below the floor
    if (own.lane < L::kPositions) {
        const bool ok = own.vector_inside();
        const float l = ok ? args.evals[own.vector_offset()] : 0.f;
        sL[own.lane] = l;
        sR[own.lane] = ed ? (l != 0.f ? 1.0f / l : 0.f) : sqrtf(fmaxf(l, args.param));
        sGl[own.lane] = (ok && args.g_evals) ? args.g_evals[own.vector_offset()] : 0.f;
        low = ok && !(l >= args.param);
    }
    low = __ballot(low) != 0;

    typename T::acc c{};
    if (ed) {
        if (args.g_mat) {
#pragma unroll
            for (int v = 0; v < R; ++v) c = T::mfma(vc[v], gc[v], c);
#pragma unroll
            for (int v = 0; v < R; ++v) c = T::mfma(-gc[v], vc[v], c);
        }
    } else {
        float gr[R];
        own.transpose(gr, gc, buffer);
        typename T::acc t{};
#pragma unroll
        for (int v = 0; v < R; ++v) t = T::mfma(0.5f * (gc[v] + gr[v]), vc[v], t);
#pragma unroll
        for (int v = 0; v < R; ++v) c = T::mfma(vc[v], own.in_block(v) ? t[v] : 0.f, c);
    }
    float vr[R];
    own.transpose(vr, vc, buffer);                         // and makes sL, sR, sGl visible
    float li[R], ri[R];
    own.rows_of(li, sL);
    own.rows_of(ri, sR);
    const int jp = own.own_position();
    const float lj = sL[jp], rj = sR[jp];
    float m[R];
    if (ed) {
        couplings(m, li, lj, ri, rj, [&](int v) { return own.lo > T::row(v, own.lane); }, args.mode, args.degree, args.param);
#pragma unroll
        for (int v = 0; v < R; ++v) m[v] = T::row(v, own.lane) == own.lo ? sGl[jp] : 0.5f * m[v] * c[v];
    } else if (low) {
#pragma unroll
        for (int v = 0; v < R; ++v) m[v] = divided_difference(li[v], lj, args.mode, args.param) * c[v];
    } else {
        // every eigenvalue at or above the floor: the form without cancellation, from the roots
#pragma unroll
        for (int v = 0; v < R; ++v)
            m[v] = ((args.mode == kGradSqrt) ? reciprocal(ri[v] + rj) : -reciprocal(ri[v] * rj * (ri[v] + rj))) * c[v];
    }
#pragma unroll
    for (int v = 0; v < R; ++v) m[v] = own.inside(v) ? m[v] : 0.f;
    typename T::acc w{}, g{};
#pragma unroll
    for (int v = 0; v < R; ++v) w = T::mfma(m[v], vr[v], w);
#pragma unroll
    for (int v = 0; v < R; ++v) g = T::mfma(vr[v], own.in_block(v) ? w[v] : 0.f, g);
    own.store(args.g_A, g);
}

// F = V f(max(Lambda, floor)) V^T from a decomposition in memory, 4 < n <= 32, the same way (up to 4 rows the decomposition forms it).
template <int TS, int PB>
__global__ __launch_bounds__(64) void tile_spectral_kernel(KernelArgs args) {
    using L = Lanes<TS, PB>;
    using T = Tile<TS>;
    constexpr int R = T::regs;
    __shared__ __align__(16) float buffer[L::kBuffer];
    __shared__ __align__(16) float sf[L::kPositions];
    const L own(args.batch, args.n);
    float vc[R], vr[R], f[R];
    own.load(vc, args.evecs);
    if (own.lane < L::kPositions) {
        const bool ok = own.vector_inside();
        const float x = fmaxf(ok ? args.evals[own.vector_offset()] : 0.f, args.fn_floor);
        sf[own.lane] = ok ? ((args.fn == kFnInvSqrt) ? __builtin_amdgcn_rsqf(x) : __builtin_amdgcn_sqrtf(x)) : 0.f;
    }
    own.transpose(vr, vc, buffer);
    own.rows_of(f, sf);
    typename T::acc F{};
#pragma unroll
    for (int v = 0; v < R; ++v) F = T::mfma(own.in_block(v) ? vr[v] * f[v] : 0.f, vr[v], F);
    own.store(args.fn_out, F);
}

// ---- n > 32 ----
// One workgroup per matrix, NT = ceil(n / 16) wavefronts: wavefront w owns columns 16 w .. 16 w + 15 of every product, in tiles of
// v_mfma_f32_16x16x4.  Register v of lane l of tile t is the entry of row 16 t + 4 (l / 16) + v and column 16 w + l % 16, and as it stands
// a right operand, so that a product's result is the next one's right operand without leaving the registers; the left operands
// are rows in LDS, four contracted indices to a 128-bit read, which serves four matrix instructions.  With sym(G) formed before the
// products, C = V^T (sym(G) V) is symmetric and nothing is exchanged before the last product, g_A = (V M) V^T: there the
// wavefronts need each other's columns of V M.  It is symmetric too: a tile of it is formed once and stored twice.
// Bound by the matrix cores for many large matrices (n = 128: 3.5 n^3 multiply-adds, 24 us a matrix and compute unit, after the
// 10 us in which its bytes arrive), else by the chain of loads, products and barriers.
// us per launch with 32 x 32 tiles, every product through LDS and up to 64 or 128 rows in one instantiation / this, the function's gradient
// and the decomposition's: 256 x 36x36 9.4 / 7.2 and 8.6 / 7.7, 2048 x 48x48 43 / 27 and 37 / 26, 256 x 64x64 12.3 / 9.6 and 11.0 / 8.7,
// 256 x 80x80 33.9 / 18.0 and 30.3 / 17.1, 8 x 100x100 37.7 / 29 and 34.6 / 27, 256 x 128x128 51 / 39.5 and 43 / 34.
template <int NT>
struct Strip {
    static constexpr int NP = 16 * NT;
    static constexpr int LD = NP + 4;     // rows start on 128 bits; 16 rows at the same four columns lie in 64 different banks
    int w, i, g, n;
    __device__ __forceinline__ explicit Strip(int n_)
        : w(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), i(threadIdx.x & 15), g((threadIdx.x >> 4) & 3), n(n_) {}
    __device__ __forceinline__ int row(int t, int v) const { return 16 * t + 4 * g + v; }
    __device__ __forceinline__ int col() const { return 16 * w + i; }
    __device__ __forceinline__ bool inside(int t, int v) const { return row(t, v) < n && col() < n; }
    // does n cut into tile t (the same in all lanes)?  Into the last of a row or column only.
    __device__ __forceinline__ bool edge(int t) const { return (t == NT - 1 || w == NT - 1) && n < NP; }
    // this lane's entries of a matrix in memory, zero outside
    __device__ __forceinline__ void load(floatx4 (&x)[NT], const float* __restrict__ M) const {
        const int at = 4 * g * n + col();
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[t][v] = M[min(at + (16 * t + v) * n, n * n - 1)];
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (edge(t))
#pragma unroll
                for (int v = 0; v < 4; ++v) x[t][v] = inside(t, v) ? x[t][v] : 0.f;
    }
    // S[r][c] = X[r][c], and S[c][r] = X[r][c]
    __device__ __forceinline__ void put(float* S, const floatx4 (&x)[NT]) const {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[row(t, v) * LD + col()] = x[t][v];
    }
    __device__ __forceinline__ void put_transposed(float* S, const floatx4 (&x)[NT]) const {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<floatx4*>(S + col() * LD + row(t, 0)) = x[t];
    }
    // S[16 r + i][the rows of tile t]: the left operand of its four steps
    __device__ __forceinline__ floatx4 left(const float* S, int r, int t) const {
        return *reinterpret_cast<const floatx4*>(S + (16 * r + i) * LD + row(t, 0));
    }
    static __device__ __forceinline__ floatx4 mfma(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    // out += S x
    __device__ __forceinline__ void product(floatx4 (&out)[NT], const float* S, const floatx4 (&x)[NT]) const {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            floatx4 a[NT];
#pragma unroll
            for (int r = 0; r < NT; ++r) a[r] = left(S, r, t);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int r = 0; r < NT; ++r) out[r] = mfma(a[r][v], x[t][v], out[r]);
        }
    }
    // M = S x, which is symmetric: tile rows w, w + 1, ... (cyclic), every pair of strips once, and their mirror images (which turn in
    // `turn`, rows 16 w .. 16 w + 15 of it, where they cannot be stored four columns at a time)
    __device__ __forceinline__ void store_symmetric(float* __restrict__ M, const float* S, const floatx4 (&x)[NT], float* turn) const {
        // rows start on 128 bits
        const bool aligned = n % 4 == 0 && (reinterpret_cast<uintptr_t>(M) & 15) == 0;
        constexpr int ND = NT / 2 + 1;
        const bool opposite = NT % 2 || w < NT / 2;                // of a pair half way round, the first
        floatx4 out[ND] = {};
        int rows[ND];
#pragma unroll
        for (int d = 0; d < ND; ++d) rows[d] = w + d < NT ? w + d : w + d - NT;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            floatx4 a[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) a[d] = left(S, rows[d], t);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int d = 0; d < ND; ++d)
                    if (d < ND - 1 || opposite) out[d] = mfma(a[d][v], x[t][v], out[d]);
        }
        auto formed = [&](int d) { return d < ND - 1 || opposite; };
        const int c = col();
        if (!aligned) {
#pragma unroll
            for (int d = 1; d < ND; ++d)
                if (formed(d)) *reinterpret_cast<floatx4*>(turn + c * LD + row(rows[d], 0)) = out[d];
            wave_sync();
        }
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            if (!formed(d)) continue;
            const int r = row(rows[d], 0), at = 4 * g * n + c + 16 * rows[d] * n;       // r n + c
            if (!edge(rows[d])) {
#pragma unroll
                for (int v = 0; v < 4; ++v) M[at + v * n] = out[d][v];
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (r + v < n && c < n) M[at + v * n] = out[d][v];
            }
            // four columns at a time are inside or not
            if (d > 0 && aligned && r < n && c < n) *reinterpret_cast<floatx4*>(M + c * n + r) = out[d];
        }
        if (!aligned) {
#pragma unroll
            for (int d = 1; d < ND; ++d) {
                if (!formed(d)) continue;
                const int mirrored = (16 * w + 4 * g) * n + 16 * rows[d] + i;
                float m[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) m[v] = turn[row(w, v) * LD + 16 * rows[d] + i];
                if (!edge(rows[d])) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) M[mirrored + v * n] = m[v];
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (row(w, v) < n && 16 * rows[d] + i < n) M[mirrored + v * n] = m[v];
                }
            }
        }
    }
};

// Wavefronts asked for on a SIMD: as many as LDS has room for up to 64 rows (with three, 2048 x 64x64 took 48.6 instead of 43.2 us).
template <int NT>
__global__ __launch_bounds__(64 * NT, NT == 3 ? 5 : NT == 4 ? 4 : 2) void grad_kernel(GradArgs args) {
    using S = Strip<NT>;
    constexpr int NP = S::NP;
    __shared__ __align__(16) float sA[NP * S::LD];   // V^T, then V
    __shared__ __align__(16) float sB[NP * S::LD];   // C^T; for a spectral function G^T and sym(G); then V M
    __shared__ __align__(16) float sL[NP];           // eigenvalues
    __shared__ __align__(16) float sR[NP];           // their reciprocals; for a spectral function sqrt(max(lambda, floor))
    __shared__ float sGl[NP];                        // upstream gradient of the eigenvalues

    const int tid = threadIdx.x, n = args.n;
    const S own(n);
    const size_t base = (size_t)blockIdx.x * n * n;
    const bool ed = (args.mode == kGradExact || args.mode == kGradTaylor);

    floatx4 vc[NT], gc[NT] = {}, c[NT] = {};
    own.load(vc, args.evecs + base);
    if (args.g_mat) own.load(gc, args.g_mat + base);  // the same in all lanes
    bool low = false;                                 // an eigenvalue below the floor
    if (tid < NP) {
        const bool ok = tid < n;
        const size_t at = (size_t)blockIdx.x * n + tid;
        const float l = ok ? args.evals[at] : 0.f;
        sL[tid] = l;
        sR[tid] = ed ? (l != 0.f ? 1.0f / l : 0.f) : sqrtf(fmaxf(l, args.param));
        sGl[tid] = (ok && args.g_evals) ? args.g_evals[at] : 0.f;
        low = ok && !(l >= args.param);
    }
    own.put_transposed(sA, vc);
    if (!ed) own.put_transposed(sB, gc);
    low = __syncthreads_or(low);
    if (ed) {
        if (args.g_mat) {
            // C - C^T
            own.product(c, sA, gc);
            own.put_transposed(sB, c);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) c[t][v] -= sB[own.row(t, v) * S::LD + own.col()];
        }
    } else {
        floatx4 T[NT] = {};
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) gc[t][v] = 0.5f * (gc[t][v] + sB[own.row(t, v) * S::LD + own.col()]);
        __syncthreads();
        own.put_transposed(sB, gc);
        __syncthreads();
        own.product(T, sB, vc);
        own.product(c, sA, T);
    }
    {
        const int j = own.col();
        const float lj = sL[j], rj = sR[j];
        // two to four tiles side by side: their chains of dependent instructions overlap
        constexpr int V = NT % 4 == 0 ? 16 : NT % 3 == 0 ? 12 : 4 * ((NT + 1) / 2);
#pragma unroll
        for (int t0 = 0; t0 < NT; t0 += V / 4) {
            float li[V], ri[V], m[V];
#pragma unroll
            for (int k = 0; k < V; k += 4) {
                const floatx4 l4 = *reinterpret_cast<const floatx4*>(sL + own.row(min(t0 + k / 4, NT - 1), 0));
                const floatx4 r4 = *reinterpret_cast<const floatx4*>(sR + own.row(min(t0 + k / 4, NT - 1), 0));
#pragma unroll
                for (int v = 0; v < 4; ++v) li[k + v] = l4[v], ri[k + v] = r4[v];
            }
            auto row = [&](int k) { return own.row(t0 + k / 4, k % 4); };
            if (ed) couplings(m, li, lj, ri, rj, [&](int k) { return j > row(k); }, args.mode, args.degree, args.param);
#pragma unroll
            for (int k = 0; k < V; ++k) {
                if (t0 + k / 4 >= NT) continue;
                float x = c[t0 + k / 4][k % 4];
                if (ed) {
                    x = row(k) == j ? sGl[j] : 0.5f * m[k] * x;
                } else if (low) {
                    x *= divided_difference(li[k], lj, args.mode, args.param);
                } else {
                    // every eigenvalue at or above the floor: the form without cancellation, from the roots
                    x *= (args.mode == kGradSqrt) ? reciprocal(ri[k] + rj) : -reciprocal(ri[k] * rj * (ri[k] + rj));
                }
                c[t0 + k / 4][k % 4] = x;
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (own.edge(t))
#pragma unroll
                for (int v = 0; v < 4; ++v) c[t][v] = own.inside(t, v) ? c[t][v] : 0.f;
    }
    __syncthreads();
    own.put(sA, vc);
    __syncthreads();
    {
        floatx4 u[NT] = {};
        own.product(u, sA, c);
        own.put(sB, u);
    }
    floatx4 vr[NT];                                   // V^T, this wavefront's columns
#pragma unroll
    for (int t = 0; t < NT; ++t) vr[t] = own.left(sA, own.w, t);
    __syncthreads();
    own.store_symmetric(args.g_A + base, sB, vr, sA);
}

// The same for 32 < n <= 64 (larger n forms F in the kernel that decomposes).
template <int NT>
__global__ __launch_bounds__(64 * NT, 2) void spectral_kernel(KernelArgs args) {
    using S = Strip<NT>;
    __shared__ __align__(16) float sV[S::NP * S::LD], turn[S::NP * S::LD];
    __shared__ float sf[S::NP];
    const int tid = threadIdx.x, n = args.n;
    const S own(n);
    const size_t base = (size_t)blockIdx.x * n * n;
    floatx4 vc[NT], vr[NT];
    own.load(vc, args.evecs + base);
    if (tid < S::NP) {
        const float x = fmaxf(tid < n ? args.evals[(size_t)blockIdx.x * n + tid] : 0.f, args.fn_floor);
        sf[tid] = tid < n ? ((args.fn == kFnInvSqrt) ? __builtin_amdgcn_rsqf(x) : __builtin_amdgcn_sqrtf(x)) : 0.f;
    }
    own.put(sV, vc);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        vr[t] = own.left(sV, own.w, t);
#pragma unroll
        for (int v = 0; v < 4; ++v) vr[t][v] *= sf[own.row(t, v)];
    }
    own.store_symmetric(args.fn_out + base, sV, vr, turn);
}

}  // namespace

hipError_t launch_spectral(const KernelArgs& args, hipStream_t stream) {
    const int n = args.n, B = args.batch;
    if (n <= 8) return enqueue(tile_spectral_kernel<16, 8>, dim3((B + 1) / 2), dim3(64), stream, args);
    if (n <= 16) return enqueue(tile_spectral_kernel<16, 0>, dim3(B), dim3(64), stream, args);
    if (n <= 32) return enqueue(tile_spectral_kernel<32, 0>, dim3(B), dim3(64), stream, args);
    if (n <= 48) return enqueue(spectral_kernel<3>, dim3(B), dim3(192), stream, args);
    if (n <= 64) return enqueue(spectral_kernel<4>, dim3(B), dim3(256), stream, args);
    return hipErrorInvalidValue;
}

hipError_t launch_grad(const GradArgs& args, hipStream_t stream) {
    if (args.batch == 0) return hipSuccess;
    if (args.batch > kMostPerLaunch) return in_parts(args, [&](const GradArgs& part) { return launch_grad(part, stream); });
    const int n = args.n, B = args.batch;
    if (n <= 4) return enqueue(tile_grad_kernel<4, 0>, dim3((B + 15) / 16), dim3(64), stream, args);
    if (n <= 8) return enqueue(tile_grad_kernel<16, 8>, dim3((B + 1) / 2), dim3(64), stream, args);
    if (n <= 16) return enqueue(tile_grad_kernel<16, 0>, dim3(B), dim3(64), stream, args);
    if (n <= 24) return enqueue(tile_grad_kernel<32, 0, 24>, dim3(B), dim3(64), stream, args);
    if (n <= 32) return enqueue(tile_grad_kernel<32, 0>, dim3(B), dim3(64), stream, args);
    switch ((n + 15) / 16) {
        case 3: return enqueue(grad_kernel<3>, dim3(B), dim3(192), stream, args);
        case 4: return enqueue(grad_kernel<4>, dim3(B), dim3(256), stream, args);
        case 5: return enqueue(grad_kernel<5>, dim3(B), dim3(320), stream, args);
        case 6: return enqueue(grad_kernel<6>, dim3(B), dim3(384), stream, args);
        case 7: return enqueue(grad_kernel<7>, dim3(B), dim3(448), stream, args);
        default: return enqueue(grad_kernel<8>, dim3(B), dim3(512), stream, args);
    }
}

}  // namespace bed
