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
// One wavefront owns one matrix (four wavefronts for n > 32, eight for n > 64).
// The three (four) n x n x n products are dense
// contractions and run on v_mfma_f32_32x32x2_f32 (full fp32 operands and
// accumulation); operands are staged in LDS with an odd row stride so that row
// and column (transposed) operand reads are both conflict-free, and every
// product's result is written back to LDS in row-major order to become an
// operand of the next one.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bed_kernel.h"

namespace bed {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// Operand and result layout of v_mfma_f32_32x32x2_f32 (A is 32x2, B is 2x32, D is 32x32):
//   A: lane l holds A[l % 32][l / 32]
//   B: lane l holds B[l / 32][l % 32]
//   D: register v (0..15) of lane l holds D[8 * (v / 4) + 4 * (l / 32) + v % 4][l % 32]
__device__ __forceinline__ int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

// Tiles of one wavefront: all NT x NT of them when it works alone, else one tile row and every JSTEP-th
// tile column.
template <int NT, int NWV>
struct Tiles {
    static_assert(NWV == 1 || NWV % NT == 0, "a wavefront owns tiles of one row");
    static constexpr int TI = NWV == 1 ? NT : 1;
    static constexpr int JSTEP = NWV == 1 ? 1 : NWV / NT;
    static constexpr int TJ = NT / JSTEP;
    static constexpr int LD = 32 * NT + 1;
    int wv;
    __device__ __forceinline__ int row(int ti) const { return NWV == 1 ? ti : wv % NT; }
    __device__ __forceinline__ int col(int tj) const { return NWV == 1 ? tj : wv / NT + tj * JSTEP; }

    // acc = sum_k X[i][k] * Y[k][j] over k < kdim (a multiple of 8; entries from n on are zero).
    // XT / YT: the operand is stored transposed in its LDS buffer.  Four k steps of operands are read
    // before their matrix instructions: one at a time, every instruction waits for LDS.
    template <bool XT, bool YT>
    __device__ __forceinline__ void product(floatx16 (&acc)[TI][TJ], const float* X, const float* Y, int kdim,
                                            int lane) const {
        const int lo = lane & 31, hi = lane >> 5;
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) acc[ti][tj] = floatx16{};
        for (int k0 = 0; k0 < kdim; k0 += 8) {
            float a[TI][4], b[TJ][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 2 * u + hi;
#pragma unroll
                for (int t = 0; t < TI; ++t) {
                    const int r = 32 * row(t) + lo;
                    a[t][u] = XT ? X[k * LD + r] : X[r * LD + k];
                }
#pragma unroll
                for (int t = 0; t < TJ; ++t) {
                    const int r = 32 * col(t) + lo;
                    b[t][u] = YT ? Y[r * LD + k] : Y[k * LD + r];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                    for (int tj = 0; tj < TJ; ++tj)
                        acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ti][u], b[tj][u], acc[ti][tj], 0, 0, 0);
        }
    }

    __device__ __forceinline__ void spill(const floatx16 (&acc)[TI][TJ], float* dst, int lane) const {
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    dst[(32 * row(ti) + acc_row(v, lane)) * LD + 32 * col(tj) + (lane & 31)] = acc[ti][tj][v];
    }
};

// 1 / x: the hardware reciprocal (one unit in the last place) and one Newton step; the division itself
// where one of the two would leave the normal range
__device__ __forceinline__ float reciprocal(float x) {
    if (!(fabsf(x) > 1e-37f && fabsf(x) < 1e37f)) return 1.0f / x;
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, r, 1.f), r, r);
}

// Coupling of the pair (a, b) = (lambda_i, lambda_j), i != j; ra, rb their reciprocals.
__device__ __forceinline__ float coupling(float a, float b, float ra, float rb, bool j_later, int mode, int degree,
                                          float gap_floor) {
    if (mode == kGradExact) {
        const float d = b - a;
        return (fabsf(d) >= gap_floor && d != 0.f) ? 1.0f / d : 0.f;
    }
    // truncated series: with b the larger in magnitude, 1/(b - a) ~ (1/b) sum_{k<=degree} (a/b)^k;
    // mirrored otherwise.  Equal magnitudes: the later index counts as the larger, which keeps
    // K antisymmetric.
    const bool big_b = fabsf(b) > fabsf(a) || (fabsf(b) == fabsf(a) && j_later);
    const float num = big_b ? a : b, den = big_b ? b : a;
    if (den == 0.f) return 0.f;
    const float rden = big_b ? rb : ra;
    const float rho = num * rden;
    float s = 1.f;
    for (int k = 0; k < degree; ++k) s = fmaf(s, rho, 1.f);
    const float kk = s * rden;
    return big_b ? kk : -kk;
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

// NT tiles of 32 per side (1: n <= 32, 2: n <= 64, 4: n <= 128); NWV wavefronts per matrix.
// PB > 0 (n <= PB <= 16, NT = NWV = 1): 32 / PB matrices share the wavefront as the diagonal
// blocks of one 32 x 32 operand; products of block-diagonal matrices are block diagonal, so
// the same instruction stream serves all of them.
// The floor of a large batch is the matrix cores' fp32 rate (n = 128: 16 tiles x 64 steps x 64 cycles x 4
// products on four of them = 27 us a matrix and compute unit); a small one is bound by the
// serial path of loads, four products and the exchange between them, which is why operands are read four steps
// ahead, the inputs eight loads at a time, and a matrix of n > 32 gets four or eight wavefronts.
template <int NT, int NWV, int PB>
__global__ __launch_bounds__(64 * NWV) void grad_kernel(GradArgs args) {
    static_assert(PB == 0 || (NT == 1 && NWV == 1 && 32 % PB == 0), "packing needs one 32 x 32 tile");
    using Own = Tiles<NT, NWV>;
    constexpr int NMAT = PB ? 32 / PB : 1;       // matrices per workgroup
    constexpr int NP = 32 * NT;
    constexpr int LD = NP + 1;
    constexpr int TI = Own::TI, TJ = Own::TJ;
    constexpr int NTH = 64 * NWV;
    __shared__ __align__(16) float sV[NP * LD];      // V, row-major, zero padded
    __shared__ __align__(16) float sW[NP * LD];      // G, then the intermediate products
    __shared__ float sL[NP];           // eigenvalues
    __shared__ float sR[NP];           // their reciprocals; for a spectral function sqrt(max(lambda, floor))
    __shared__ float sGl[NP];          // upstream gradient of the eigenvalues

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const Own own{tid >> 6};
    const int b = blockIdx.x * NMAT;           // first matrix of this workgroup
    const int count = min(NMAT, args.batch - b);
    const int n = args.n;
    const int kdim = PB ? 32 : ((n + 7) & ~7);
    const bool ed = (args.mode == kGradExact || args.mode == kGradTaylor);
    // position p of the (padded) operand -> matrix p / PB, local index p % PB
    auto blk = [](int p) { return PB ? p / (PB ? PB : 1) : 0; };
    auto loc = [](int p) { return PB ? p % (PB ? PB : 1) : p; };
    // LDS written by one wavefront and read by another needs a workgroup barrier
    auto sync = [&]() {
        if (NWV == 1) wave_sync();
        else __syncthreads();
    };

    {
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int idx = tid; idx < NP * LD / 4; idx += NTH) {
            reinterpret_cast<float4*>(sV)[idx] = zero;
            reinterpret_cast<float4*>(sW)[idx] = zero;
        }
    }
    bool low = false;                  // an eigenvalue below the floor
    if (tid < NP) {
        const bool ok = blk(tid) < count && loc(tid) < n;
        const size_t at = (size_t)(b + blk(tid)) * n + loc(tid);
        const float l = ok ? args.evals[at] : 0.f;
        sL[tid] = l;
        sR[tid] = ed ? (l != 0.f ? 1.0f / l : 0.f) : sqrtf(fmaxf(l, args.param));
        sGl[tid] = (ok && args.g_evals) ? args.g_evals[at] : 0.f;
        low = ok && !(l >= args.param);
    }
    sync();
    {
        // the workgroup's matrices are contiguous in memory: one coalesced pass over all of them
        const float* __restrict__ Vb = args.evecs + (size_t)b * n * n;
        const float* __restrict__ Gb = args.g_mat ? args.g_mat + (size_t)b * n * n : nullptr;
        const float rcp_n = 1.0f / (float)n;
        const float rcp_nn = rcp_n * rcp_n;
        const int total = count * n * n;
        for (int base = tid; base < total; base += 8 * NTH) {
            float v[8], g[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int idx = base + k * NTH;
                v[k] = idx < total ? Vb[idx] : 0.f;
                g[k] = (Gb && idx < total) ? Gb[idx] : 0.f;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int idx = base + k * NTH;
                const int m = PB ? (int)(((float)idx + 0.5f) * rcp_nn) : 0;
                const int r = idx - m * n * n;
                const int i = (int)(((float)r + 0.5f) * rcp_n);
                const int at = (m * PB + i) * LD + m * PB + r - i * n;
                if (idx < total) {
                    sV[at] = v[k];
                    sW[at] = g[k];
                }
            }
        }
    }
    if (NWV == 1) {
        low = __ballot(low) != 0;
        sync();
    } else {
        low = __syncthreads_or(low);
    }

    floatx16 acc[TI][TJ];
    if (!ed) {
        // spectral function: T = G V first, so that C = V^T G V
        own.template product<false, false>(acc, sW, sV, kdim, lane);
        sync();
        own.spill(acc, sW, lane);
        sync();
    }
    // C = V^T T  (T = g_V for the eigendecomposition itself)
    own.template product<true, false>(acc, sV, sW, kdim, lane);
    sync();
    own.spill(acc, sW, lane);
    sync();
    // M: element (i, j) needs C_ij (own register), C_ji, lambda_i, lambda_j
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) {
            const int j = 32 * own.col(tj) + (lane & 31);
            const float lj = sL[j], rj = sR[j];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = 32 * own.row(ti) + acc_row(v, lane);
                const float cij = acc[ti][tj][v];
                const float cji = sW[j * LD + i];
                const float li = sL[i], ri = sR[i];
                float m;
                if (ed) {
                    m = (i == j) ? sGl[i]
                                 : 0.5f * coupling(li, lj, ri, rj, j > i, args.mode, args.degree, args.param) * (cij - cji);
                } else if (low) {
                    m = 0.5f * divided_difference(li, lj, args.mode, args.param) * (cij + cji);
                } else {
                    // every eigenvalue at or above the floor: the form without cancellation, from the roots
                    const float phi = (args.mode == kGradSqrt) ? reciprocal(ri + rj) : -reciprocal(ri * rj * (ri + rj));
                    m = 0.5f * phi * (cij + cji);
                }
                const bool inside = blk(i) == blk(j) && blk(i) < count && loc(i) < n && loc(j) < n;
                acc[ti][tj][v] = inside ? m : 0.f;
            }
        }
    sync();
    own.spill(acc, sW, lane);
    sync();
    // U = V M
    own.template product<false, false>(acc, sV, sW, kdim, lane);
    sync();
    own.spill(acc, sW, lane);
    sync();
    // g_A = U V^T
    own.template product<false, true>(acc, sW, sV, kdim, lane);
    float* __restrict__ Ob = args.g_A + (size_t)b * n * n;
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = 32 * own.row(ti) + acc_row(v, lane);
                const int j = 32 * own.col(tj) + (lane & 31);
                const bool inside = blk(i) == blk(j) && blk(i) < count && loc(i) < n && loc(j) < n;
                if (inside) Ob[(size_t)blk(i) * n * n + loc(i) * n + loc(j)] = acc[ti][tj][v];
            }
}

// F = V f(max(Lambda, floor)) V^T from a decomposition in memory, n <= 64 (larger n forms F in the kernel
// that decomposes).  Same tiles and packing as grad_kernel; one product, so the call is bound by its
// launch for small batches and by reading V and writing F for large ones.
template <int NT, int PB>
__global__ __launch_bounds__(64) void spectral_kernel(KernelArgs args) {
    static_assert(PB == 0 || (NT == 1 && 32 % PB == 0), "packing needs one 32 x 32 tile");
    constexpr int NMAT = PB ? 32 / PB : 1;
    constexpr int NP = 32 * NT, LD = NP + 1;
    __shared__ float sV[NP * LD];
    __shared__ float sW[NP * LD];      // V f
    __shared__ float sf[NP];
    const int lane = threadIdx.x;
    const int b = blockIdx.x * NMAT;
    const int count = min(NMAT, args.batch - b);
    const int n = args.n;
    auto blk = [](int p) { return PB ? p / (PB ? PB : 1) : 0; };
    auto loc = [](int p) { return PB ? p % (PB ? PB : 1) : p; };
    for (int idx = lane; idx < NP * LD; idx += 64) {
        sV[idx] = 0.f;
        sW[idx] = 0.f;
    }
    if (lane < NP) {
        float f = 0.f;
        if (blk(lane) < count && loc(lane) < n) {
            const float x = fmaxf(args.evals[(size_t)(b + blk(lane)) * n + loc(lane)], args.fn_floor);
            f = (args.fn == kFnInvSqrt) ? __builtin_amdgcn_rsqf(x) : __builtin_amdgcn_sqrtf(x);
        }
        sf[lane] = f;
    }
    wave_sync();
    const float* __restrict__ Vb = args.evecs + (size_t)b * n * n;
    const float rcp_n = 1.0f / (float)n;
    const float rcp_nn = rcp_n * rcp_n;
    chunked_copy<8>(
        count * n * n, lane, [&](int idx) { return Vb[idx]; },
        [&](int idx, float x) {
            const int m = PB ? (int)(((float)idx + 0.5f) * rcp_nn) : 0;
            const int r = idx - m * n * n;
            const int i = (int)(((float)r + 0.5f) * rcp_n);
            const int j = m * PB + r - i * n;
            sV[(m * PB + i) * LD + j] = x;
            sW[(m * PB + i) * LD + j] = x * sf[j];
        });
    wave_sync();
    floatx16 acc[NT][NT];
    Tiles<NT, 1>{0}.template product<false, true>(acc, sW, sV, PB ? 32 : ((n + 7) & ~7), lane);
    float* __restrict__ Fb = args.fn_out + (size_t)b * n * n;
#pragma unroll
    for (int ti = 0; ti < NT; ++ti)
#pragma unroll
        for (int tj = 0; tj < NT; ++tj)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = 32 * ti + acc_row(v, lane);
                const int j = 32 * tj + (lane & 31);
                const bool inside = blk(i) == blk(j) && blk(i) < count && loc(i) < n && loc(j) < n;
                if (inside) Fb[(size_t)blk(i) * n * n + loc(i) * n + loc(j)] = acc[ti][tj][v];
            }
}

}  // namespace

hipError_t launch_spectral(const KernelArgs& args, hipStream_t stream) {
    const int n = args.n, B = args.batch;
    if (n <= 4) return enqueue(spectral_kernel<1, 4>, dim3((B + 7) / 8), dim3(64), stream, args);
    if (n <= 8) return enqueue(spectral_kernel<1, 8>, dim3((B + 3) / 4), dim3(64), stream, args);
    if (n <= 16) return enqueue(spectral_kernel<1, 16>, dim3((B + 1) / 2), dim3(64), stream, args);
    if (n <= 32) return enqueue(spectral_kernel<1, 0>, dim3(B), dim3(64), stream, args);
    if (n <= 64) return enqueue(spectral_kernel<2, 0>, dim3(B), dim3(64), stream, args);
    return hipErrorInvalidValue;
}

hipError_t launch_grad(const GradArgs& args, hipStream_t stream) {
    if (args.batch == 0) return hipSuccess;
    const int n = args.n, B = args.batch;
    if (n <= 4)
        return enqueue(grad_kernel<1, 1, 4>, dim3((B + 7) / 8), dim3(64), stream, args);
    else if (n <= 8)
        return enqueue(grad_kernel<1, 1, 8>, dim3((B + 3) / 4), dim3(64), stream, args);
    else if (n <= 16)
        return enqueue(grad_kernel<1, 1, 16>, dim3((B + 1) / 2), dim3(64), stream, args);
    else if (n <= 32)
        return enqueue(grad_kernel<1, 1, 0>, dim3(B), dim3(64), stream, args);
    else if (n <= 64)
        return enqueue(grad_kernel<2, 4, 0>, dim3(B), dim3(256), stream, args);
    else
        return enqueue(grad_kernel<4, 8, 0>, dim3(B), dim3(512), stream, args);
}

}  // namespace bed
