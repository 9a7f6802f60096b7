// Divide and conquer for the symmetric tridiagonal eigenproblem, one matrix per workgroup.
//
// T is torn into blocks of at most four rows, which Jacobi's method solves (four lanes each): every coupling e between two blocks is taken out as a
// rank-one term, T = diag(T1', T2') + rho z z^T with |z| = 1 (Cuppen 1981), and the blocks are
// merged pairwise, all merges of a level at once.  A merge of m eigenvalues
//   - deflates components of z that are negligible and pairs of poles that a plane rotation
//     decouples (Dongarra and Sorensen 1987), to rounding of the pole itself and not of the largest
//     one, which keeps small eigenvalues of graded matrices,
//   - finds the roots of the secular equation 1/rho + sum z_j^2 / (d_j - lambda) = 0, one root per
//     thread, from rational interpolation with the two neighbouring poles (Bunch, Nielsen and
//     Sorensen 1978) through two derivatives, inside a bracket and measured from the nearer pole,
//   - recomputes z from the roots so that the eigenvectors are orthogonal to working precision
//     whatever the last bits of the roots are (Gu and Eisenstat 1994),
//   - multiplies the block's eigenvectors with those of the merge on the matrix cores (fp32).
// The rotation-by-rotation QR iteration is one serial chain of about 1.1 n^2 rotations (188 cycles
// per pair); here the serial depth is log2(n) merges whose inner loops run over m poles.
#ifndef BED_DC_HPP
#define BED_DC_HPP
#include "bed_wave_kernel.hpp"
#include "bed_secular.hpp"

namespace bed {

// Matrix instructions in fp32: v_mfma_f32_32x32x2_f32, and v_mfma_f32_16x16x4_f32 for n <= 16.
// With S the tile size, lane l holds the operands A[l % S][l / S] and B[l / S][l % S]; register v
// of the result is D[dc_row<S>(v, l)][l % S].
typedef float dc_acc32 __attribute__((ext_vector_type(16)));
typedef float dc_acc16 __attribute__((ext_vector_type(4)));
template <int N>
struct DcTile {
    static constexpr int size = 32;
    using acc = dc_acc32;
};
template <>
struct DcTile<16> {
    static constexpr int size = 16;
    using acc = dc_acc16;
};
template <int TS>
__device__ __forceinline__ int dc_row(int v, int lane) {
    return TS == 16 ? 4 * (lane >> 4) + v : 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
}
__device__ __forceinline__ dc_acc32 dc_mfma(float a, float b, dc_acc32 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ dc_acc16 dc_mfma(float a, float b, dc_acc16 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr float kDcTol = 4.7683716e-7f;         // 8 units of rounding (2^-24)
constexpr float kDcFloor = 9.5367432e-7f;       // poles below 2^-20 of the block's norm deflate by that
constexpr float kDcTiny = 1.5258789e-5f;        // blocks below 2^-16 of the pre-scaled matrix deflate by that
constexpr float kDcFar = 1.0e10f;               // a pole beyond every eigenvalue of a block, in units of its rho (poles stay below 1 / kDcTol)
constexpr int kDcMaxIter = 60;                  // seven times what any root has been seen to take

// N: rows covered (16, 32, 64, 128); TPE: threads per eigenvalue.
// The arrays that the inner loops read are laid out per block with the block size rounded up to
// 4 TPE: trip counts are the same in every lane, each thread takes four poles from 128-bit reads,
// and the entries behind a block's end (and those of deflated poles) hold kDcFar with z = 0.
template <int N, int TPE, bool WANT_V>
struct DcShared {
    static constexpr int LD = N + 1;
    // Every merge of a level takes as many entries as its largest, rounded up to 4 TPE.  The first level is the fullest: the largest of
    // its 2^(L-1) merges has 5 to 8 poles (others 4, n = 17 .. 19, 33 .. 39, 65 .. 79), so 4 TPE entries each.
    static constexpr int NP = N * TPE / 2;
    alignas(16) float Dp[NP];            // by column: eigenvalues
    alignas(16) float2 dz[NP];           // by slot (kept poles ascending, then the deflated ones): d in units of the merge, z^2
    alignas(16) float2 om[NP];           // by slot: the pole the root is measured from, and the distance, in units of the merge
    alignas(16) float2 zs[NP];           // by slot: z, and the offset of its row in U (as an integer)
    alignas(16) float2 fl[NP];           // by slot: entries of the first and last row
    float4 rot[N];                       // deflating rotations: two columns (as integers), cosine, sine
    // V[r * LD + c].  N > 32: the tiles of the merges' products read up to 15 columns and rows behind a block and up to 31 factors
    // behind its columns; what is behind the last row of V and row N of U is zero, what is behind rn only meets results that are dropped
    static constexpr int kTail = N > 32 ? 16 : 0;
    alignas(16) float V[WANT_V ? N * LD + kTail : 1];
    static constexpr int UR = N > 32 ? N + 16 : N + 1;
    alignas(16) float U[WANT_V ? UR * LD : 1];       // eigenvectors of the current merges, same layout; row N takes what is not wanted
    alignas(16) float D[N];              // by column: eigenvalues (the result); +inf from n on
    float first[N], last[N];             // by column: first and last row of its block's eigenvectors
    float dS[N], zS[N];                  // sorted by d
    float dd[N];                         // by slot: d, also of deflated poles
    float rho[N], za[N], zb[N];          // per coupling: weight of the rank-one term, its two sides in z
    float rn[N + 2 * kTail];             // reciprocal norm of a column of U
    int perm[N];                         // sorted position -> column
    int nrot[N];                         // rotations of the block that starts here
    int unresolved;                      // T > 64: sum of the wavefronts' counts
};

template <int TPE>
__device__ __forceinline__ float dc_sum(float x) {
    if (TPE >= 2) x += dpp0<kQuadXor1>(x);
    if (TPE >= 4) x += dpp0<kQuadXor2>(x);
    return x;
}
template <int TPE>
__device__ __forceinline__ float dc_product(float x) {
    if (TPE >= 2) x *= dpp0<kQuadXor1>(x);
    if (TPE >= 4) x *= dpp0<kQuadXor2>(x);
    return x;
}

// Sets of up to 128 positions, wave-uniform.
template <int NB>
struct DcMask {
    uint64_t w[NB];
    __device__ __forceinline__ bool has(int p) const { return ((NB > 1 && p >= 64 ? w[NB - 1] : w[0]) >> (p & 63)) & 1; }
    __device__ __forceinline__ int below(int p) const {      // members < p, p in 0..64 NB
        int c = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int q = p - 64 * b;
            const uint64_t m = q >= 64 ? ~0ull : (q <= 0 ? 0ull : ((1ull << q) - 1ull));
            c += __builtin_popcountll(w[b] & m);
        }
        return c;
    }
    __device__ __forceinline__ int next(int p) const {       // smallest member > p, or 64 NB
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int q = p - 64 * b;
            const uint64_t m = q >= 63 ? 0ull : (q < 0 ? ~0ull : ~((2ull << q) - 1ull));
            if (w[b] & m) return 64 * b + __builtin_ctzll(w[b] & m);
        }
        return 64 * NB;
    }
};

// Are two neighbouring kept poles dp <= dq with components zp, zq decoupled by a rotation?  |gap c s| within
// the tolerance of the larger pole, c, s = zp, zq normalised; as a ratio, so that nothing underflows.
__device__ __forceinline__ bool dc_close(float dp, float dq, float zp, float zq, float floor) {
    const float hi = fmaxf(fabsf(zp), fabsf(zq)), lo = fminf(fabsf(zp), fabsf(zq));
    const float q = lo * __builtin_amdgcn_rcpf(hi);
    return (dq - dp) * q <= kDcTol * fmaxf(fmaxf(fabsf(dp), fabsf(dq)), floor) * fmaf(q, q, 1.f);
}

// 1 / sqrt(x) to the last bit or two
__device__ __forceinline__ float dc_rsqrt(float x) {
    const float r = __builtin_amdgcn_rsqf(x);
    return r * fmaf(-0.5f * x * r, r, 1.5f);
}

// Eigenvalues (S.D, by column) and eigenvectors (S.V) of the tridiagonal with entries dget(k), eget(k) (coupling k
// and k+1), k < n, in LDS, visible to all T threads.  The caller has pre-scaled T to a norm of about one.
// With a non-finite entry in T every output is NaN.  Returns the number of roots that the cap stopped.
template <int N, int T, bool WANT_V, typename Dget, typename Eget>
__device__ __forceinline__ int dc_solve(DcShared<N, T / N, WANT_V>& S, const int n, const int tid, Dget&& dget, Eget&& eget) {
    constexpr int TPE = T / N;                      // threads per eigenvalue, neighbours in a wavefront
    constexpr int LD = DcShared<N, TPE, WANT_V>::LD;
    constexpr int CH = 4 * TPE;                     // poles per step of an inner loop
    constexpr int PP = N / TPE;                     // poles of one thread
    constexpr int NB = (N + 63) / 64;
    static_assert(T % N == 0 && (TPE == 2 || TPE == 4), "2 or 4 threads per eigenvalue");
    constexpr int NWV = T / 64;
    const int lane = tid & 63, wv = tid >> 6;
    const int e = tid / TPE, part = tid % TPE;
    const bool valid = e < n;
    auto sync = [&]() {
        if (T == 64) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };

    int L = 0;
    while ((4 << L) < n) ++L;       // 2^L leaves of at most four rows
    // leaf that holds row r: the largest i with floor(i n / 2^L) <= r
    const float rcp_n = 1.f / (float)n;
    int unresolved = 0;
    if (T > 64 && tid == 0) S.unresolved = 0;
    auto leaf_of = [&](int r) { return (int)(((float)(((r + 1) << L) - 1) + 0.5f) * rcp_n); };
    const int leaf = valid ? leaf_of(e) : 0;
    int leafq[NB];
    bool bad = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int q = lane + 64 * b;
        leafq[b] = q < n ? leaf_of(q) : 0;
        if (q < n) bad = bad || !(fabsf(dget(q)) < __builtin_inff()) || (q < n - 1 && !(fabsf(eget(q)) < __builtin_inff()));
    }
    bad = __ballot(bad) != 0;

    // ---- leaves ----
    if (WANT_V) {
        constexpr int QV = (N * LD + DcShared<N, TPE, WANT_V>::kTail) / 4, QU = N > 32 ? DcShared<N, TPE, WANT_V>::UR * LD / 4 : QV;
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < (QU + T - 1) / T; ++i) {
            const int at = tid + i * T;
            if (at < QV) reinterpret_cast<float4*>(S.V)[at] = zero;
            if (at < QU) reinterpret_cast<float4*>(S.U)[at] = zero;
        }
        sync();
    }
    // Couplings.  e is torn out as rho w w^T with w = (a, +-b) on the two rows, which takes |e| tau and
    // |e| / tau off their diagonal entries.  tau = 1 unless the two diagonal entries differ in size:
    // then tau ~ sqrt(d_k / d_k+1), and where |e|^2 <= d_k d_k+1 (positive definite T) each side loses no
    // more than its own size.  With tau = 1 small rows of a graded T would be left with the
    // rounding of a large e: A^(-1/2) of 128x128 covariances with power-law spectra, condition
    // 1e3, was off by 9e-5 instead of 5e-6.  tau is a power of two.
    if (part == 0 && e < n - 1) {
        const float a = fabsf(dget(e)), c = fabsf(dget(e + 1)), ec = eget(e), b = fabsf(ec);
        int ex = 0;
        if (b * b <= a * c && b != 0.f) ex = min(max((__builtin_amdgcn_frexp_expf(a) - __builtin_amdgcn_frexp_expf(c)) >> 1, -30), 30);
        const float tau = ldexpf(1.f, ex), taken = ldexpf(b, -ex);
        const float w = dc_rsqrt(fmaf(tau, tau, 1.f));
        S.dd[e] = b * tau;                              // what the rows e and e + 1 lose where the coupling is torn out
        S.dS[e] = taken;
        S.rho[e] = fmaf(b, tau, taken);
        S.za[e] = tau * w;
        S.zb[e] = ec < 0.f ? -w : w;
    }
    if (part == 0) {
        S.rn[e] = 1.f;
        S.perm[e] = e;
        if (!valid) S.first[e] = S.last[e] = 0.f;
    }
    sync();
    // Four lanes solve a leaf (bed_jacobi.hpp: lane j has column j, register k row j ^ k).  Leaves of two rows took 3 k cycles and the
    // merge that these save 8 to 14 k (16 to 128 rows); these take 5.9 k to 8.7 k.
    if (tid < (4 << L)) {
        const int j = tid & 3, lo = ((tid >> 2) * n) >> L, hi = (((tid >> 2) + 1) * n) >> L, m = hi - lo;
        const bool in = j < m;
        auto coupling = [&](int k) { return k < m - 1 ? eget(min(lo + k, n - 1)) : 0.f; };      // of rows k and k + 1 of the leaf
        float d = in ? dget(lo + j) : 0.f;
        const float before = S.dS[max(lo - 1, 0)], behind = S.dd[hi - 1];
        d -= j == 0 && lo > 0 ? before : 0.f;
        d -= j == m - 1 && hi < n ? behind : 0.f;
        const float e01 = coupling(j & 2), e12 = coupling(1);
        float x[4] = {d, e01, 0.f, j == 1 || j == 2 ? e12 : 0.f}, v[4] = {1.f, 0.f, 0.f, 0.f};
        bool work = !bad;
        for (int it = 0; it < jacobi::kMaxSweeps; ++it) {
            work = jacobi::sweep<true>(x, v, d, work, j);
            if (__ballot(work) == 0) break;
        }
        jacobi::orthonormalise(v);
        if (bad) d = v[0] = __builtin_nanf("");
        auto entry = [&](int r) { const int k = j ^ r; return k == 0 ? v[0] : k == 1 ? v[1] : k == 2 ? v[2] : v[3]; };
        if (in) {
            S.D[lo + j] = d;
            S.first[lo + j] = entry(0);
            S.last[lo + j] = entry(m - 1);
            if (WANT_V) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if ((j ^ k) < m) S.V[(lo + (j ^ k)) * LD + lo + j] = v[k];
            }
        }
    }
    sync();
    float lam = valid ? S.D[e] : __builtin_inff();      // eigenvalue of column e
    if (bad) {
        if (part == 0) S.D[e] = lam;
        sync();
        return 0;
    }

    for (int level = 1; level <= L; ++level) {
        const int sh = L - level;
        auto lo_of = [&](int i) { return (i * n) >> sh; };
        auto mid_of = [&](int i) { return ((2 * i + 1) * n) >> (sh + 1); };
        const int blk = leaf >> level;
        const int lo = valid ? lo_of(blk) : 0, hi = valid ? lo_of(blk + 1) : 0;
        const int mid = valid ? mid_of(blk) : 0;
        const int m = hi - lo, k = e - lo;
        const int M = (n + (1 << sh) - 1) >> sh;               // size of the largest block
        const int Mp = (M + CH - 1) & ~(CH - 1);
        const int base = blk * Mp;                              // first entry of the block in the padded arrays
        if (valid && part == 0) {
            S.Dp[base + e - lo] = lam;
            for (int i = e - lo + m; i < Mp; i += m) S.Dp[base + i] = __builtin_inff();
        }
        sync();

        // ---- z, and the order of the poles ----
        if (valid) {
            const float zr = e < mid ? S.last[e] : S.first[e];
            const float ze = zr * (e < mid ? S.za : S.zb)[mid - 1];
            const float de = lam;
            int cnt = 0;
#pragma unroll
            for (int c = 0; c < PP; c += 4) {
                if (c * TPE < M) {
                    const int j = c * TPE + 4 * part;
                    const float4 q = *reinterpret_cast<const float4*>(S.Dp + base + j);
                    const int ahead = k - j;                        // ties: the earlier column first
                    cnt += (q.x < de || (q.x == de && ahead > 0)) ? 1 : 0;
                    cnt += (q.y < de || (q.y == de && ahead > 1)) ? 1 : 0;
                    cnt += (q.z < de || (q.z == de && ahead > 2)) ? 1 : 0;
                    cnt += (q.w < de || (q.w == de && ahead > 3)) ? 1 : 0;
                }
            }
            const int pos = lo + (int)dc_sum<TPE>((float)cnt);
            if (part == 0) {
                S.dS[pos] = de;
                S.zS[pos] = ze;
                S.perm[pos] = e;
                (e < mid ? S.last : S.first)[e] = 0.f;
            }
        }
        sync();

        // ---- deflation; every wavefront looks at all positions, so the masks need no exchange ----
        DcMask<NB> kept, close;
        float flq[NB], rhoq[NB];        // floor for the size of a pole, weight

#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int q = lane + 64 * b;
            bool k = false;
            flq[b] = rhoq[b] = 0.f;
            if (q < n) {
                const int bq = leafq[b] >> level;
                rhoq[b] = S.rho[mid_of(bq) - 1];
                const float dmax = fmaxf(fabsf(S.dS[lo_of(bq)]), fabsf(S.dS[lo_of(bq + 1) - 1]));
                flq[b] = kDcFloor * fmaxf(fmaxf(dmax, rhoq[b]), kDcTiny);
                k = rhoq[b] * fabsf(S.zS[q]) > kDcTol * fmaxf(fabsf(S.dS[q]), flq[b]);
            }
            kept.w[b] = __ballot(k);
        }
        uint64_t any = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int q = lane + 64 * b;
            bool c = false;
            if (q < n && kept.has(q)) {
                const int nx = kept.next(q);
                if (nx < lo_of((leafq[b] >> level) + 1)) c = dc_close(S.dS[q], S.dS[nx], S.zS[q], S.zS[nx], flq[b]);
            }
            close.w[b] = __ballot(c);
            any |= close.w[b];
        }
        if (any) {
            // one thread per block walks its close pairs in order and rotates them; the lower pole of
            // the pair loses its component of z
            sync();
            if (valid && part == 0 && e == lo) {
                int nr = 0;
                int p = close.has(lo) ? lo : close.next(lo);    // the lower pole of a close pair
                if (p < hi) {
                    const float dmax = fmaxf(fabsf(S.dS[lo]), fabsf(S.dS[hi - 1]));
                    const float fl = kDcFloor * fmaxf(fmaxf(dmax, S.rho[mid - 1]), kDcTiny);
                    float dp = S.dS[p], zp = S.zS[p];
                    while (true) {
                        const int q = kept.next(p);
                        if (q >= hi) break;
                        float dq = S.dS[q], zq = S.zS[q];
                        if (dc_close(dp, dq, zp, zq, fl)) {
                            const float big = fmaxf(fabsf(zp), fabsf(zq)), r = fminf(fabsf(zp), fabsf(zq)) / big;
                            const float tau = big * sqrtf(fmaf(r, r, 1.f));
                            const float c = zq / tau, s = -zp / tau;
                            const float np = dp * c * c + dq * s * s, nq = dp * s * s + dq * c * c;
                            const int cp = S.perm[p], cq = S.perm[q];
                            S.dS[p] = np;
                            S.zS[p] = 0.f;
                            S.dS[q] = dq = nq;
                            S.zS[q] = zq = tau;
                            S.rot[lo + nr] = make_float4(__int_as_float(cp), __int_as_float(cq), c, s);
                            ++nr;
                            const float fp = S.first[cp], fq = S.first[cq], lp = S.last[cp], lq = S.last[cq];
                            S.first[cp] = fmaf(c, fp, s * fq);
                            S.first[cq] = fmaf(c, fq, -s * fp);
                            S.last[cp] = fmaf(c, lp, s * lq);
                            S.last[cq] = fmaf(c, lq, -s * lp);
                            p = q;                              // has moved: its upper neighbour may be close now
                            dp = dq;
                            zp = zq;
                        } else {
                            p = close.next(p);                  // untouched poles in between stay apart
                            if (p >= hi) break;
                            dp = S.dS[p];
                            zp = S.zS[p];
                        }
                    }
                }
                S.nrot[lo] = nr;
            }
            sync();
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int q = lane + 64 * b;
                const float d = S.dS[q < n ? q : 0], z = S.zS[q < n ? q : 0];
                kept.w[b] = __ballot(q < n && rhoq[b] * fabsf(z) > kDcTol * fmaxf(fabsf(d), flq[b]));
            }
        }

        // ---- slots: kept poles in ascending order, then the deflated ones ----
        // From here to the eigenvalues the merge is in units of a power of two that takes rho to [0.5, 1): the poles that deflation leaves are
        // then below 2.1e6 and at least 4e-13 apart, and the third power of a distance is a number.  In units of the matrix they may be
        // 1e-17 apart; merges of blocks of 1e-9 to 1e-12 of it, whose third powers overflowed, took up to 50 evaluations of bisections instead of 6
        // (256 matrices, us per launch: 32x32 with such a block 42.6, 64x64 81.7; without 26, 57).
        const int K = kept.below(hi) - kept.below(lo);
        if (valid && part == 0) {
            const int before = kept.below(e) - kept.below(lo);
            const bool in = kept.has(e);
            const int slot = in ? before : K + k - before;
            const float d = S.dS[e], z = S.zS[e];
            const int col = S.perm[e];
            const int unit = __builtin_amdgcn_frexp_expf(S.rho[mid - 1]);
            S.dz[base + slot] = in ? make_float2(ldexpf(d, -unit), z * z) : make_float2(kDcFar, 0.f);
            S.zs[base + slot] = make_float2(in ? z : 0.f, __int_as_float(col * LD));
            S.dd[lo + slot] = d;
            S.fl[base + slot] = make_float2(S.first[col], S.last[col]);
            for (int i = k + m; i < Mp; i += m) {
                S.dz[base + i] = make_float2(kDcFar, 0.f);
                S.zs[base + i] = make_float2(0.f, __int_as_float(N * LD));
                S.fl[base + i] = make_float2(0.f, 0.f);
            }
        }
        sync();
        // poles that the loops visit: the same count in every lane
        const int trip = sh == 0 ? __builtin_amdgcn_readfirstlane(kept.below(n)) : M;

        // ---- secular equation: thread e finds root k of its block ----
        const bool root = valid && k < K;
        float dorg = 0.f, mu = 0.f;
        float dl[PP], z2[PP];               // distances from the origin of the root, squares of z
        {
            const float2* const pz = S.dz + base;
            const float weight = valid ? S.rho[mid - 1] : 1.f;
            const int unit = __builtin_amdgcn_frexp_expf(weight);
            const float rho = __builtin_amdgcn_frexp_mantf(weight);
            const float rinv = __builtin_amdgcn_rcpf(rho);
            const bool many = root && K > 1;
            const int i1 = many ? min(k, K - 2) : 0;
            const bool last = k == K - 1;
            const float2 pk = pz[root ? k : 0], p1 = pz[i1], p2 = pz[many ? i1 + 1 : 0];
            const float gap = last ? 1.00001f * rho : p2.x - pk.x;       // |z| <= 1
            const float half = 0.5f * gap;
            // this thread's poles stay in registers for all iterations
            float fm = 0.f, dm = 0.f, hm = 0.f;     // at the middle of the gap: value, first and half the second derivative
#pragma unroll
            for (int c = 0; c < PP; c += 4) {
                if (c * TPE < trip) {
                    const float4* const q = reinterpret_cast<const float4*>(pz + c * TPE + 4 * part);
                    const float4 q0 = q[0], q1 = q[1];
                    dl[c] = q0.x, dl[c + 1] = q0.z, dl[c + 2] = q1.x, dl[c + 3] = q1.z;
                    z2[c] = q0.y, z2[c + 1] = q0.w, z2[c + 2] = q1.y, z2[c + 3] = q1.w;
#pragma unroll
                    for (int i = c; i < c + 4; ++i) {
                        const float r = __builtin_amdgcn_rcpf((dl[i] - pk.x) - half), w = z2[i] * r, wr = w * r;
                        fm += w;
                        dm += wr;
                        hm = fmaf(wr, r, hm);
                    }
                } else {
#pragma unroll
                    for (int i = c; i < c + 4; ++i) dl[i] = kDcFar, z2[i] = 0.f;
                }
            }
            fm = dc_sum<TPE>(fm) + rinv;
            dm = dc_sum<TPE>(dm);
            hm = dc_sum<TPE>(hm);
            const bool right = !last && fm < 0.f;
            dorg = right ? p2.x : pk.x;
            // the pole at the origin leaves the sums: its term is known exactly, and near a root that almost
            // touches it would swamp what the other poles contribute
            const int org = right ? k + 1 : k;
            const float zo = right ? p2.y : pk.y;
#pragma unroll
            for (int c = 0; c < PP; c += 4) {
                const int j = c * TPE + 4 * part;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    dl[c + i] -= dorg;
                    z2[c + i] = j + i == org ? 0.f : z2[c + i];
                }
            }
            // Do: the other pole of the interpolation
            SecularRoot x(last, right, zo, (right || last ? p1.x : p2.x) - dorg, gap, fm, dm, hm);
            bool open = many;
            int it = 0;
            for (; it < kDcMaxIter && __ballot(open) != 0; ++it) {
                float F = 0.f, mag = 0.f, dF = 0.f, hF = 0.f;       // over all poles but the origin
#pragma unroll
                for (int c = 0; c < PP; c += 4) {
                    if (c * TPE < trip) {
#pragma unroll
                        for (int i = c; i < c + 4; ++i) {
                            const float r = __builtin_amdgcn_rcpf(dl[i] - x.mu);
                            const float w = z2[i] * r, wr = w * r;
                            F += w;
                            mag += fabsf(w);
                            dF += wr;
                            hF = fmaf(wr, r, hF);
                        }
                    }
                }
                F = dc_sum<TPE>(F);
                mag = dc_sum<TPE>(mag);
                dF = dc_sum<TPE>(dF);
                hF = dc_sum<TPE>(hF);
                open = x.step(open, rinv, F, mag, dF, hF);
            }
            if (it == kDcMaxIter) unresolved += (int)__builtin_popcountll(__ballot(open && part == 0));
            mu = x.mu;
            if (root && !many) {
                dorg = pk.x;
                mu = rho * pk.y;
            }
            lam = root ? ldexpf(dorg + mu, unit) : S.dd[valid ? e : 0];
            if (valid && part == 0) S.om[base + k] = make_float2(dorg, mu);
            if (valid && part == 0)
                for (int i = k + m; i < Mp; i += m) S.om[base + i] = make_float2(0.f, 0.f);
        }
        sync();

        // ---- the z of which these are the exact roots, up to a common factor ----
        {
            float prod = 1.f;
            const float dk = S.dz[base + (root ? k : 0)].x;
            auto ratio = [&](int i, float d, float ox, float oy) {
                const float x = ((dk - ox) - oy) * __builtin_amdgcn_rcpf(i == k ? 1.f : dk - d);
                prod *= i < K ? x : 1.f;
            };
#pragma unroll
            for (int c = 0; c < PP; c += 4) {
                if (c * TPE < trip) {
                    const int i = c * TPE + 4 * part;
                    const float4* const q = reinterpret_cast<const float4*>(S.dz + base + i);
                    const float4* const o = reinterpret_cast<const float4*>(S.om + base + i);
                    const float4 q0 = q[0], q1 = q[1], o0 = o[0], o1 = o[1];
                    ratio(i, q0.x, o0.x, o0.y);
                    ratio(i + 1, q0.z, o0.z, o0.w);
                    ratio(i + 2, q1.x, o1.x, o1.y);
                    ratio(i + 3, q1.z, o1.z, o1.w);
                }
            }
            prod = dc_product<TPE>(prod);
            if (root && part == 0) S.zs[base + k].x = copysignf(__builtin_amdgcn_sqrtf(fabsf(prod)), S.zs[base + k].x);
        }
        sync();

        // ---- eigenvectors of the merge ----
        {
            // the first and last row follow by dot products, so that eigenvalues only, without any of
            // the rest, are the same numbers
            float nrm = 0.f, f = 0.f, l = 0.f;
            const int visit = WANT_V ? M : trip;
#pragma unroll
            for (int c = 0; c < PP; c += 4) {
                if (c * TPE < visit && valid) {
                    const int j = c * TPE + 4 * part;
                    const float4* const w = reinterpret_cast<const float4*>(S.zs + base + j);
                    const float4* const g = reinterpret_cast<const float4*>(S.fl + base + j);
                    const float4 w0 = w[0], w1 = w[1], g0 = g[0], g1 = g[1];
                    const float z[4] = {w0.x, w0.z, w1.x, w1.z}, off[4] = {w0.y, w0.w, w1.y, w1.w};
                    const float fr[4] = {g0.x, g0.z, g1.x, g1.z}, la[4] = {g0.y, g0.w, g1.y, g1.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float u = z[i] * __builtin_amdgcn_rcpf(dl[c + i] - mu);
                        nrm = fmaf(u, u, nrm);
                        f = fmaf(u, fr[i], f);
                        l = fmaf(u, la[i], l);
                        if (WANT_V) S.U[__float_as_int(off[i]) + e] = root ? u : (j + i == k ? 1.f : 0.f);
                    }
                }
            }
            const float rn = root ? dc_rsqrt(dc_sum<TPE>(nrm)) : 1.f;
            f = dc_sum<TPE>(f) * rn;
            l = dc_sum<TPE>(l) * rn;
            if (valid && !root) {
                const float2 own = S.fl[base + k];
                f = own.x;
                l = own.y;
            }
            if (valid && part == 0) {
                S.first[e] = f;
                S.last[e] = l;
                if (WANT_V) S.rn[e] = rn;
            }
        }
        if (WANT_V) {
            if (any) {
                if (TPE > 1) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
                if (valid && part == 0) {
                    for (int r = S.nrot[lo] - 1; r >= 0; --r) {
                        const float4 g = S.rot[lo + r];
                        float* const up = S.U + __float_as_int(g.x) * LD + e;
                        float* const uq = S.U + __float_as_int(g.y) * LD + e;
                        const float a = *up, b = *uq;
                        *up = fmaf(g.z, a, -g.w * b);
                        *uq = fmaf(g.w, a, g.z * b);
                    }
                }
            }
            sync();
            // ---- V <- V U, block diagonal times block diagonal ----
            if (M <= 8) {
                // blocks of at most four rows before the merge: this thread's column from plain FMAs
                // (the matrix cores would spend a whole tile product on it)
                const int k0 = part & 1 ? mid : lo, k1 = part & 1 ? hi : mid;      // rows and columns of one half
                float out[4], u[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = k0 + i < k1 ? S.U[(k0 + i) * LD + e] : 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    out[r] = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) out[r] = fmaf(S.V[min(k0 + r, N - 1) * LD + min(k0 + i, N - 1)], u[i], out[r]);
                }
                const float rn = S.rn[e];
                sync();
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (valid && part < 2 && k0 + r < k1) S.V[(k0 + r) * LD + e] = out[r] * rn;
            } else if constexpr (NWV == 1) {
                // one tile (32 x 32, 16 x 16 for N = 16)
                constexpr int TS = DcTile<N>::size, KT = 64 / TS, AR = TS * TS / 64;
                const int loT = lane & (TS - 1), hiT = lane / TS;
                const float* const va = S.V + loT * LD + hiT;
                const float* const ub = S.U + hiT * LD + loT;
                typename DcTile<N>::acc acc{};
                for (int kk = 0; kk < n; kk += 4 * KT) {
                    float a[4], u[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        // behind n the operands are read within bounds, and dropped
                        const int at = min(kk + i * KT, N - KT);
                        a[i] = va[at];
                        u[i] = kk + i * KT < n ? ub[at * LD] : 0.f;
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc = dc_mfma(a[i], u[i], acc);
                }
                sync();
                const float r = S.rn[loT];
#pragma unroll
                for (int v = 0; v < AR; ++v) S.V[dc_row<TS>(v, lane) * LD + loT] = acc[v] * r;
            } else {
                // Tiles of 16 x 16 that start where the blocks do: a task is 16 rows of one half, times all columns of its block. It holds
                // its rows of V (only it reads them) as left operands, so each result goes straight back over them.  With
                // 32 x 32 tiles at fixed places the blocks of n = 100 (7, 13, 25, 50 rows), which straddle them, took 48 k cycles over
                // all levels, 36 rows 11.3 k; now 28 k and 9.2 k.
                // Nothing is clamped or masked on the way in: what lies behind a half or a block is zero in one of the operands or
                // belongs to a row or column of the result that is dropped; the arrays reach as far as these reads (DcShared).
                constexpr int KG = N / 32;                                  // groups of four steps (16 rows) of the longest half
                const int loT = lane & 15, hiT = lane >> 4;
                const int rows = (n + (2 << sh) - 1) >> (sh + 1);           // of the largest half
                for (int t = __builtin_amdgcn_readfirstlane(wv); t < ((rows + 15) >> 4) << (sh + 1); t += NWV) {
                    const int half = t & ((2 << sh) - 1), k0 = (half * n) >> (sh + 1), k1 = ((half + 1) * n) >> (sh + 1);
                    const int r0 = k0 + 16 * (t >> (sh + 1)), c0 = lo_of(half >> 1), c1 = lo_of((half >> 1) + 1);
                    if (r0 >= k1) continue;
                    const float* const va = S.V + min(r0 + loT, N - 1) * LD + k0 + hiT;
                    float a[KG][4];
#pragma unroll
                    for (int g = 0; g < KG; ++g)
                        if (g == 0 || k0 + 16 * g < k1)
#pragma unroll
                            for (int i = 0; i < 4; ++i) a[g][i] = va[16 * g + 4 * i];
                    for (int col = c0; col < c1; col += 32) {
                        const float* const u = S.U + (k0 + hiT) * LD + col + loT;
                        const float ra = S.rn[col + loT], rb = S.rn[col + 16 + loT];
                        dc_acc16 xa = dc_acc16{}, xb = dc_acc16{};
                        float ua[2][4], ub[2][4];                           // a group ahead
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            ua[0][i] = u[4 * i * LD];
                            ub[0][i] = u[4 * i * LD + 16];
                        }
#pragma unroll
                        for (int g = 0; g < KG; ++g) {
                            if (g == 0 || k0 + 16 * g < k1) {
                                if (g + 1 < KG && k0 + 16 * (g + 1) < k1) {
#pragma unroll
                                    for (int i = 0; i < 4; ++i) {
                                        ua[(g + 1) & 1][i] = u[(16 * (g + 1) + 4 * i) * LD];
                                        ub[(g + 1) & 1][i] = u[(16 * (g + 1) + 4 * i) * LD + 16];
                                    }
                                }
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    xa = dc_mfma(a[g][i], ua[g & 1][i], xa);
                                    xb = dc_mfma(a[g][i], ub[g & 1][i], xb);
                                }
                            }
                        }
                        float* const out = S.V + (r0 + 4 * hiT) * LD + col + loT;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const bool in = r0 + 4 * hiT + v < k1;
                            if (in && col + loT < c1) out[v * LD] = xa[v] * ra;
                            if (in && col + 16 + loT < c1) out[v * LD + 16] = xb[v] * rb;
                        }
                    }
                }
            }
            sync();
        }
    }
    if (part == 0) S.D[e] = valid ? lam : __builtin_inff();
    if (T > 64 && unresolved && lane == 0) atomicAdd(&S.unresolved, unresolved);
    sync();
    return T > 64 ? S.unresolved : unresolved;
}

// Rank of column e's eigenvalue among all n (ties by column): the ascending output order; thread `part` of the TPE that
// share an eigenvalue looks at every TPE-th group of four.  With a non-finite eigenvalue among them (`odd`) the columns
// stay where they are.
template <int N, int TPE, bool WANT_V>
__device__ __forceinline__ int dc_rank(const DcShared<N, TPE, WANT_V>& S, int n, int e, int part, bool odd) {
    const float de = S.D[e];
    int rank = 0;
    for (int j = 4 * part; j < n; j += 4 * TPE) {           // D is +inf from n on
        const float4 q = *reinterpret_cast<const float4*>(S.D + j);
        rank += (q.x < de || (q.x == de && j < e)) ? 1 : 0;
        rank += (q.y < de || (q.y == de && j + 1 < e)) ? 1 : 0;
        rank += (q.z < de || (q.z == de && j + 2 < e)) ? 1 : 0;
        rank += (q.w < de || (q.w == de && j + 3 < e)) ? 1 : 0;
    }
    rank = (int)dc_sum<TPE>((float)rank);
    return odd ? e : rank;
}

// Number of non-finite eigenvalues (the same in every wavefront).
template <int N, int TPE, bool WANT_V>
__device__ __forceinline__ int dc_non_finite(const DcShared<N, TPE, WANT_V>& S, int n, int lane) {
    int count = 0;
#pragma unroll
    for (int b = 0; b < (N + 63) / 64; ++b) {
        const int q = lane + 64 * b;
        count += (int)__builtin_popcountll(__ballot(q < n && !(fabsf(S.D[q < n ? q : 0]) < __builtin_inff())));
    }
    return count;
}

}  // namespace bed
#endif
