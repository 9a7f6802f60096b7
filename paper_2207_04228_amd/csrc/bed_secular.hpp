// One root of the secular equation 1/rho + sum z_j^2 / (d_j - lambda) = 0 from sums over the poles that the caller forms: bracket, rational
// interpolation, end of the iteration.  Nothing here depends on the lane: a CPU build takes it too, with the two hardware functions
// (reciprocal, square root) defined before it.
#ifndef BED_SECULAR_HPP
#define BED_SECULAR_HPP

namespace bed {

// Root of c x^2 - 2 a x + b that interpolates a root between the two poles (s = 1) or right of both (s = -1).
__device__ __forceinline__ float dc_quadratic(float a, float b, float c, float s) {
    const float disc = s * __builtin_amdgcn_sqrtf(fmaxf(fmaf(a, a, -b * c), 0.f));
    const bool neg = s * a <= 0.f;
    const float num = neg ? a - disc : b;
    const float den = neg ? c : a + disc;
    return num * __builtin_amdgcn_rcpf(den);
}

struct SecularRoot {
    float mu, lb, ub;           // the iterate and its bracket, measured from the origin: the pole that is nearer to the root
    float zo, Do, rDo, sgn;     // z^2 of the origin, the other pole of the interpolation (from the origin), its reciprocal, -1 right of all poles
    float enough;               // a step of less than this much of the distance of the nearer pole is the last

    // The gap between two poles (last: right of all poles, where it ends at a bound), and the function, its first and half its second
    // derivative at the middle of it.  right: the origin is the upper pole.
    __device__ __forceinline__ SecularRoot(bool last, bool right, float zo_, float Do_, float gap, float fm, float dm, float hm) {
        const float half = 0.5f * gap;
        zo = zo_;
        Do = Do_;
        lb = last ? (fm < 0.f ? half : 0.f) : (right ? -half : 0.f);
        ub = last ? (fm < 0.f ? gap : half) : (right ? 0.f : half);
        rDo = __builtin_amdgcn_rcpf(Do);
        sgn = last ? -1.f : 1.f;
        // The next error is of the order of the cube of the step over the distance of the nearer pole: below 2^-9 of that distance the next step
        // would be below the rounding of mu.  Right of all poles it is of the order of the square: with 2^-9 there the worst residuals of the
        // largest roots (random merges of 8 to 128 poles, units of the rounding of their sums) were 5.8 to 6.4, with 2^-10, which leaves a
        // quarter, 4.0 to 4.6, as with 2^-12: the iteration stops at 4.  Evaluations of that root 1.82 / 1.89 / 1.97 (64 poles).
        enough = last ? 9.765625e-4f : 1.953125e-3f;
        const float at = right ? -half : half;
        const float r = __builtin_amdgcn_rcpf(at), w = zo * r;              // less the term of the origin, -zo / at
        const float x = interpolate(true, at, fm + w, fmaf(-w, r, dm), fmaf(w * r, r, hm));
        mu = (x > lb) & (x < ub) ? x : 0.5f * (lb + ub);
    }

    // The root of c + s / (Do - x) - so / x = 0, where c + s / (Do - x) - (so - zo) / x has the value R, the derivative dR and half
    // the second derivative hR that 1/rho and the terms of all poles but the origin have at `at` (Gragg 1965 for two poles;
    // third order).  Every pole's share of s and of so - zo is positive, right of all poles excepted, where so = zo, exact,
    // and Do takes the whole derivative (second order).  Written in x and with `at` for Do - d, so that nothing cancels however near the
    // root is to the origin.  Evaluations, largest of a level's roots, added over the levels, in float32 on the CPU, full-rank, decaying and
    // rank-deficient covariances of 8 / 16 / 32 / 64 / 128 rows: fixed weight and middle way in turn (second order), from a start
    // without derivatives, 4.1 / 8.3 / 13.9 / 19.1 / 25.8, this 2.8 / 5.8 / 9.2 / 13.5 / 17.7; of 6000 merges with random poles and weights
    // down to 1e-12 none took more than 8 (before: 11).  us per launch: 512 x 32x32 35.1 -> 33.3, 16384 x 32x32 273 -> 261,
    // 256 x 64x64 66.2 -> 64.1, 256 x 128x128 155 -> 151.
    // From the start, where x is far from a root next to an origin of small weight, so - zo is left out if it swamps zo (24 rows of rank 18
    // took 13.1 evaluations with it, 9.0 without, 12.6 before).
    __device__ __forceinline__ float interpolate(bool start, float at, float R, float dR, float hR) const {
        const float d = Do - at;
        float side = fmaxf(at * fmaf(-d, hR, dR) * rDo, 0.f);                  // (so - zo) / at^2
        if (start) side = side * at * at > 128.f * zo ? 0.f : side;
        const float rest = fmaxf(dR - side, 0.f);
        const float sa = side * at, rd = rest * d;
        const float so = fmaf(sa, at, zo);
        const float c = sa + (R - rd);
        const float a = fmaf(Do, sa + R, fmaf(-rd, at, so));
        return dc_quadratic(0.5f * a, so * Do, c, sgn);
    }

    // At mu, over all poles but the origin: the sum F, that of the magnitudes, first and half the second derivative.  Goes on to the
    // next mu; false where this was the last.
    __device__ __forceinline__ bool step(bool open, float rinv, float F, float mag, float dF, float hF) {
        const float own = zo * __builtin_amdgcn_rcpf(mu);
        mag += fabsf(own) + rinv;
        const float R = F + rinv;
        F = R - own;
        const float err = fmaf(2.3841858e-7f, mag, 5.9604645e-8f * fabsf(mu) * dF);
        lb = F < 0.f ? mu : lb;
        ub = F < 0.f ? ub : mu;
        const float x = interpolate(false, mu, R, dF, hF);
        const bool ok = (x > lb) & (x < ub);            // mu is one of the two; & everywhere, without branches
        const bool small = ok & (fabsf(x - mu) <= enough * fminf(fabsf(mu), fabsf(Do - mu)));
        const float y = ok ? x : 0.5f * (lb + ub);
        const bool go = open & !(fabsf(F) <= err) & (y > lb) & (y < ub);
        mu = go ? y : mu;
        return go & !small;
    }
};

}  // namespace bed
#endif
