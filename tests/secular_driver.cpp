// The root finder of the divide and conquer (csrc/bed_secular.hpp) on the CPU: random merges of K poles, the residual that each root leaves in
// long double in units of the rounding of its sums, and the evaluations it took.
// Prints: largest residual of the last root of a merge, largest of the others, most evaluations, roots left open.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#define __device__
#define __forceinline__ inline
static inline float __builtin_amdgcn_rcpf(float x) { return 1.f / x; }
static inline float __builtin_amdgcn_sqrtf(float x) { return sqrtf(x); }
#include "bed_secular.hpp"

struct Found {
    float origin, mu;
    int evaluations;
    bool open;
};

// As dc_solve has one thread do it, K > 1.
static Found find(const std::vector<float>& d, const std::vector<float>& z2, float rho, int k) {
    const int K = (int)d.size(), i1 = std::min(k, K - 2);
    const bool last = k == K - 1;
    const float rinv = 1.f / rho, gap = last ? 1.00001f * rho : d[k + 1] - d[k], half = 0.5f * gap;
    float fm = rinv, dm = 0.f, hm = 0.f;
    for (int i = 0; i < K; ++i) {
        const float r = 1.f / ((d[i] - d[k]) - half), w = z2[i] * r, wr = w * r;
        fm += w, dm += wr, hm = fmaf(wr, r, hm);
    }
    const bool right = !last && fm < 0.f;
    const int org = right ? k + 1 : k;
    bed::SecularRoot x(last, right, z2[org], d[right || last ? i1 : i1 + 1] - d[org], gap, fm, dm, hm);
    bool open = true;
    int it = 0;
    for (; it < 60 && open; ++it) {
        float F = 0.f, mag = 0.f, dF = 0.f, hF = 0.f;
        for (int i = 0; i < K; ++i) {
            if (i == org) continue;
            const float r = 1.f / ((d[i] - d[org]) - x.mu), w = z2[i] * r, wr = w * r;
            F += w, mag += fabsf(w), dF += wr, hF = fmaf(wr, r, hF);
        }
        open = x.step(open, rinv, F, mag, dF, hF);
    }
    return {d[org], x.mu, it, open};
}

int main(int argc, char** argv) {
    const int K = atoi(argv[1]), merges = atoi(argv[2]);
    const double spread = atof(argv[3]);            // the poles lie within this of each other
    std::mt19937 gen(20 + K);
    auto uniform = [&]() { return gen() / 4294967296.0; };
    double worst_last = 0, worst = 0;
    int most = 0, left = 0;
    for (int t = 0; t < merges; ++t) {
        std::vector<double> pole(K), z(K);
        double norm = 0;
        for (int i = 0; i < K; ++i) {
            pole[i] = (t & 4 ? 0.5 : 0.0) + spread * uniform();
            z[i] = (t % 3 == 0 && uniform() < 0.3 ? pow(10, -4 * uniform()) : 1.0) * (uniform() - 0.5);
            norm += z[i] * z[i];
        }
        std::sort(pole.begin(), pole.end());
        const float rho = (float)pow(10, -3 * uniform() * (t & 1));
        // what deflation leaves of a block of norm one
        std::vector<float> d, z2;
        for (int i = 0; i < K; ++i) {
            const float p = (float)pole[i], c = (float)(fabs(z[i]) / sqrt(norm)), size = std::max(fabsf(p), 1e-6f);
            if (rho * c <= 4.8e-7f * size) continue;
            if (!d.empty()) {
                const float b = sqrtf(z2.back()), q = std::min(b, c) / std::max(b, c);
                if ((p - d.back()) * q <= 4.8e-7f * size * (q * q + 1)) continue;
            }
            d.push_back(p);
            z2.push_back(c * c);
        }
        const int kept = (int)d.size();
        for (int k = 0; kept > 1 && k < kept; ++k) {
            const Found f = find(d, z2, rho, k);
            long double F = 1 / (long double)rho, mag = F, dF = 0;
            for (int i = 0; i < kept; ++i) {
                const long double distance = ((long double)d[i] - f.origin) - f.mu, w = z2[i] / distance;
                F += w, mag += fabsl(w), dF += w / distance;
            }
            const double residual = (double)(fabsl(F) / (ldexpl(1, -24) * (mag + fabsl(f.mu) * dF)));
            (k == kept - 1 ? worst_last : worst) = std::max(k == kept - 1 ? worst_last : worst, residual);
            most = std::max(most, f.evaluations);
            left += f.open;
        }
    }
    std::printf("%.3f %.3f %d %d\n", worst_last, worst, most, left);
}
