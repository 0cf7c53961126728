// The secular iteration of the device header, built for the CPU with g++ (the
// hardware estimates replaced by 24-bit ones), against f evaluated in
// quadruple precision: prints the roots tried, the largest backward error
// |f(lambda)| / (1 + rho sum |z_j^2/(D_j - lambda)|) in units of 2^-52 and the
// mean sweeps per root, per kind of problem.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#define TDE_DEV inline
static inline double cut24(double x) {
    union { double d; unsigned long long u; } c;
    c.d = x;
    c.u &= ~((1ULL << 28) - 1);
    return c.d;
}
#define TDE_RCP_ESTIMATE(x) cut24(1.0 / (x))
#define TDE_RSQ_ESTIMATE(x) cut24(1.0 / std::sqrt(x))
#define TDE_ATOMIC_MAX_U64(p, v) (*(p) = std::max(*(p), (v)))
#define TDE_ATOMIC_OR(p, v) (*(p) |= (v))
#include "../../paper_2605_26599_amd/csrc/tde_device.h"

typedef __float128 quad;

int main(int argc, char** argv) {
    const int kind = argc > 1 ? std::atoi(argv[1]) : 0;
    std::mt19937_64 rng(11 + (unsigned)kind);
    auto u = [&] { return (double)(rng() >> 11) * 0x1p-53; };
    const double tol = 8.0 * DBL_EPSILON;
    long roots = 0, sweeps = 0, capped = 0;
    double worst = 0.0;
    for (int t = 0; t < 60; ++t) {
        const int n = 2 + (int)(rng() % 130);
        std::vector<double> d((size_t)n), z((size_t)n);
        for (int i = 0; i < n; ++i) {
            const double x = 2.0 * u() - 1.0;
            d[i] = kind == 1 ? std::cos(3.14159 * (i + 1) / (n + 1))                    // Jacobi-like
                 : kind == 2 ? std::copysign(std::pow(10.0, -8.0 * u()), x)             // graded
                 : kind == 3 ? (double)(rng() % 8) * 0.1 + 1e-12 * n * u() : x;         // clusters
            z[i] = kind == 4 ? std::pow(10.0, -14.0 * u()) : kind == 1 ? 0.5 + u() : std::pow(10.0, -6.0 * u() * u());
        }
        std::sort(d.begin(), d.end());
        double norm = 0.0;
        for (double x : z) norm += x * x;
        const double rho = 2.0 * std::pow(10.0, -3.0 * u());
        // what deflation would leave
        std::vector<double> D, Z, W;
        for (int i = 0; i < n; ++i) {
            const double zi = z[i] / std::sqrt(norm);
            if (!(rho * zi > tol)) continue;
            if (!D.empty() && !(d[i] > D.back() && !tde::close_pair(D.back(), Z.back(), d[i], zi, tol))) continue;
            D.push_back(d[i]);
            Z.push_back(zi);
            W.push_back(zi * zi);
        }
        const int K = (int)D.size();
        for (int k = 0; k < K && K > 1; ++k) {
            int o;
            double tau;
            const int it = tde::secular_root<tde::RedSerial>(k, K, D.data(), Z.data(), W.data(), rho, 0, 1,
                                                             tde::kSecMaxIter, &o, &tau);
            if (it < 0) ++capped;
            sweeps += it < 0 ? tde::kSecMaxIter : it;
            ++roots;
            quad f = 1, size = 1;
            for (int j = 0; j < K; ++j) {
                const quad x = (quad)rho * Z[j] * Z[j] / (((quad)D[j] - (quad)D[o]) - (quad)tau);
                f += x;
                size += x < 0 ? -x : x;
            }
            worst = std::max(worst, std::fabs((double)(f / size)) / DBL_EPSILON);
            // strictly inside the bracket, on its own side of the origin
            if (!(o == k ? tau > 0.0 : (o == k + 1 && tau < 0.0)) || (k < K - 1 && std::fabs(tau) >= D[k + 1] - D[k]))
                worst = INFINITY;
        }
    }
    std::printf("%ld %ld %.3f %.3f\n", roots, capped, worst, (double)sweeps / (double)roots);
    return 0;
}
