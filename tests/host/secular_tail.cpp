// The secular iteration of the device header on problems that drive its
// safeguard: poles and weights over fifteen decades, clusters of poles with
// gaps down to 1e-15, weak couplings.  Prints the roots tried, those that hit
// the cap, the most sweeps any of them took, how many took more than twelve,
// and the largest backward error in quadruple precision (units of 2^-52).
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
    std::mt19937_64 rng(1000 + (unsigned)kind);
    auto u = [&] { return (double)(rng() >> 11) * 0x1p-53; };
    const double tol = 8.0 * DBL_EPSILON;
    long roots = 0, capped = 0, slow = 0;
    int most = 0;
    double worst = 0.0;
    for (int t = 0; t < 3000; ++t) {
        const int n = 2 + (int)(rng() % 60);
        std::vector<double> d((size_t)n), z((size_t)n);
        for (int i = 0; i < n; ++i) {
            const double x = 2.0 * u() - 1.0;
            d[i] = kind == 0 ? x
                 : kind == 2 ? (double)(rng() % 4) * 0.3 + std::pow(10.0, -15.0 * u())
                             : std::copysign(std::pow(10.0, -15.0 * u()), x);
            z[i] = kind != 3 ? std::pow(10.0, -14.0 * u())
                 : rng() % 3 ? 1e-15 * (1.0 + u()) : std::pow(10.0, -7.0 * u());
        }
        std::sort(d.begin(), d.end());
        double norm = 0.0;
        for (double x : z) norm += x * x;
        const double rho = 2.0 * std::pow(10.0, -12.0 * u() * u());
        std::vector<double> D, Z, W;  // what deflation would leave
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
            most = std::max(most, it < 0 ? tde::kSecMaxIter : it);
            slow += it < 0 || it > 12;
            ++roots;
            quad f = 1, size = 1;
            for (int j = 0; j < K; ++j) {
                const quad x = (quad)rho * Z[j] * Z[j] / (((quad)D[j] - (quad)D[o]) - (quad)tau);
                f += x;
                size += x < 0 ? -x : x;
            }
            worst = std::max(worst, std::fabs((double)(f / size)) / DBL_EPSILON);
        }
    }
    std::printf("%ld %ld %d %ld %.3f\n", roots, capped, most, slow, worst);
    return 0;
}
