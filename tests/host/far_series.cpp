// The far-field series of the wide merges (tde_far.h), built for the CPU,
// against the sums they stand for in quadruple precision: poles at the edges of
// the three tiers (and just past them) and in between, on either side, one
// alone or many together, at points over the whole block.  Prints the largest
// error of value, first derivative, half the second, norm and logarithm, each
// of the sum of its terms' sizes (the logarithm of the largest |u - v| sum).
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#define TDE_DEV inline
#define TDE_ANY(c) (c)
#include "../../paper_2605_26599_amd/csrc/tde_far.h"

typedef __float128 quad;
static quad mag(quad x) { return x < 0 ? -x : x; }

// log(1 + x), |x| < 1/2, by the series of 2 atanh(x / (2 + x))
static quad log1q(quad x) {
    const quad s = x / (2 + x), s2 = s * s;
    quad p = s, t = 0;
    for (int k = 1; k < 120; k += 2) {
        t += p / k;
        p *= s2;
    }
    return 2 * t;
}

int main() {
    using namespace tde;
    std::mt19937_64 rng(5);
    auto uni = [&] { return (double)(rng() >> 11) * 0x1p-53; };
    double worst[5] = {0, 0, 0, 0, 0};
    for (int trial = 0; trial < 3000; ++trial) {
        const double c = 2.0 * uni() - 1.0, h = std::pow(10.0, -10.0 * uni());
        const int n = trial % 3 ? 1 : 1 + (int)(rng() % 50);
        double mv[kFarFold] = {0}, mn[kFarFold] = {0}, ml[kFarFold] = {0};
        std::vector<quad> del, wt, lam;  // D - c, weights, lambda - c
        for (int i = 0; i < n; ++i) {
            // distance in half-widths: at an edge (to rounding), past it, or anywhere
            const double edge[3] = {kFarRatio, 1.0 / kFarHalf, 1.0 / kFarShort};
            const double at = edge[rng() % 3];
            const double q = rng() % 3 == 0 ? at : rng() % 2 ? at * (1.0 + 1e-9) : kFarRatio * std::pow(10.0, 3.0 * uni());
            const double dd = (rng() % 2 ? 1.0 : -1.0) * q * h;  // D - c
            const double w = std::pow(10.0, -3.0 * uni());
            const double r = 1.0 / dd, u = h * r;
            far_add(mv, w * r, u);
            const double y = std::sqrt(w) * r;
            far_add(mn, y * y, u);
            // the root paired with the pole: further out, at a distance of its own
            const double tk = dd * std::pow(10.0, -8.0 * uni()), dl = dd + tk, rl = 1.0 / dl;
            const double off = dl - dd;  // exact
            far_add_log(ml, u, h * rl, u * (off * rl));
            del.push_back(dd);
            wt.push_back(w);
            lam.push_back(dl);
        }
        for (int k = 0; k < kFarFold; ++k) {
            mn[k] *= k + 1;
            ml[k] /= k + 1;
        }
        for (int p = 0; p <= 16; ++p) {
            const double t = p / 8.0 - 1.0;
            const quad x = (quad)t * h;
            quad s[5] = {0, 0, 0, 0, 0}, z[5] = {0, 0, 0, 0, 0};
            for (size_t i = 0; i < del.size(); ++i) {
                const quad r = 1 / (del[i] - x);
                const quad y = sqrt((double)wt[i]);
                const quad v[5] = {wt[i] * r, wt[i] * r * r, wt[i] * r * r * r, y * y * r * r,
                                   log1q(-x / lam[i]) - log1q(-x / del[i])};
                for (int k = 0; k < 5; ++k) s[k] += v[k], z[k] += mag(v[k]);
                z[4] += mag((quad)h / del[i] - (quad)h / lam[i]) - mag(v[4]);
            }
            double d1, d2;
            const double val = far_value(mv, t, &d1, &d2);
            const double got[5] = {val, d1 / h, d2 / (h * h), far_value(mn, t), t * far_value(ml, t)};
            for (int k = 0; k < 5; ++k)
                if (z[k] > 0) worst[k] = std::max(worst[k], (double)(mag(got[k] - s[k]) / z[k]));
            if (far_value(mv, t) != val) worst[0] = INFINITY;
        }
    }
    std::printf("%.3e %.3e %.3e %.3e %.3e\n", worst[0], worst[1], worst[2], worst[3], worst[4]);
    return 0;
}
