// The series behind the far-field expansions of the wide merges: moments of
// poles D outside a block [c - h, c + h] of the spectrum and their polynomials
// in t = (x - c)/h, |t| <= 1, with u = h/(D - c), |u| <= 1/kFarRatio:
//   value      1/(D - x) = (u/h) sum_k (u t)^k, and its derivatives by x;
//   norm       1/(D - x)^2 = (u/h)^2 sum_k (k + 1) (u t)^k;
//   logarithm  log((1 - v t)/(1 - u t)) = sum_(m >= 1) (u^m - v^m) t^m / m,
//              v = h/(lambda - c) of the root paired with the pole.
// What kFarTerms = 28 terms leave out at |u| = 1/kFarRatio, 16 terms at |u| =
// kFarHalf and 8 terms at |u| = kFarShort, of the sum itself (y = u t, N terms):
//   value      y^N:                 1.4e-17, 5.4e-18, 1.4e-17
//   norm       y^N (N + 1 - N y):   5.0e-16, 9.9e-17, 1.3e-16
//   logarithm  u^N (1 + u)/(1 - u): 2.3e-17, 6.4e-18, 1.4e-17
// All are below the last bit but the norm's, which reaches 2.3 eps of the nearest
// far poles' share in a sum that the block's own poles dominate.  The value's
// derivatives (1.9e-15, 1.1e-15, 1.4e-14 and 1.3e-13, 1.1e-13, 6.5e-12) only
// steer the secular iteration.
#pragma once
#include <math.h>

#ifndef TDE_DEV
#define TDE_DEV __device__ __forceinline__
#endif
// Whether the condition holds in any lane of the wave.
#ifndef TDE_ANY
#define TDE_ANY(c) __any(c)
#endif

namespace tde {

constexpr int kFarTerms = 28;
constexpr int kFarFold = 32;  // kFarTerms padded to the fold's power of two
constexpr double kFarRatio = 4.0;
constexpr double kFarHalf = 1.0 / 12.0, kFarShort = 1.0 / 128.0;

// Adds v u^k to m[k] for the k that count: four moments per step of u^4 (37
// operations for 28 moments instead of the 56 of taking each power from the
// last one), 8 or 16 moments where every lane's u is small enough.
TDE_DEV void far_add(double (&m)[kFarFold], double v, double u) {
    const double au = fabs(u);
    const double u2 = u * u, u3 = u2 * u, u4 = u2 * u2;
    auto four = [&](int k) {
        m[k] += v;
        m[k + 1] = fma(v, u, m[k + 1]);
        m[k + 2] = fma(v, u2, m[k + 2]);
        m[k + 3] = fma(v, u3, m[k + 3]);
        v *= u4;
    };
    four(0);
    four(4);
    if (TDE_ANY(au > kFarShort)) {
        four(8);
        four(12);
        if (TDE_ANY(au > kFarHalf)) {
            four(16);
            four(20);
            four(24);
        }
    }
}
// Adds u^(k+1) - v^(k+1) to m[k], du = u - v, by
// u^(k+j) - v^(k+j) = u^j (u^k - v^k) + v^k (u^j - v^j).
TDE_DEV void far_add_log(double (&m)[kFarFold], double u, double v, double du) {
    const double au = fmax(fabs(u), fabs(v));
    const double u2 = u * u, v2 = v * v, u3 = u2 * u, u4 = u2 * u2, v4 = v2 * v2;
    const double d2 = du * (u + v), d3 = fma(u, d2, v2 * du), d4 = d2 * (u2 + v2);
    double em = du;  // u^(k+1) - v^(k+1)
    double vm = v;   // v^(k+1)
    auto four = [&](int k) {
        m[k] += em;
        m[k + 1] = fma(u, em, fma(vm, du, m[k + 1]));
        m[k + 2] = fma(u2, em, fma(vm, d2, m[k + 2]));
        m[k + 3] = fma(u3, em, fma(vm, d3, m[k + 3]));
        em = fma(u4, em, vm * d4);
        vm *= v4;
    };
    four(0);
    four(4);
    if (TDE_ANY(au > kFarShort)) {
        four(8);
        four(12);
        if (TDE_ANY(au > kFarHalf)) {
            four(16);
            four(20);
            four(24);
        }
    }
}
static_assert(kFarTerms == 28, "far_add and far_add_log write the steps out");


// The polynomial sum_k coef[k] t^k, and with its first derivative by t and half
// its second one.
TDE_DEV double far_value(const double* coef, double t) {
    double s = coef[kFarTerms - 1];
#pragma unroll
    for (int k = kFarTerms - 2; k >= 0; --k) s = fma(s, t, coef[k]);
    return s;
}
TDE_DEV double far_value(const double* coef, double t, double* d1, double* d2) {
    double s = coef[kFarTerms - 1], d = 0.0, c = 0.0;
#pragma unroll
    for (int k = kFarTerms - 2; k >= 0; --k) {
        c = fma(c, t, d);
        d = fma(d, t, s);
        s = fma(s, t, coef[k]);
    }
    *d1 = d;
    *d2 = c;
    return s;
}

}  // namespace tde
