// The scale of a problem over the whole range of its largest entry: the power
// of two and its reciprocal are finite and exact inverses, the scaled entry is
// exact, and in [1/2, 1) except at the ends of the range.
#include <cmath>
#include <cstdio>
#include <initializer_list>

#define TDE_DEV inline
#define TDE_RCP_ESTIMATE(x) (1.0 / (x))
#define TDE_RSQ_ESTIMATE(x) (1.0 / std::sqrt(x))
#include "../../paper_2605_26599_amd/csrc/tde_device.h"

int main() {
    int bad = 0;
    for (int ex = -1074; ex <= 1023; ++ex)
        for (double f : {1.0, 1.25, 1.5, 2.0 - 0x1p-52}) {
            const double mx = std::ldexp(f, ex);
            if (!(mx > 0.0) || std::isinf(mx)) continue;
            const double s = tde::scale_of(tde::dbits(mx)), inv = 1.0 / s, x = mx * inv;
            const bool ok = std::isfinite(s) && std::isfinite(inv) && s * inv == 1.0 && x > 0.0 && x * s == mx &&
                            x < (mx >= 0x1p1023 ? 2.0 : 1.0) && (mx < 0x1p-1024 || x >= 0.5);
            if (!ok && ++bad < 10) std::printf("%a: scale %a, reciprocal %a, scaled %a\n", mx, s, inv, x);
        }
    if (tde::scale_of(tde::dbits(0.0)) != 1.0) ++bad;
    std::puts(bad ? "scale bad" : "scale ok");
    return bad != 0;
}
