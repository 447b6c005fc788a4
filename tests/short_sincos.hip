// sincos_fast on the host against the libm functions in long double (built and run by
// tests/test_short_sincos.py): "bits worst-error largest-value" per range
// 2^(bits-1) <= |x| < 2^bits, then the values at arguments that are not finite.
#include <cmath>
#include <cstdio>
#include "quadrature_device.h"
int main() {
    unsigned long long st = 12345;
    auto uniform = [&] {
        st = st * 6364136223846793005ull + 1442695040888963407ull;
        return 0.5 + 0.5 * double(st >> 11) / 9007199254740992.0;
    };
    double s, c;
    for (int e : {-20, 0, 3, 8, 16, 24, 32, 40, 43, 44, 46, 48, 50, 52, 60, 300, 1023}) {
        double worst = 0, largest = 0;
        for (int i = 0; i < 100000; ++i) {
            const double x = std::ldexp(i & 1 ? -uniform() : uniform(), e);
            igb::sincos_fast(x, s, c);
            worst = std::fmax(worst, std::fmax(std::fabs(double(s - sinl(x))), std::fabs(double(c - cosl(x)))));
            largest = std::fmax(largest, std::fmax(std::fabs(s), std::fabs(c)));
        }
        std::printf("%d %.3e %.6f\n", e, worst, largest);
    }
    for (double x : {double(NAN), double(INFINITY), -double(INFINITY)}) {
        igb::sincos_fast(x, s, c);
        std::printf("%d %d\n", std::isnan(s) ? 1 : 0, std::isnan(c) ? 1 : 0);
    }
    igb::sincos_fast(0.0, s, c);
    std::printf("%g %g\n", s, c);
    return 0;
}
