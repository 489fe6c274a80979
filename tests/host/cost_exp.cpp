// cost_exp (csrc/sample_math.h) on the host against expl: prints one line per range of arguments, "from to largest rms" of the relative error
// (in steps of the smallest number where the result is subnormal), then "value of <x> <result>" lines for arguments at and past the ends.
#include "sample_math.h"
#include <cmath>
#include <cstdio>
#include <limits>

int main()
{
    const double ends[][2] = {{-708, -20}, {-20, -1}, {-1, -0.35}, {-0.35, -1e-3}, {-1e-3, 0}, {0, 1e-3}, {1e-3, 0.35}, {0.35, 1}, {1, 20}, {20, 709}};
    unsigned long long state = 88172645463325252ull;
    auto uniform = [&] {                     // xorshift64, 53 bits
        state ^= state << 13;
        state ^= state >> 7;
        state ^= state << 17;
        return (double)(state >> 11) * 0x1p-53;
    };
    for (const auto &e : ends) {
        long double most = 0, squares = 0;
        const int count = 130000;
        for (int i = 0; i < count; ++i) {
            const double x = e[0] + (e[1] - e[0]) * uniform();
            const long double want = expl((long double)x), d = fabsl((long double)cost_exp(x) - want) / want;
            if (d > most) most = d;
            squares += d * d;
        }
        printf("range %g %g %.4Le %.4Le\n", e[0], e[1], most, sqrtl(squares / count));
    }
    long double most = 0;
    for (int i = 0; i < 100000; ++i) {
        const double x = -746.0 + 37.6 * uniform();
        const long double d = fabsl((long double)cost_exp(x) - expl((long double)x)) / (long double)0x1p-1074;
        if (d > most) most = d;
    }
    printf("subnormal %.4Lf\n", most);
    const double inf = std::numeric_limits<double>::infinity();
    const double at[] = {0.0, -0.0, -745.0, -746.0, -747.0, -1e10, -1e17, -1e300, -inf, 709.75, 709.79, 710.0, 711.0, 1e10, 1e16, 1e17, 1e25, 1e300, inf, std::nan("")};
    for (double x : at) printf("value of %.17g %.17g\n", x, cost_exp(x));
}
