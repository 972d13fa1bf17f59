// CPU test of log_normal (zb_log.h), the logarithm of a positive normal double from its
// mantissa and exponent: bit by bit log_series on every kind of argument, with approximate
// reciprocals perturbed to their assumed bound.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <random>

#include "zb_log.h"

int main()
{
    std::mt19937_64 g(4711);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    long bad = 0;
    auto run = [&](double x, double eps) {
        int e;
        const double mf = frexp(x, &e);
        const double a = zbm::log_normal(mf, e, [&](double d) { return (1.0 + eps) / d; }, [](double c) { return c; });
        const double b = zbm::log_series(x);
        if (memcmp(&a, &b, sizeof a)) {
            if (++bad < 10) printf("x %a: %a, series %a\n", x, a, b);
        }
    };
    for (int i = 0; i < 3000000; ++i) {
        const double eps = (2.0 * u(g) - 1.0) * 0x1p-20;
        run(exp2(-1022.0 + 2046.0 * u(g)), eps);
        run(exp(log(30.0) + (log(1e5) - log(30.0)) * u(g)), eps);
        run(1.0 + (u(g) - 0.5) * 1e-3, eps);
        run(0x1.6a09e667f3bcdp+0 * (1.0 + (u(g) - 0.5) * 1e-6), eps);
    }
    for (double x : {1.0, 2.0, 0.5, 0x1.6a09e667f3bcdp+0, nextafter(1.0, 2.0), nextafter(1.0, 0.0),
                     0x1.6a09e667f3bccp+0, 0x1.6a09e667f3bcep+0, 0x1p-1022, 1.7976931348623157e308})
        for (double eps : {0.0, 0x1p-20, -0x1p-20}) run(x, eps);
    printf(bad ? "log_normal: %ld differ\n" : "log_normal ok\n", bad);
    return bad ? 1 : 0;
}
