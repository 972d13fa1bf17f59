// CPU test of div_small (zb_stepmath.h): the quotient by 2..7 bit by bit the division's, over the
// norms a step can have (down to 2^-900, where the remainder is still exact), and the special
// values.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <random>

#include "zb_stepmath.h"

int main()
{
    std::mt19937_64 g(99);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    long bad = 0;
    auto run = [&](double x) {
        for (int d = 2; d <= 7; ++d) {
            const double a = zbm::div_small(x, (double)d, 1.0 / (double)d), b = x / (double)d;
            if (memcmp(&a, &b, sizeof a) && !(isnan(a) && isnan(b))) {
                if (++bad < 10) printf("%a / %d: %a, %a\n", x, d, a, b);
            }
        }
    };
    for (int i = 0; i < 3000000; ++i) {
        run(exp2(-900.0 + 1923.0 * u(g)));
        run(exp2(-40.0 + 80.0 * u(g)));
    }
    for (double x : {0.0, 1.0, 3.0, 7.0, (double)INFINITY, (double)NAN, 1.7976931348623157e308}) run(x);
    printf(bad ? "div_small: %ld differ\n" : "div_small ok\n", bad);
    return bad ? 1 : 0;
}
