// Host check of log_by_table (paper_2106_05373_amd/csrc/fp64_log.h) against the C library's long
// double log: at most 1.5 units in the last place of the result (half of one for the last sum, and
// half of one of log(1 + r), at most twice the result, for the sum before it; the rest is exact or
// below 2^-58), near one and on every cell's edges included.
#include <stdint.h>
#include <stdio.h>

#include <cmath>

#include "fp64_log.h"

int main() {
    static constexpr bcpnn::LogTable table = bcpnn::log_table();
    const bcpnn::LogCell* cells = table.cell;
    uint64_t st = 88172645463325252ull;
    double worst = 0.0, wx = 0.0;
    auto check = [&](double x) {
        const long double want = logl((long double)x);
        const double got = bcpnn::log_by_table(x, cells);
        const double ulp = std::nextafter(std::fabs((double)want), 1e300) - std::fabs((double)want);
        const double off = want == 0.0L ? (got == 0.0 ? 0.0 : 1e9) : (double)(fabsl(got - want) / ulp);
        if (off > worst) { worst = off; wx = x; }
    };
    for (int it = 0; it < 6000000; ++it) {
        st ^= st << 13;
        st ^= st >> 7;
        st ^= st << 17;
        const double u = (double)(st >> 11) * 0x1p-53;
        check(it % 4 == 0 ? std::exp(-40.0 + 80.0 * u) : it % 4 == 1 ? 1.0 + (u - 0.5) * 1e-3
              : it % 4 == 2 ? 1.0 + (u - 0.5) * 1e-8 : 0.5 + 1.5 * u);
    }
    for (int e = -130; e <= 130; ++e)
        for (int q = 0; q < bcpnn::kLogCells; ++q) {
            const double edge = std::ldexp(1.0 + q / (double)bcpnn::kLogCells, e);
            check(edge);
            check(std::nextafter(edge, 0.0));
            check(std::nextafter(edge, 1e300));
        }
    printf("max error %.3f ulp (x = %.17g)\n", worst, wx);
    return worst <= 1.5 ? 0 : 1;
}
