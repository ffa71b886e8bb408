// Natural logarithm of a positive normal double, about one ulp from the correctly rounded value
// (host and device, so that a host test can check it against the C library); the kernel takes the
// table form further down, and this one stays as the form without a table.  The method is the
// argument reduction and s = f / (2 + f) form of the public-domain fdlibm e_log.c (Sun
// Microsystems, 1993), with its split of ln 2 into a 32-bit head and a tail; the polynomial here
// is the plain atanh Taylor series, not fdlibm's minimax coefficients.
//
// x = 2^k m with m in [sqrt(1/2), sqrt(2)) and f = m - 1.  With s = f / (2 + f),
//   log(1 + f) = log((1 + s) / (1 - s)) = 2 atanh(s) = 2 s + s R(z),   z = s^2,
// R(z) = sum_{n >= 1} 2 z^n / (2n + 1) (the Taylor series of atanh; |s| <= 0.172 so ten terms
// leave a remainder below 2^-56 of the result), and 2 s = f - s f = f - h + s h with h = f^2 / 2,
// so log(1 + f) = f - (h - s (h + R)): the large terms f and h are exact or nearly so and the
// rounding of the small correction s (h + R) hardly matters.  k ln 2 is added as
// k * ln2_hi + k * ln2_lo with ln2_hi carrying 32 significant bits (exact for |k| < 2^21).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace bcpnn {

__host__ __device__ inline double log_positive(double x) {
    constexpr double kLn2Hi = 0x1.62e42fee00000p-1;    // ln 2 to 32 bits
    constexpr double kLn2Lo = 0x1.a39ef35793c76p-33;   // ln 2 - kLn2Hi
    int e;
    double m = frexp(x, &e);                            // [1/2, 1)
    if (m < 0.70710678118654752440) {
        m *= 2.0;
        e -= 1;
    }
    const double f = m - 1.0;
    const double s = f / (2.0 + f);
    const double z = s * s;
    double r = 2.0 / 23;
    r = fma(r, z, 2.0 / 21);
    r = fma(r, z, 2.0 / 19);
    r = fma(r, z, 2.0 / 17);
    r = fma(r, z, 2.0 / 15);
    r = fma(r, z, 2.0 / 13);
    r = fma(r, z, 2.0 / 11);
    r = fma(r, z, 2.0 / 9);
    r = fma(r, z, 2.0 / 7);
    r = fma(r, z, 2.0 / 5);
    r = fma(r, z, 2.0 / 3);
    r *= z;
    const double h = 0.5 * f * f;
    const double k = (double)e;
    return k * kLn2Hi - ((h - fma(s, h + r, k * kLn2Lo)) - f);
}

// The same logarithm from a table, for kernels that take many: no division and 14 fp64
// instructions.  x = 2^k m with m in [1, 2), cell q = the top seven mantissa bits of m; with the
// cell's c (a short reciprocal of its middle) r = m c - 1 is small (|r| <= 2^-7) and exact to
// 2^-61, and
//   log x = k ln 2 - log c + log(1 + r),   log(1 + r) = r + r^2 (-1/2 + r/3 - ... - r^6/8)
// (the alternating series of log(1 + r); its remainder r^9/9 is below 2^-58 of the result).
// Cells from 53 on (m >= sqrt 2) count as 2^(k+1) (m / 2), so that x near 1 takes k = 0 on both
// sides, and the cells at both ends have c = 1 and 1/2: there -log c is 0 and log x = log(1 + r)
// without cancellation.  -log c has two parts, of which the first is a multiple of 2^-40, as k ln 2
// (first part) is of 2^-32: their sum is exact, so that only the last two sums round, at most half
// an ulp of the result and half an ulp of log(1 + r), which is at most twice the result: 1.5 ulp
// (measured: 0.83).
struct LogCell {
    double c, log_hi, log_lo;                           // c and -log c (less ln 2 for q >= 53)
};
constexpr int kLogCells = 128;
constexpr int kLogFold = 53;
struct LogTable {
    LogCell cell[kLogCells];
};

// -log(n / d) in fixed point, for n / d in (0.7, 1.42): -2 atanh(s) with s = (n - d) / (n + d).
constexpr __int128 kLogOne = (__int128)1 << 80;
constexpr __int128 minus_log_ratio(int64_t n, int64_t d) {
    const int64_t num = n - d, den = n + d;
    __int128 power = kLogOne * num / den, sum = 0;
    for (int j = 1; j < 41; j += 2) {
        sum += power / j;
        power = power * (num * num) / (den * den);
    }
    return -2 * sum;
}

constexpr LogTable log_table() {
    LogTable t{};
    t.cell[0] = LogCell{1.0, 0.0, 0.0};
    t.cell[kLogCells - 1] = LogCell{0.5, 0.0, 0.0};
    for (int q = 1; q < kLogCells - 1; ++q) {
        // c = n / 2048 nearest to 1 / (1 + (q + 1/2) / 128): 11 bits, so m c is exact but for 2^-63
        const int64_t n = (2048 * 256 + (257 + 2 * q) / 2) / (257 + 2 * q);
        const __int128 v = minus_log_ratio(n, q >= kLogFold ? 1024 : 2048);
        const __int128 hi = v >> 40;                    // in units of 2^-40 (rounded down)
        t.cell[q].c = (double)n / 2048.0;
        t.cell[q].log_hi = (double)(int64_t)hi * 0x1p-40;
        t.cell[q].log_lo = (double)(int64_t)(v - hi * ((int64_t)1 << 40)) * 0x1p-80;
    }
    return t;
}

__host__ __device__ inline double log_by_table(double x, const LogCell* cells) {
    constexpr double kLn2Hi = 0x1.62e42fee00000p-1;
    constexpr double kLn2Lo = 0x1.a39ef35793c76p-33;
    const uint64_t bits = __builtin_bit_cast(uint64_t, x);
    const uint32_t hi = (uint32_t)(bits >> 32);
    const LogCell cell = cells[(hi >> 13) & (kLogCells - 1)];
    const double k = (double)((int32_t)((hi + ((kLogCells - kLogFold) << 13)) >> 20) - 1023);
    const double m = __builtin_bit_cast(
        double, ((uint64_t)((hi & 0x000fffffu) | 0x3ff00000u) << 32) | (bits & 0xffffffffu));
    const double r = fma(m, cell.c, -1.0);
    double p = -1.0 / 8;
    p = fma(p, r, 1.0 / 7);
    p = fma(p, r, -1.0 / 6);
    p = fma(p, r, 1.0 / 5);
    p = fma(p, r, -1.0 / 4);
    p = fma(p, r, 1.0 / 3);
    p = fma(p, r, -1.0 / 2);
    const double head = fma(k, kLn2Hi, cell.log_hi);
    return head + (r + fma(r * r, p, fma(k, kLn2Lo, cell.log_lo)));
}

}  // namespace bcpnn
