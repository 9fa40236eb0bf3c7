// rt_planck.hpp -- FP64 Planck edge integrals from a small table.
//
// planck_edge<double> (rt_physics.hpp) sums up to 28 terms below x = 3 and up to 52
// above it, each term an FMA and two scalar instructions that build its coefficient:
// about 100 vector and 170 scalar instructions per (level, bin) of the solve, a
// third of a wavefront's issue.  Here the integral is one polynomial of degree 11
// in the cell of x, its coefficients gathered from a table of 2.6 KB in LDS:
//   x < 3:  Q(x) / x^3 = 1/3 - x/8 + sum_k B_2k x^2k / ((2k+3)(2k)!)
//   x >= 3: P(x) e^x, which is x^3 + 3x^2 + 6x + 6 and terms that fall like e^-x
// Cells: [0, 1), then four per octave up to 64 (the leading bits of x), beyond which
// the cubic alone is left.  Both functions are analytic up to x = +-2 pi i, at least 7
// (x < 3: 6.4) from a cell's centre and 13 (x < 1: 12) of its half-widths where the
// terms in e^-x matter, so interpolation at the Chebyshev nodes of a cell is off by
// less than one unit of roundoff (checked against quadruple precision: 4e-16 of the
// integral with the evaluation's own rounding, 7e-16 for the series above).
// (A table of 256 cells of degree 8 for P itself, in memory, needs no exponential,
// but its gathers took 825 cycles per 64 edges of a wavefront against 650 here.)
#pragma once

#include "rt_internal.hpp"
#include "rt_math.hpp"
#include "rt_physics.hpp"

#include <math.h>

namespace rtk {

constexpr int kPlanckCells = 25, kPlanckCoefs = 12;
constexpr int kPlanckSplit = 7;                          // the first cell above x = 3
constexpr int kExpCells = 32;                            // 2^(-j/32), j = 0 .. 31, after the cells
constexpr int kPlanckTable = kPlanckCells * kPlanckCoefs + kExpCells;   // doubles

// Cell of x >= 0: its index (past the last cell: too large) and its centre.
__host__ __device__ __forceinline__ int planck_cell(double x, double &centre)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const int hi = __double2hiint(x);
    centre = __hiloint2double((hi & 0x7ffc0000) | 0x20000, 0);
#else
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const int hi = (int)(u >> 32);
    centre = __builtin_bit_cast(double, (uint64_t)(uint32_t)((hi & 0x7ffc0000) | 0x20000) << 32);
#endif
    const int k = (hi >> 18) - 1023 * 4 + 1;
    if (k <= 0) centre = 0.5;
    return k > 0 ? k : 0;
}

// zeta(s), s >= 2 even, by Euler-Maclaurin summation from M on
inline long double planck_zeta(int s)
{
    constexpr int M = 32;
    long double sum = 0.0L;
    for (int n = M - 1; n >= 1; --n) sum += powl(1.0L / n, s);
    const long double Mi = 1.0L / M, Ms = powl(Mi, s), ds = s;
    long double term = Ms, r = Ms * M / (ds - 1.0L) + 0.5L * Ms;
    // B_2j / (2j)! s (s+1) .. (s+2j-2) / M^(s+2j-1)
    const long double b[] = {1.0L / 12, -1.0L / 720, 1.0L / 30240, -1.0L / 1209600, 1.0L / 47900160};
    long double rise = ds;
    for (int j = 0; j < 5; ++j) {
        term *= j == 0 ? Mi : Mi * Mi;
        r += b[j] * rise * term;
        rise *= (ds + 2 * j + 1) * (ds + 2 * j + 2);
    }
    return sum + r;
}

// Coefficients of every cell's polynomial in x - centre, and the powers of two.
inline void planck_table(double *out)
{
    const long double pi = 3.14159265358979323846264338327950288L;
    constexpr int NT = 34, n = kPlanckCoefs;
    long double c[NT];   // B_2k / ((2k+3) (2k)!)
    for (int k = 1; k < NT; ++k)
        c[k] = (k % 2 ? 2.0L : -2.0L) * planck_zeta(2 * k) / (powl(2.0L * pi, 2 * k) * (2 * k + 3));
    auto value = [&](int k, long double x) -> long double {
        if (k < kPlanckSplit) {
            long double s = 0.0L;
            for (int j = NT - 1; j >= 1; --j) s = (s + c[j]) * x * x;
            return 1.0L / 3 - x / 8 + s;
        }
        long double s = 0.0L;
        for (int m = 20; m >= 1; --m) {
            const long double i = 1.0L / m;
            s += expl((1 - m) * x) * (x * x * x * i + 3 * x * x * i * i + 6 * x * i * i * i + 6 * i * i * i * i);
        }
        return s;
    };
    for (int k = 0; k < kPlanckCells; ++k) {
        const double x0 = k == 0 ? 0.0 : ldexp(1.0 + 0.25 * ((k - 1) % 4), (k - 1) / 4);
        const double width = k == 0 ? 1.0 : ldexp(0.25, (k - 1) / 4);
        const long double half = 0.5L * width, mid = x0 + half;
        long double a[n] = {};   // Chebyshev coefficients in s = (x - centre) / half
        for (int i = 0; i < n; ++i) {
            const long double th = pi * (i + 0.5L) / n;
            const long double f = value(k, mid + half * cosl(th));
            for (int m = 0; m < n; ++m) a[m] += f * cosl(m * th) * (m ? 2.0L : 1.0L) / n;
        }
        long double p[n] = {}, t0[n] = {1.0L}, t1[n] = {0.0L, 1.0L};   // powers of s; T_m-1, T_m
        p[0] = a[0];
        for (int m = 1; m < n; ++m) {
            for (int j = 0; j < n; ++j) p[j] += a[m] * t1[j];
            long double t2[n];
            for (int j = 0; j < n; ++j) t2[j] = (j ? 2 * t1[j - 1] : 0.0L) - t0[j];
            for (int j = 0; j < n; ++j) t0[j] = t1[j], t1[j] = t2[j];
        }
        long double scale = 1.0L;
        for (int j = 0; j < n; ++j, scale /= half) out[k * n + j] = double(p[j] * scale);
    }
    for (int j = 0; j < kExpCells; ++j) out[kPlanckCells * n + j] = double(exp2l(-(long double)j / kExpCells));
}

struct ExpCoef6 {
    static constexpr double coef(int j) { return inv_fact(j + 1); }
};

// e^-x, 0 <= x <= 800 (from 746 on 0): x = k ln2 / 32 + r, |r| <= ln2 / 64, from the table's 2^(-j/32), j = k
// mod 32, and the Taylor polynomial of e^-r - 1 (next term below 4e-18).
__host__ __device__ __forceinline__ double exp_neg(double x, const double *table)
{
    constexpr double M = 6755399441055744.0;   // 1.5 x 2^52: x + M holds rint(x) in its low bits
    const double m = fma(x, 32.0 * ExpCfg<double>::LOG2E, M), k = m - M;
    double r = fma(k, -ExpCfg<double>::LN2_HI / 32.0, x);
    r = fma(k, -ExpCfg<double>::LN2_LO / 32.0, r);
#if defined(__HIP_DEVICE_COMPILE__)
    const int ki = __double2loint(m);
#else
    const int ki = (int)(uint32_t)__builtin_bit_cast(uint64_t, m);
#endif
    const double T = table[kPlanckCells * kPlanckCoefs + (ki & (kExpCells - 1))];
    const double q = -r * horner_s<ExpCoef6, 0, 6>(-r, opaque_zero());
    return ldexp(fma(T, q, T), -(ki >> 5));
}

// The integral at x: Q(x) below x = 3, -P(x) above (planck_edge's values and sign
// convention; -0 for NaN and x beyond every exponent).  No branch: the lanes of a
// wavefront fall on both sides of x = 3, and two calls overlap.  table: 16-byte aligned.
__host__ __device__ __forceinline__ double planck_lookup(double x, const double *table)
{
    x = fmin(x, 800.0);   // (and NaN: e^-800 is 0)
    double c;
    const int k = planck_cell(x, c), kc = k < kPlanckCells ? k : kPlanckCells - 1;
    const double t = x - c;
    struct alignas(16) Pair {
        double a, b;
    };
    const Pair *p = reinterpret_cast<const Pair *>(table + kc * kPlanckCoefs);
    double s = p[5].b;
    s = fma(s, t, p[5].a);
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
    for (int j = 4; j >= 0; --j) {
        s = fma(s, t, p[j].b);
        s = fma(s, t, p[j].a);
    }
    s = k >= kPlanckCells ? fma(x, fma(x, x + 3.0, 6.0), 6.0) : s;
    const double f = k < kPlanckSplit ? x * x * x : -exp_neg(x, table);
    return f * s;
}

}  // namespace rtk
