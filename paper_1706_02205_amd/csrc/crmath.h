// Correctly rounded exponential and the Matern closed forms for gfx950.
//
// The factorization must start from bit-identical covariance entries for its
// results to be reproducible entry by entry, so exp is correctly rounded, in two
// phases (Ziv, ACM TOMS 17(3), 1991).  The first (exp_fast) reaches about 68 bits
// with a 256-entry table and some 30 FP64 operations and accepts its result
// when the error bound leaves the rounding no choice.  One argument in 2^13 goes
// on to the second (exp_full), about 100 bits in double-double arithmetic (some
// 300 operations), rounded once:
//   x = k ln2 + r            Cody-Waite reduction, ln2 split into three parts
//   r' = r / 2^8             exact
//   expm1(r') = r' + r'^2 P(r'),  P the Taylor series to degree 10 (double-double)
//   expm1(2s) = 2 expm1(s) + expm1(s)^2, eight times
//   exp(x) = 2^k (1 + expm1(r))
// The double-double result (hi, lo) is normalised, so hi is the correctly
// rounded value unless the true value lies within the evaluation error of a
// rounding midpoint; such cases are reported through `hard` (probability about
// 2^-40 per call).  Results below the normal range are rounded onto the
// subnormal grid with integer arithmetic so they are correctly rounded too.
#pragma once

#include <hip/hip_runtime.h>

#include "exp_table.h"

namespace kcdev {

struct dd {
    double hi, lo;
};

__device__ __forceinline__ dd two_sum(double a, double b) {
    double s = a + b;
    double bb = s - a;
    double e = (a - (s - bb)) + (b - bb);
    return {s, e};
}

__device__ __forceinline__ dd quick_two_sum(double a, double b) {  // |a| >= |b|
    double s = a + b;
    return {s, b - (s - a)};
}

__device__ __forceinline__ dd two_prod(double a, double b) {
    double p = a * b;
    return {p, __builtin_fma(a, b, -p)};
}

__device__ __forceinline__ dd dd_add(dd a, dd b) {
    dd s = two_sum(a.hi, b.hi);
    dd t = two_sum(a.lo, b.lo);
    s.lo += t.hi;
    s = quick_two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return quick_two_sum(s.hi, s.lo);
}

__device__ __forceinline__ dd dd_mul(dd a, dd b) {
    dd p = two_prod(a.hi, b.hi);
    p.lo = __builtin_fma(a.hi, b.lo, __builtin_fma(a.lo, b.hi, p.lo));
    return quick_two_sum(p.hi, p.lo);
}

// ln 2 = C1 + C2 + C3; C1 has 42 significant bits so k*C1 is exact for |k| < 2^11.
constexpr double kLn2C1 = 0x1.62e42fefa3800p-1;
constexpr double kLn2C2 = 0x1.ef35793c76730p-45;
constexpr double kLn2C3 = 0x1.f97b57a079a19p-103;
constexpr double kInvLn2 = 0x1.71547652b82fep+0;

__device__ __forceinline__ dd expm1_small(dd r) {
    // 1/n! for n = 2..10 as double-double
    const dd c[9] = {{0x1.0000000000000p-1, 0.0},
                     {0x1.5555555555555p-3, 0x1.5555555555555p-57},
                     {0x1.5555555555555p-5, 0x1.5555555555555p-59},
                     {0x1.1111111111111p-7, 0x1.1111111111111p-63},
                     {0x1.6c16c16c16c17p-10, -0x1.f49f49f49f49fp-65},
                     {0x1.a01a01a01a01ap-13, 0x1.a01a01a01a01ap-73},
                     {0x1.a01a01a01a01ap-16, 0x1.a01a01a01a01ap-76},
                     {0x1.71de3a556c734p-19, -0x1.c154f8ddc6c00p-73},
                     {0x1.27e4fb7789f5cp-22, 0x1.cbbc05b4fa99ap-76}};
    dd p = c[8];
#pragma unroll
    for (int i = 7; i >= 0; --i) p = dd_add(c[i], dd_mul(r, p));
    return dd_add(r, dd_mul(dd_mul(r, r), p));
}

// Whether hi is the rounding of every value within tol of hi + lo (|lo| <= ulp(hi)/2).
__device__ __forceinline__ bool rounding_certain(double hi, double lo, double tol) {
    const long long bits = __double_as_longlong(hi);
    const int ex = int((bits >> 52) & 0x7ff);
    const double ulp = __longlong_as_double((long long)(ex - 52) << 52);
    const bool pow2 = (bits & 0xfffffffffffffLL) == 0;
    const double half = (lo < 0.0 && pow2) ? 0.25 * ulp : 0.5 * ulp;
    return half - __builtin_fabs(lo) > tol;
}

// First phase, -700 < x <= 0: x = n ln2/256 + r with |r| <= ln2/512 (2^-9.5),
// n = 256 m + j, exp(x) = 2^m 2^(j/256) exp(r).  ln2/256 = D1 + D2 with 34 bits
// in D1, so n D1 and x - n D1 are exact and r = rh + rl is good to 2^-78.
// exp(r) - 1 = rh + (rl + rh^2 q(rh)), q the Taylor series through r^6/6!
// (truncation 2^-78); what is neglected or rounded there (rh rl, rh^2, q, the
// sum) is below 2^-71 together.  2^(j/256) = hi + lo from the table, and the
// products are carried in two doubles: the result is within 2^-69 relative.
constexpr double kLn2d256D1 = 0x1.62e42fef80000p-9;
constexpr double kLn2d256D2 = 0x1.1cf79abc9e3b4p-44;
constexpr double k256dLn2 = 0x1.71547652b82fep+8;

__device__ __forceinline__ bool exp_fast(double x, double& out) {
    const double kf = __builtin_rint(x * k256dLn2);
    const double t = __builtin_fma(-kf, kLn2d256D1, x);  // exact
    const dd p2 = two_prod(kf, kLn2d256D2);
    dd r = two_sum(t, -p2.hi);
    r.lo -= p2.lo;
    double q = __builtin_fma(r.hi, 1.0 / 720.0, 1.0 / 120.0);
    q = __builtin_fma(r.hi, q, 1.0 / 24.0);
    q = __builtin_fma(r.hi, q, 1.0 / 6.0);
    q = __builtin_fma(r.hi, q, 0.5);
    const dd e = quick_two_sum(r.hi, __builtin_fma(r.hi * r.hi, q, r.lo));  // exp(r) - 1
    const int n = int(kf);
    const ExpPair w = kExp2Table[n & 255];
    const dd me = two_prod(w.hi, e.hi);
    const dd h = quick_two_sum(w.hi, me.hi);
    const double lo = h.lo + (__builtin_fma(w.hi, e.lo, me.lo) + __builtin_fma(w.lo, e.hi, w.lo));
    const dd v = quick_two_sum(h.hi, lo);
    out = __builtin_ldexp(v.hi, n >> 8);  // above 2^-1011: normal
    return rounding_certain(v.hi, v.lo, v.hi * 0x1p-67);
}

// Second phase.  hard |= 1 when the rounding could not be certified.
__device__ inline double exp_full(double x, int& hard) {
    if (x != x) return x;
    if (x < -745.2) return 0.0;          // below half the smallest subnormal
    if (x > 709.79) return __builtin_inf();
    double kd = __builtin_rint(x * kInvLn2);
    int k = int(kd);
    double t1 = x - kd * kLn2C1;         // exact
    dd p2 = two_prod(kd, kLn2C2);
    dd r = two_sum(t1, -p2.hi);
    r.lo = (r.lo - p2.lo) - kd * kLn2C3;
    r = quick_two_sum(r.hi, r.lo);
    r.hi *= 0x1p-8;
    r.lo *= 0x1p-8;
    dd e = expm1_small(r);
#pragma unroll
    for (int i = 0; i < 8; ++i) {        // expm1(2s) = 2 expm1(s) + expm1(s)^2
        dd e2 = dd_mul(e, e);
        e = dd_add({2.0 * e.hi, 2.0 * e.lo}, e2);
    }
    dd v = dd_add({1.0, 0.0}, e);        // exp(r), normalised: |lo| <= ulp(hi)/2
    if (k >= -1021) {  // 2^k * [0.7, 1.42] is a normal number: the scaling is exact
        if (!rounding_certain(v.hi, v.lo, v.hi * 0x1p-92)) hard = 1;
        return __builtin_ldexp(v.hi, k);
    }
    // result below 2^-1021 * 1.42: round (hi + lo) * 2^(k+1074) to an integer number
    // of 2^-1074 (the spacing of subnormals and of normals below 2^-1021; z < 2^53)
    int s = k + 1074;
    double z = __builtin_ldexp(v.hi, s);
    double zl = __builtin_ldexp(v.lo, s);
    double nn = __builtin_rint(z);
    dd h = two_sum(z - nn, zl);
    if (h.hi > 0.5 || (h.hi == 0.5 && h.lo > 0.0)) nn += 1.0;
    else if (h.hi < -0.5 || (h.hi == -0.5 && h.lo < 0.0)) nn -= 1.0;
    else if (h.hi == 0.5 && h.lo == 0.0) nn = (__builtin_fmod(nn, 2.0) == 0.0) ? nn : nn + 1.0;
    else if (h.hi == -0.5 && h.lo == 0.0) nn = (__builtin_fmod(nn, 2.0) == 0.0) ? nn : nn - 1.0;
    if (__builtin_fabs(__builtin_fabs(h.hi) - 0.5) < 0x1p-40) hard = 1;
    return nn * 0x1p-1074;
}

// Correctly rounded exp(x).
__device__ __forceinline__ double cr_exp(double x, int& hard) {
    double v;
    if (x > -700.0 && x <= 0.0 && exp_fast(x, v)) return v;
    return exp_full(x, hard);
}

// Euclidean distance, coordinates summed in ascending order without fusion
// (the library is compiled with -ffp-contract=off).  Past three coordinates they
// are requested four at a time: the loop of one load, then its use, waited for
// memory d times over.
__device__ __forceinline__ double dist(const double* __restrict__ a, const double* __restrict__ b, int d) {
    double s = 0.0;
    int t = 0;
    for (; t + 4 <= d; t += 4) {
        double x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = a[t + u];
            y[u] = b[t + u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double df = x[u] - y[u];
            s = s + df * df;
        }
    }
    for (; t < d; ++t) {
        const double df = a[t] - b[t];
        s = s + df * df;
    }
    return __builtin_sqrt(s);
}

// Matern covariance with unit variance at nu = TWONU/2 (Section 4.4 closed forms).
template <int TWONU>
__device__ __forceinline__ double matern(double r, double ell, int& hard) {
    if constexpr (TWONU == 1) {
        double a = r / ell;
        return cr_exp(-a, hard);
    } else if constexpr (TWONU == 3) {
        double a = (0x1.bb67ae8584caap+0 * r) / ell;  // sqrt(3), correctly rounded
        return (1.0 + a) * cr_exp(-a, hard);
    } else {
        double a = (0x1.1e3779b97f4a8p+1 * r) / ell;  // sqrt(5), correctly rounded
        return ((1.0 + a) + (a * a) / 3.0) * cr_exp(-a, hard);
    }
}

// FP32 Matern for the mixed-precision factorization.
template <int TWONU>
__device__ __forceinline__ float matern_f32(float r, float ell) {
    if constexpr (TWONU == 1) {
        return expf(-(r / ell));
    } else if constexpr (TWONU == 3) {
        float a = (1.7320508f * r) / ell;
        return (1.0f + a) * expf(-a);
    } else {
        float a = (2.2360680f * r) / ell;
        return ((1.0f + a) + (a * a) * (1.0f / 3.0f)) * expf(-a);
    }
}

}  // namespace kcdev
