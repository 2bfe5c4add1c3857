// Compact FP64 elementary functions for the fluctuation/dissipation update
// and the particle passes (square roots).
//
// Their arguments are always positive, finite and well ranged (uniform draws
// in (0, 1), energies, ratios of friction amplitudes, squared distances
// below h^2; a zero distance is handled by the caller), so the special-case
// handling of a general math library is not needed.  Accuracy: a few ulp,
// far below the 1e-10 agreement required with the FP64 oracle.
//   * log: x = m 2^e with m in [sqrt(1/2), sqrt(2)), ln m = 2 atanh(f),
//     f = (m - 1)/(m + 1), |f| <= 0.1716, atanh series to f^23;
//     e ln 2 added with a two-part ln 2 (32-bit head, so e * head is exact).
//   * log1p: log(1 + x) plus the exact rounding error of 1 + x divided by
//     1 + x (the error is recovered with the Fast2Sum step).
//   * sin(pi t), cos(pi t): t reduced by multiples of 1/2 to |r| <= 1/4,
//     Taylor polynomials of sin(pi r) and cos(pi r) to degree 19 / 18, then a
//     quarter-turn rotation.
//   * reciprocal, reciprocal square root and square root: the hardware
//     estimate (relative error below 6e-8) and one second-order correction.
//   * expm1: x = k ln 2 + r with |r| <= ln 2 / 2 (two-part ln 2), the Taylor
//     polynomial of expm1(r) to degree 13 (its tail is below 2^-53 |r|), and
//     expm1(x) = 2^k expm1(r) + (2^k - 1) in one fused step; for |x| <= ln 2 / 2
//     k = 0 and the polynomial alone is the result.  When no active lane of
//     a wave has |x| > 2^-5 the wave takes the Taylor polynomial of expm1(x)
//     to degree 8 instead.
// Every function with more than a few coefficients takes them from a table t
// (any pointer to double): the device code passes tables in constant memory
// (fd_math.hpp), the plain forms fd_* the same coefficients as literals.
#pragma once

// expm1: 1/13! ... 1/3!, 1/2; log2 e, ln 2 in two parts
#define SDPD_EXPM1_COEF                                                                       \
    1.6059043836821613e-10, 2.08767569878681e-09, 2.505210838544172e-08,                      \
        2.755731922398589e-07, 2.7557319223985893e-06, 2.48015873015873e-05,                  \
        0.0001984126984126984, 0.001388888888888889, 0.008333333333333333,                    \
        0.041666666666666664, 0.16666666666666666, 0.5, 1.4426950408889634,                   \
        0.6931471803691238, 1.9082149292705877e-10
// log: 2/23, 2/21, ... 2/3; sqrt(1/2), ln 2 in two parts
#define SDPD_LOG_COEF                                                                         \
    0.08695652173913043, 0.09523809523809523, 0.10526315789473684, 0.11764705882352941,       \
        0.13333333333333333, 0.15384615384615385, 0.18181818181818182, 0.2222222222222222,    \
        0.2857142857142857, 0.4, 0.6666666666666666, 0.7071067811865476, 0.6931471803691238,  \
        1.9082149292705877e-10
// sin(pi r)/r in r^2 (r^21 down to r^1), then cos(pi r) in r^2 (r^18 down to r^2)
#define SDPD_SINCOS_COEF                                                                      \
    5.392664662608129e-10, -2.2948428997269873e-08, 7.952054001475513e-07,                    \
        -2.1915353447830217e-05, 0.00046630280576761255, -0.0073704309457143504,              \
        0.08214588661112823, -0.5992645293207921, 2.5501640398773455, -5.16771278004997,      \
        3.141592653589793, -1.3878952462213771e-07, 4.303069587032947e-06,                    \
        -0.0001046381049248457, 0.0019295743094039231, -0.02580689139001406,                  \
        0.2353306303588932, -1.3352627688545895, 4.0587121264167685, -4.934802200544679

namespace sdpd {

// reciprocal to about one ulp: the hardware estimate r (relative error
// below 5e-8 on gfx950) and one second-order step, r (1 + e + e^2) with
// e = 1 - x r, whose own error is e^3 (three dependent operations where two
// Newton steps take four)
__device__ __forceinline__ double fast_rcp(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// reciprocal square root to about one ulp: the hardware estimate y and one
// second-order step, y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2 (error of order
// e^3)
__device__ __forceinline__ double fast_rsq(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// sqrt(x) as x / sqrt(x) from the reciprocal square root alone (within
// about two ulp); the host check of these functions holds it beside fd_sqrt
__device__ __forceinline__ double fd_sqrt_pair(double x) { return x * fast_rsq(x); }

// sqrt(x) from the estimate y and s = x y: with r = (1 - s y)/2, measured on
// the rounded s, sqrt(x) = s (1 + r + 3 r^2/2) to order r^3, below one ulp
// (half of the rounding of s remains)
__device__ __forceinline__ double fd_sqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double s = x * y;
    const double r = fma(-s, 0.5 * y, 0.5);
    return fma(s, r * fma(1.5, r, 1.0), s);
}

constexpr double kExpm1Coef[15] = {SDPD_EXPM1_COEF};
constexpr double kLogCoef[14] = {SDPD_LOG_COEF};
constexpr double kSinCosCoef[20] = {SDPD_SINCOS_COEF};

// expm1(x) for finite x with |x| < 700 (t: the expm1 table)
template <class T>
__device__ __forceinline__ double elem_expm1(double x, T t)
{
    const double k = rint(x * t[12]);
    const double r = fma(-k, t[14], fma(-k, t[13], x));
    double p = t[0];
#pragma unroll
    for (int i = 1; i < 12; ++i) p = fma(p, r, t[i]);
    p = fma(p * r, r, r);                  // r + r^2 (1/2 + r/6 + ...)
    const double s = ldexp(1.0, (int)k);
    return fma(s, p, s - 1.0);
}
__device__ __forceinline__ double fd_expm1(double x) { return elem_expm1(x, kExpm1Coef); }

// expm1(x) for |x| <= 2^-5: its Taylor polynomial to x^8 (the first term
// left out, x^9/9!, is below 2^-58 |x| there)
template <class T>
__device__ __forceinline__ double elem_expm1_small(double x, T t)
{
    double p = t[5];                       // 1/8!
#pragma unroll
    for (int i = 6; i < 12; ++i) p = fma(p, x, t[i]);
    return fma(p * x, x, x);               // x + x^2 (1/2 + x/6 + ...)
}
__device__ __forceinline__ double fd_expm1_small(double x)
{
    return elem_expm1_small(x, kExpm1Coef);
}

// expm1 with the short form when no active lane of the wave has |x| > 2^-5
// (the friction exponents of a step of ordinary size), else in full; the table
// of the full form is asked for only where it runs
template <class T, class Full>
__device__ __forceinline__ double elem_expm1_wave(double x, T t, Full full)
{
    if (__ballot(fabs(x) > 0x1p-5) == 0ull) return elem_expm1_small(x, t);
    return elem_expm1(x, full());
}
__device__ __forceinline__ double fd_expm1_wave(double x)
{
    return elem_expm1_wave(x, kExpm1Coef, [] { return kExpm1Coef; });
}

// log(x) (t: the log table)
template <class T>
__device__ __forceinline__ double elem_log(double x, T t)
{
    int e;
    double m = frexp(x, &e);   // m in [0.5, 1)
    const bool low = m < t[11];
    m = low ? 2.0 * m : m;
    e = low ? e - 1 : e;
    const double f = (m - 1.0) * fast_rcp(m + 1.0);
    const double s = f * f;
    // 2 atanh(f) = 2 f + f s (2/3 + 2/5 s + 2/7 s^2 + ... + 2/23 s^10)
    double p = t[0];
#pragma unroll
    for (int i = 1; i < 11; ++i) p = fma(p, s, t[i]);
    const double de = (double)e;
    return fma(de, t[12], fma(de, t[13], fma(f * s, p, 2.0 * f)));
}
__device__ __forceinline__ double fd_log(double x) { return elem_log(x, kLogCoef); }

// log(1 + x) for x > -1
template <class T>
__device__ __forceinline__ double elem_log1p(double x, T t)
{
    const double y = 1.0 + x;
    const double c = fabs(x) < 1.0 ? x - (y - 1.0) : 1.0 - (y - x);
    return elem_log(y, t) + c * fast_rcp(y);
}
__device__ __forceinline__ double fd_log1p(double x) { return elem_log1p(x, kLogCoef); }

// sin(pi a), cos(pi a) for 0 <= a <= 2 (t: the sine and cosine table)
template <class T>
__device__ __forceinline__ void elem_sincospi(double a, double &s, double &c, T t)
{
    const double k = rint(2.0 * a);   // quarter turns, 0..4
    const double r = a - 0.5 * k;     // exact, |r| <= 1/4
    const double z = r * r;
    double ps = t[1], pc = t[11];
#pragma unroll
    for (int i = 2; i < 11; ++i) ps = fma(ps, z, t[i]);
#pragma unroll
    for (int i = 12; i < 20; ++i) pc = fma(pc, z, t[i]);
    const double sr = r * ps, cr = fma(pc, z, 1.0);
    // quarter-turn rotation as selects (no branches): odd q swaps sin and
    // cos; sin changes sign for q = 2, 3 and cos for q = 1, 2
    const int q = ((int)k) & 3;
    const bool sw = (q & 1) != 0;
    const double u = sw ? cr : sr, v = sw ? sr : cr;
    s = (q & 2) ? -u : u;
    c = ((q + 1) & 2) ? -v : v;
}
__device__ __forceinline__ void fd_sincospi(double t, double &s, double &c)
{
    elem_sincospi(t, s, c, kSinCosCoef);
}

// cos(pi a) alone for 0 <= a <= 2, as sin(pi r) with r = 1/2 - a or a - 3/2 in
// [-1/2, 1/2] (exact for multiples of 2^-32): one polynomial, the Taylor series
// of sin(pi r) to r^21 (tail below 2^-59), instead of the two that the
// quarter-turn form selects from
template <class T>
__device__ __forceinline__ double elem_cospi(double a, T t)
{
    const double r = a <= 1.0 ? 0.5 - a : a - 1.5;
    const double z = r * r;
    double p = t[0];
#pragma unroll
    for (int i = 1; i < 11; ++i) p = fma(p, z, t[i]);
    return r * p;
}
__device__ __forceinline__ double fd_cospi(double a) { return elem_cospi(a, kSinCosCoef); }

}  // namespace sdpd
