// FP64 template math, one source for the host calls and the device kernel:
// the predicted normalised Fourier response of a constant-fdot signal
// (Sec. 2, text before eq. 23; eq. 22 defines z as the number of bins
// drifted over the observation).
//
//   R(q, z) = int_0^1 exp(i 2 pi [q u + z (u^2 - u)/2]) du,  q = r - k.
//
// Evaluated through the Fresnel auxiliary function G(x) = g(x) + i f(x),
// defined by  C(x) + i S(x) = (1+i)/2 - G(x) exp(i pi x^2 / 2)  for x >= 0,
// which makes the closed form free of large phases and of the cancellation
// of the Fresnel integrals' 1/2 limits.  With q' = q - z/2, s = sqrt(2/z),
// x1 = s q', x2 = s (q' + z) and  exp(i pi (x2^2 - x1^2)/2) = exp(i 2 pi q):
//   x1 >= 0      : R = (G(x1) - e^{i2 pi q} G(x2)) / sqrt(2z)
//   x2 <= 0      : R = (e^{i2 pi q} G(-x2) - G(-x1)) / sqrt(2z)
//   x1 < 0 < x2  : R = ((1+i) e^{-i pi q'^2/z} - e^{i2 pi q} G(x2) - G(-x1)) / sqrt(2z)
// and R(q, z) = conj R(-q, -z) for z < 0,  R(q, 0) = (e^{i2 pi q} - 1)/(i 2 pi q).
//
// G itself: for x <= 2 from the power series
//   C(x) + i S(x) = sum_k (i pi/2)^k x^{2k+1} / (k! (2k+1)),
// and for x > 2 from G(x) = (1+i)/2 * erfcx(w), w = (sqrt(pi)/2)(1-i) x,
// with erfcx evaluated by the Laplace continued fraction (DLMF 7.9.3)
//   sqrt(pi) erfcx(w) = 2w / (2w^2+1 - 1*2/(2w^2+5 - 3*4/(2w^2+9 - ...))).
//
// Everything is written with IEEE operations alone (+, -, *, /, sqrt, rint;
// the library is built without FMA contraction), the trigonometry included,
// so the device's templates equal the host's bit for bit.
#pragma once

#include <cmath>

#include <hip/hip_runtime.h>

namespace fdas {

struct cplx64 {
    double re, im;
};

__host__ __device__ inline cplx64 operator+(cplx64 a, cplx64 b) { return {a.re + b.re, a.im + b.im}; }
__host__ __device__ inline cplx64 operator-(cplx64 a, cplx64 b) { return {a.re - b.re, a.im - b.im}; }
__host__ __device__ inline cplx64 operator*(cplx64 a, cplx64 b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__host__ __device__ inline cplx64 operator*(cplx64 a, double s) { return {a.re * s, a.im * s}; }

constexpr double kPi64 = 3.14159265358979323846264338327950288;

// exp(i pi t): the nearest multiple of 1/2 is taken off exactly, the rest
// (|pi y| <= pi/4) goes through the Taylor series of sine and cosine.
__host__ __device__ inline cplx64 cis_pi(double t)
{
    const double r = t - 2.0 * rint(0.5 * t);      // [-1, 1], exact
    const double n = rint(2.0 * r);                // -2 .. 2
    const double y = kPi64 * (r - 0.5 * n);
    const double y2 = y * y;
    // 1/19! .. 1/3! and 1/18! .. 1/2!, alternating signs folded into y2
    double s = -1.0 / 121645100408832000.0;
    s = s * y2 + 1.0 / 355687428096000.0;
    s = s * y2 - 1.0 / 1307674368000.0;
    s = s * y2 + 1.0 / 6227020800.0;
    s = s * y2 - 1.0 / 39916800.0;
    s = s * y2 + 1.0 / 362880.0;
    s = s * y2 - 1.0 / 5040.0;
    s = s * y2 + 1.0 / 120.0;
    s = s * y2 - 1.0 / 6.0;
    s = y + y * (y2 * s);
    double c = -1.0 / 6402373705728000.0;
    c = c * y2 + 1.0 / 20922789888000.0;
    c = c * y2 - 1.0 / 87178291200.0;
    c = c * y2 + 1.0 / 479001600.0;
    c = c * y2 - 1.0 / 3628800.0;
    c = c * y2 + 1.0 / 40320.0;
    c = c * y2 - 1.0 / 720.0;
    c = c * y2 + 1.0 / 24.0;
    c = 1.0 - y2 * (0.5 - y2 * c);
    const int k = (int)n & 3;                      // quarter turns
    const cplx64 e = (k & 1) ? cplx64{-s, c} : cplx64{c, s};
    return (k & 2) ? cplx64{-e.re, -e.im} : e;
}

// Coefficients (-1)^m / ((2m)! (4m+1)) and (-1)^m / ((2m+1)! (4m+3)) of the
// Fresnel series in t^2, t = pi x^2 / 2 <= 2 pi: 23 terms end below FP64
// rounding.
struct FresnelSeries {
    static constexpr int kTerms = 23;
    double c[kTerms], s[kTerms];
    constexpr FresnelSeries() : c(), s()
    {
        double f = 1.0;                            // (2m)!
        for (int m = 0; m < kTerms; ++m) {
            const double sign = (m & 1) ? -1.0 : 1.0;
            c[m] = sign / (f * (4 * m + 1));
            f *= 2 * m + 1;
            s[m] = sign / (f * (4 * m + 3));
            f *= 2 * m + 2;
        }
    }
};

// C(x) + i S(x), 0 <= x <= 2
__host__ __device__ inline cplx64 fresnel_series(double x)
{
    constexpr FresnelSeries k;
    const double t = 0.5 * kPi64 * x * x, u = t * t;
    double c = k.c[FresnelSeries::kTerms - 1], s = k.s[FresnelSeries::kTerms - 1];
#pragma unroll
    for (int m = FresnelSeries::kTerms - 2; m >= 0; --m) {
        c = c * u + k.c[m];
        s = s * u + k.s[m];
    }
    return {x * c, x * (t * s)};
}

// 2w / (2w^2+1 - 1*2/(2w^2+5 - ...)) for w = (sqrt(pi)/2)(1-i) x, x > 2, by
// the forward recurrence of numerators and denominators (no division per
// step; they grow by at most (2w^2 + 4n) a step, far inside the FP64 range).
// 2w^2 = -i pi x^2.  The fraction needs 31 steps at x = 2 to reach FP64
// rounding, 124/x^2 + a few in between, and none from x = 10^6 on, where the
// first step changes it by 2/(pi x^2)^2.
__host__ __device__ inline cplx64 erfcx_fraction(double x)
{
    const double wi = kPi64 * x * x;               // 2w^2 = -i wi
    const int steps = x > 1e6 ? 0 : 8 + (int)(128.0 / (x * x));
    cplx64 p0 = {1.0, 0.0}, p1 = {1.0, -wi};       // numerators of f
    cplx64 q0 = {0.0, 0.0}, q1 = {1.0, 0.0};       // denominators
    for (int n = 1; n <= steps; ++n) {
        const double a = (double)(2 * n - 1) * (double)(2 * n);
        const double br = (double)(1 + 4 * n);
        const cplx64 p2 = cplx64{br * p1.re + wi * p1.im, br * p1.im - wi * p1.re} - p0 * a;
        const cplx64 q2 = cplx64{br * q1.re + wi * q1.im, br * q1.im - wi * q1.re} - q0 * a;
        p0 = p1;
        p1 = p2;
        q0 = q1;
        q1 = q2;
    }
    // 2w / (p1/q1) = 2w q1 conj(p1) / |p1|^2
    const double c = sqrt(kPi64) * x;
    const double inv = 1.0 / (p1.re * p1.re + p1.im * p1.im);
    const cplx64 r = q1 * cplx64{p1.re * inv, -p1.im * inv};
    return cplx64{c, -c} * r;
}

// G(x) = g(x) + i f(x), x >= 0.
__host__ __device__ inline cplx64 fresnel_aux(double x)
{
    if (x <= 2.0) {
        const cplx64 cs = fresnel_series(x);
        return cplx64{0.5 - cs.re, 0.5 - cs.im} * cis_pi(-0.5 * x * x);
    }
    return cplx64{0.5, 0.5} * erfcx_fraction(x) * (1.0 / sqrt(kPi64));
}

__host__ __device__ inline cplx64 response64(double q, double z)
{
    const bool neg = z < 0.0;
    if (neg) {
        q = -q;
        z = -z;
    }
    const cplx64 e2q = cis_pi(2.0 * (q - rint(q)));    // exp(i 2 pi q)
    cplx64 r;
    if (z < 1e-30) {           // the drift's phase is below FP64 rounding
        const double d = 1.0 / (2.0 * kPi64 * q);
        r = q == 0.0 ? cplx64{1.0, 0.0} : cplx64{e2q.im * d, (1.0 - e2q.re) * d};
    } else {
        const double qp = q - 0.5 * z;
        const double s = sqrt(2.0 / z);
        const double x1 = s * qp, x2 = s * (qp + z);
        const cplx64 g1 = fresnel_aux(fabs(x1)), g2 = e2q * fresnel_aux(fabs(x2));
        if (x1 >= 0.0)
            r = g1 - g2;
        else if (x2 <= 0.0)
            r = g2 - g1;
        else
            r = cplx64{1.0, 1.0} * cis_pi(-(qp * qp / z)) - g2 - g1;
        r = r * (1.0 / sqrt(2.0 * z));
    }
    return neg ? cplx64{r.re, -r.im} : r;
}

}  // namespace fdas
