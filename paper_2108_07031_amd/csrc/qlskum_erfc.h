// Complementary error function and exponential for the kinetic split fluxes.
//
// The split fluxes need A = erfc(y)/2 and the Gaussian exp(-S^2) at the same
// argument (|y| = |S|).  For a >= 0, erfc(a) = exp(-a^2) t R(t) with
// t = c/(c + a) and R a polynomial in u = 2t - 1 = (c - a)/(c + a)
// (monomial coefficients in qlskum_erfc_coeffs.h, generated by gen_erfc.py
// from a Chebyshev interpolant), so one exponential serves both A and B and
// erfc costs a reciprocal and a Horner recurrence of one fma per term.
// Negative arguments use erfc(y) = 2 - erfc(-y).  The reciprocal
// inv = 1/(c + |y|) is an argument: the device kernels form it with a
// refined hardware reciprocal, host callers by division.
// In FP32, small arguments (|y| <= 1) use erf's odd polynomial instead.
// The exponential is evaluated here too (exp_poly): a two-part reduction by
// ln2 and a polynomial, without the library's range branches.
// The FP64 flux body takes erf's odd polynomial where |S| <= 1.25
// (half_erfc_near: 14 fma instead of a reciprocal and 22) and comes to the
// form above only past it.
// Evaluated with explicit fma and no implicit contraction, so equal
// arguments give equal results wherever the function is inlined.
#pragma once

#include <hip/hip_runtime.h>

#include "qlskum_erfc_coeffs.h"

namespace ql {

// The FP64 coefficients as the device reads them, from memory in a loop: few waves
// of a transonic flow hold a state past kErfNear64 (local Mach above ~1.5), so the
// flux kernel keeps no registers for them.
struct ErfcTable {
    double c[kErfcN64];
};
constexpr ErfcTable erfc_table() {
    ErfcTable t{};
    for (int k = 0; k < kErfcN64; ++k) t.c[k] = kErfcPoly64[k];
    return t;
}
namespace {
__constant__ ErfcTable kErfcTable = erfc_table();
}
// (a function per side: a table that host code may see is no constant to the device's
// compiler)
__device__ __forceinline__ double erfc_coeff(int k) { return kErfcTable.c[k]; }
__host__ inline double erfc_coeff(int k) { return kErfcPoly64[k]; }

// erfc(a) exp(a^2) in FP32 for finite a >= 0, given inv = 1/(kErfcC32 + a)
__host__ __device__ inline float erfc_scaled_f(float a, float inv) {
#pragma clang fp contract(off)
    const float t = kErfcC32 * inv;
    const float u = (kErfcC32 - a) * inv;
    float r = kErfcPoly32[kErfcN32 - 1];
#pragma unroll
    for (int k = kErfcN32 - 2; k >= 0; --k) r = fmaf(r, u, kErfcPoly32[k]);
    return t * r;
}

// q 2^k for an integral k, 0 or inf where |k| is past the exponent range.
// On the device the conversion to an integer saturates by itself (two
// instructions fewer than clamping k first); NaN converts to 0.
__host__ __device__ inline double scale_pow2(double q, double k) {
#ifdef __HIP_DEVICE_COMPILE__
    int i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(k));
    return ldexp(q, i);
#else
    return ldexp(q, (int)fmin(fmax(k, -2100.0), 2100.0));
#endif
}

// exp(x): x = k ln2 + r with ln2 = hi + lo (Cody and Waite's two-part
// constant, so that r is exact to well below an ulp), |r| <= ln2/2, exp(r)
// by a degree-11 polynomial, times 2^k; 1.4e-16 relative.  No range
// branches: for x below -746 or above 710 the scaling alone gives 0 or inf
// (the exponent saturates in its conversion to an integer), and the
// reduction stays accurate for |x| < 1e15, far past that; NaN propagates.
__host__ __device__ inline double exp_poly(double x) {
#pragma clang fp contract(off)
    const double k = rint(x * kLog2e);
    double r = fma(-k, kLn2Hi, x);
    r = fma(-k, kLn2Lo, r);
    double q = kExpPoly64[kExpN64 - 1];
#pragma unroll
    for (int j = kExpN64 - 2; j >= 0; --j) q = fma(q, r, kExpPoly64[j]);
    return scale_pow2(q, k);
}

// exp(-y^2) with the square split exactly into hi + lo (hi = fl(y*y)), so
// that the rounding of y^2 does not enter: exp(-hi) (1 - lo).
__host__ __device__ inline double gauss(double y) {
#pragma clang fp contract(off)
    const double hi = y * y;
    const double lo = fma(y, y, -hi);
    const double e = exp_poly(-hi);
    return fma(-lo, e, e);
}

// erfc(y) / 2 given gauss = exp(-y^2) and inv = 1/(kErfcC64 + |y|), for every y; the
// flux body takes it past kErfNear64.  The factor erfc(|y|) exp(y^2) = t R(u) is within
// 4.4e-16 (6e-16 with u = 2 t - 1, which saves an operation).
__host__ __device__ __forceinline__ double half_erfc(double y, double gauss, double inv) {
#pragma clang fp contract(off)
    const double t = kErfcC64 * inv;
    const double u = (kErfcC64 - fabs(y)) * inv;
    double r = erfc_coeff(kErfcN64 - 1);
#pragma unroll 1
    for (int k = kErfcN64 - 2; k >= 0; --k) r = fma(r, u, erfc_coeff(k));
    const double h = (0.5 * gauss) * (t * r);
    return (y >= 0.0) ? h : 1.0 - h;
}

// erfc(-y) / 2 = 1/2 + y P(y^2) for |y| <= kErfNear64, within 2^-52 (half an
// ulp of the sum and an ulp each of y^2 and y P, |y P| < 1/2).  Measured 1.4e-16
// absolute; half_erfc there is within 2.7e-16.  For y < 0 the sum cancels and the
// relative error is the larger one, 1.7e-15 against 6.2e-16, but a flux adds u_e A to
// a term of order 1 and takes on the absolute error: with half_erfc throughout, the
// residual's rounding error is the same to 1.3 times as large.
__host__ __device__ inline double half_erfc_near(double y) {
#pragma clang fp contract(off)
    const double u = y * y;
    double r = kErfPoly64[0];
#pragma unroll
    for (int k = 1; k < kErfN64; ++k) r = fma(r, u, kErfPoly64[k]);
    return fma(y, r, 0.5);
}

// FP32: for |y| <= 1 (local Mach below ~1.2) (1 - y P(y^2)) / 2 with a short
// polynomial, so waves whose arguments all lie there skip the reciprocal and
// the recurrence; inv = 1/(kErfcC32 + |y|) is used only above 1.
__host__ __device__ inline float half_erfc_f(float y, float gauss, float inv) {
#pragma clang fp contract(off)
    if (fabsf(y) <= 1.0f) {
        const float u = y * y;
        float p = kErfP32[0];
#pragma unroll
        for (int k = 1; k < kErfP32N; ++k) p = fmaf(p, u, kErfP32[k]);
        return fmaf(-0.5f * y, p, 0.5f);
    }
    const float h = (0.5f * gauss) * erfc_scaled_f(fabsf(y), inv);
    return (y >= 0.0f) ? h : 1.0f - h;
}

}  // namespace ql
