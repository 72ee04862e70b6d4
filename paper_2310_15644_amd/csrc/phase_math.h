// e^(-j k R) / R and its parts for k = kr + j ki in FP64 and FP32.
//
// The FP64 far pairs spend nearly all their time here.  The library's sincos and
// exp cover every argument (a branch for large ones, special values) and took
// about 300 issue slots per Green's function together with the moments; a phase
// k R with R the distance of two points needs one reduction without a branch:
//   u = R (2 k / pi) as a product and its remainder (the constant in two parts, one
//   fused multiply-add each), n = rint(u) by the 1.5 * 2^52 shift (its low bits
//   are the quadrant, for |u| < 2^51), f = u - n in [-1/2, 1/2];
//   sin(pi f / 2) and cos(pi f / 2) by polynomials of degree 13 and 14 in f,
//   interpolated at Chebyshev nodes in 60 digits (errors 5e-18 and 3e-20 before
//   rounding); 2^t by degree 11 (3e-18).
// Every value is within about an ulp of the function at the rounded R, as before.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace efie {

// the wavenumber as the kernels take it
template <typename R>
struct Phase;
template <>
struct Phase<float> {
    float krev, ki;   // revolutions per unit length (hardware sine and cosine), Im k
};
template <>
struct Phase<double> {
    double khi, klo;   // 2 kr / pi in two parts
    double ehi, elo;   // ki / ln 2 in two parts
};

template <typename R>
__host__ __device__ inline Phase<R> make_phase(double kr, double ki);
template <>
__host__ __device__ inline Phase<float> make_phase<float>(double kr, double ki) {
    return {float(kr / (2.0 * 3.14159265358979323846)), float(ki)};
}
template <>
__host__ __device__ inline Phase<double> make_phase<double>(double kr, double ki) {
    constexpr double C = 0.6366197723675814, CL = -3.935735335036497e-17;     // 2 / pi
    constexpr double L = 1.4426950408889634, LL = 2.0355273740931033e-17;     // 1 / ln 2
    Phase<double> p;
    p.khi = kr * C;
    p.klo = ::fma(kr, C, -p.khi) + kr * CL;
    p.ehi = ki * L;
    p.elo = ::fma(ki, L, -p.ehi) + ki * LL;
    return p;
}

// 1 / sqrt(x): the hardware estimate and one third-order step
__device__ __forceinline__ double rsqrt_fast(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// 1 / x: the hardware estimate and one third-order step
__device__ __forceinline__ double rcp_fast(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// sqrt(x), x = 0 included
__device__ __forceinline__ double root_fast(double x) { return x * rsqrt_fast(fmax(x, 1e-300)); }

// sine and cosine of (pi / 2) x (hi + lo)
__device__ __forceinline__ void sincos_quarter(double x, double hi, double lo, double& sn, double& cs) {
    constexpr double SHIFT = 6755399441055744.0;   // 1.5 * 2^52
    const double t = fma(x, hi, SHIFT);
    const double f = fma(x, lo, fma(x, hi, -(t - SHIFT)));
    const uint32_t q = uint32_t(__double2loint(t));
    const double y = f * f;
    double s = 5.63393378153785395e-8;
    s = fma(s, y, -3.5986433529823097e-6);
    s = fma(s, y, 0.000160441150742190911);
    s = fma(s, y, -0.00468175413234097599);
    s = fma(s, y, 0.0796926262460430031);
    s = fma(s, y, -0.645964097506244316);
    s = fma(s, y, 1.57079632679489661);
    s *= f;
    double c = -6.32125686962858841e-9;
    c = fma(c, y, 4.71060972675782301e-7);
    c = fma(c, y, -0.0000252020367704602584);
    c = fma(c, y, 0.000919260274183155721);
    c = fma(c, y, -0.0208634807633112091);
    c = fma(c, y, 0.253669507901046709);
    c = fma(c, y, -1.23370055013616981);
    c = fma(c, y, 1.0);
    const bool odd = q & 1;
    const double a = odd ? c : s, b = odd ? s : c;
    // sign bits: sine from bit 1 of q, cosine from bit 1 of q + 1
    sn = __hiloint2double(__double2hiint(a) ^ int((q << 30) & 0x80000000u), __double2loint(a));
    cs = __hiloint2double(__double2hiint(b) ^ int(((q + 1) << 30) & 0x80000000u), __double2loint(b));
}

// 2^(x (hi + lo))
__device__ __forceinline__ double exp2_scaled(double x, double hi, double lo) {
    const double n = rint(x * hi);
    const double f = fma(x, lo, fma(x, hi, -n));
    double p = 4.45581790833606449e-10;
    p = fma(p, f, 7.07419429728852101e-9);
    p = fma(p, f, 1.01780570877339411e-7);
    p = fma(p, f, 1.32154325359123762e-6);
    p = fma(p, f, 0.0000152527338415567726);
    p = fma(p, f, 0.000154035304637243542);
    p = fma(p, f, 0.00133335581464064707);
    p = fma(p, f, 0.00961812910758725667);
    p = fma(p, f, 0.055504108664821627);
    p = fma(p, f, 0.240226506959101596);
    p = fma(p, f, 0.693147180559945309);
    p = fma(p, f, 1.0);
    return __builtin_amdgcn_ldexp(p, int(fmax(n, -4000.0)));   // k_im <= 0: n <= 0, flushed to zero far below 2^-1074
}

// exp(-j k R) / R from R^2.  FP64: the functions above.
__device__ __forceinline__ void green_far(const Phase<double>& ph, bool ck, double R2, double& gr, double& gi) {
    const double rinv = rsqrt_fast(R2);
    const double R = R2 * rinv;
    double s, c;
    sincos_quarter(R, ph.khi, ph.klo, s, c);
    const double e = ck ? exp2_scaled(R, ph.ehi, ph.elo) * rinv : rinv;
    gr = c * e;
    gi = -s * e;
}
// FP32: the phase in revolutions goes to the hardware sine and cosine (valid for
// |x| < 256).
__device__ __forceinline__ void green_far(const Phase<float>& ph, bool ck, float R2, float& gr, float& gi) {
    const float rinv = __builtin_amdgcn_rsqf(R2);
    const float R = R2 * rinv;
    const float x = ph.krev * R;
    const float s = __builtin_amdgcn_sinf(x);
    const float c = __builtin_amdgcn_cosf(x);
    const float e = ck ? __expf(ph.ki * R) * rinv : rinv;
    gr = c * e;
    gi = -s * e;
}

}  // namespace efie
