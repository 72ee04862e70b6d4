// The 2-D Green's function G = -(j/4) H0^(2)(kappa R) and dG/dR at one wavenumber
// kappa = kr + j ki (kr > 0, ki <= 0), FP64.
//
// With w = j kappa R these are Macdonald functions, G = K0(w) / 2 pi and
// dG/dR = -(j kappa / 2 pi) K1(w), and on the ray of one call only R varies.
//   |kappa| R >= 2:  K_nu(w) = e^-w w^(-1/2) F_nu, F_nu a smooth function of
//       t = 1 / (|kappa| R): polynomials in t with complex coefficients on
//       [0, 1/16], [1/16, 1/8], [1/8, 1/4] and [1/4, 1/2] (degrees 11, 11, 12 and 14:
//       the first coefficient left out is below 5e-17 of F), interpolated on the
//       host at Chebyshev nodes.  There F_nu = int e^(-u^2) (1 + nu u^2 / w) /
//       sqrt(2 + u^2 / w) du (the integral of K_nu over cosh, Abramowitz and Stegun
//       9.6.24, with w (cosh - 1) = u^2) by the trapezoidal rule, which converges
//       geometrically (below 1e-17 at the steps used).
//   |kappa| R < 2:  the power series of K0 and K1 (9.6.10 - 9.6.13) to (w^2/4)^11.
// The polynomials' coefficients are uniform over a launch (LDS broadcasts); a wave
// skips the ranges that none of its lanes is in.  Most pairs are in the first range:
// about 130 FP64 operations for G and dG/dR, where an asymptotic series summed to its
// smallest term with complex divisions and, below |z| = 17, a backward recurrence over
// some 40 orders took fifteen times as long.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <complex>

#include "phase_math.h"

namespace efie {

constexpr int K2_RANGES = 4;
constexpr int K2_MAX = 15;                                  // coefficients of the longest polynomial
__host__ __device__ constexpr int k2_terms(int r) { return r < 2 ? 12 : (r == 2 ? 13 : 15); }
__host__ __device__ constexpr double k2_hi(int r) { return r == 0 ? 1.0 / 16 : (r == 1 ? 1.0 / 8 : (r == 2 ? 0.25 : 0.5)); }

struct Kern2d {
    Phase<double> ph;
    double inv_abs;               // 1 / |kappa|
    double2 lnc;                  // ln(j kappa / 2) + Euler's constant
    double2 qc;                   // w^2 / 4 = qc R^2
    double2 c[K2_RANGES][2][K2_MAX];   // of G and dG/dR over e^(-j kappa R) R^(-1/2), in powers of tau in [-1, 1]
};

inline Kern2d make_kern2d(double kr, double ki) {
    using C = std::complex<double>;
    const double PI_ = 3.14159265358979323846;
    Kern2d k{};
    const C kap(kr, ki), jk = C(0, 1) * kap;
    const double a = std::abs(kap);
    k.ph = make_phase<double>(kr, ki);
    k.inv_abs = 1.0 / a;
    const C l = std::log(0.5 * jk) + 0.57721566490153286061, q = 0.25 * jk * jk;
    k.lnc = make_double2(l.real(), l.imag());
    k.qc = make_double2(q.real(), q.imag());
    const C unit = jk / a;
    // K0 / 2 pi and -(j kappa / 2 pi) K1 without e^-w R^(-1/2)
    const C f0 = 1.0 / (2.0 * PI_ * std::sqrt(jk)), f1 = -std::sqrt(jk) / (2.0 * PI_);
    double lo = 0.0;
    for (int r = 0; r < K2_RANGES; ++r) {
        const int n = k2_terms(r);
        const double hi = k2_hi(r), step = r == 3 ? 0.17 : 0.25;   // |w| >= 2, 4
        C v[2][K2_MAX];
        for (int i = 0; i < n; ++i) {
            const double t = 0.5 * (lo + hi) + 0.5 * (hi - lo) * std::cos(PI_ * (i + 0.5) / n);
            const C iw = t / unit;
            C s0 = 0.0, s1 = 0.0;
            for (int m = 0; m * step < 6.5; ++m) {
                const double u2 = (m * step) * (m * step);
                const C x = u2 * iw, g = (m ? 2.0 : 1.0) * step * std::exp(-u2) / std::sqrt(2.0 + x);
                s0 += g;
                s1 += g * (1.0 + x);
            }
            v[0][i] = s0;
            v[1][i] = s1;
        }
        for (int nu = 0; nu < 2; ++nu) {
            // Chebyshev coefficients, then powers of tau
            double tp[K2_MAX] = {}, tc[K2_MAX] = {};     // T_(j-1), T_j
            C out[K2_MAX];
            for (int j = 0; j < n; ++j) {
                C cj = 0.0;
                for (int i = 0; i < n; ++i) cj += v[nu][i] * std::cos(PI_ * j * (i + 0.5) / n);
                cj *= (j ? 2.0 : 1.0) / n;
                if (j == 0) {
                    tc[0] = 1.0;
                } else {
                    double tn[K2_MAX] = {};
                    for (int x = 0; x < n; ++x) tn[x] = (x ? (j == 1 ? 1.0 : 2.0) * tc[x - 1] : 0.0) - (j == 1 ? 0.0 : tp[x]);
                    for (int x = 0; x < n; ++x) {
                        tp[x] = tc[x];
                        tc[x] = tn[x];
                    }
                }
                for (int x = 0; x < n; ++x) out[x] += cj * tc[x];
            }
            for (int x = 0; x < n; ++x) {
                const C y = out[x] * (nu ? f1 : f0);
                k.c[r][nu][x] = make_double2(y.real(), y.imag());
            }
        }
        lo = hi;
    }
    return k;
}

// the coefficients of the power series, (w^2/4)^k: A0 = sum 1/(k!)^2, B0 = sum H_k/(k!)^2,
// A1 = sum 1/(k!(k+1)!), B1 = sum (H_k + H_(k+1))/(k!(k+1)!)
struct Series2d {
    double c[12][4];
    constexpr Series2d() : c{} {
        double f = 1.0, h = 0.0;
        for (int k = 0; k < 12; ++k) {
            if (k) {
                f /= double(k) * k;
                h += 1.0 / k;
            }
            c[k][0] = f;
            c[k][1] = f * h;
            c[k][2] = f / (k + 1);
            c[k][3] = f / (k + 1) * (2.0 * h + 1.0 / (k + 1));
        }
    }
};

__device__ constexpr Series2d series2d_table{};

struct Series2dSums {
    double2 a0m1, b0, a1, b1;   // A0 - 1, B0, A1, B1
};
__device__ __forceinline__ Series2dSums series2d(const Kern2d& K, double R2) {
    const double qr = K.qc.x * R2, qi = K.qc.y * R2;
    double pr = qr, pi = qi;
    Series2dSums o{make_double2(0, 0), make_double2(0, 0), make_double2(1.0, 0), make_double2(1.0, 0)};
#pragma unroll 1
    for (int k = 1; k < 12; ++k) {
        const double(&s)[4] = series2d_table.c[k];   // scalar loads
        o.a0m1.x += s[0] * pr; o.a0m1.y += s[0] * pi;
        o.b0.x += s[1] * pr; o.b0.y += s[1] * pi;
        o.a1.x += s[2] * pr; o.a1.y += s[2] * pi;
        o.b1.x += s[3] * pr; o.b1.y += s[3] * pi;
        const double t = pr * qr - pi * qi;
        pi = pr * qi + pi * qr;
        pr = t;
    }
    return o;
}

// G and dG/dR by the power series (a call of its own: rare in a launch, and its
// constants would be kept in the registers of every wave)
struct Small2d {
    double2 g, d;
};
static __device__ __attribute__((noinline)) Small2d green2d_small(const Kern2d& K, double R2, double rinv) {
    Small2d v;
    const Series2dSums o = series2d(K, R2);
    const double lx = K.lnc.x + 0.5 * log(R2), ly = K.lnc.y;
    constexpr double I2P = 0.15915494309189533577, IP = 0.31830988618379067154;   // 1 / 2 pi, 1 / pi
    const double ax = 1.0 + o.a0m1.x, ay = o.a0m1.y;
    v.g = make_double2(I2P * (o.b0.x - (lx * ax - ly * ay)), I2P * (o.b0.y - (lx * ay + ly * ax)));
    const double ex = lx * o.a1.x - ly * o.a1.y - 0.5 * o.b1.x, ey = lx * o.a1.y + ly * o.a1.x - 0.5 * o.b1.y;
    const double R = R2 * rinv;
    v.d = make_double2(-I2P * rinv - IP * R * (K.qc.x * ex - K.qc.y * ey), -IP * R * (K.qc.x * ey + K.qc.y * ex));
    return v;
}

// G and dG/dR at NB distances (R2 their squares; rinv receives 1/R); K in LDS.  CK: ki != 0.
// (From the kernel's arguments the compiler keeps every coefficient for all uses, 500 scalar
// registers, spilled to vector lanes; the memory barrier keeps it from doing so here.)
template <int NB, bool CK>
__device__ __forceinline__ void green2d(const Kern2d& K, const double (&R2)[NB], double2 (&G)[NB], double2 (&D)[NB],
                                        double (&rinv)[NB]) {
    asm volatile("" ::: "memory");
    double t[NB];
    bool beyond = false;   // of the first range
    bool small = false, large = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        rinv[b] = rsqrt_fast(R2[b]);
        t[b] = rinv[b] * K.inv_abs;
        beyond |= !(t[b] <= k2_hi(0));
        small |= t[b] > k2_hi(K2_RANGES - 1);
        large |= !(t[b] > k2_hi(K2_RANGES - 1));
    }
    auto range = [&](auto r_, bool select) {
        constexpr int r = decltype(r_)::value;
        constexpr double lo = r ? k2_hi(r - 1) : 0.0, hi = k2_hi(r);
        double tau[NB];
        double2 p[NB], q[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            tau[b] = fma(t[b], 2.0 / (hi - lo), -(hi + lo) / (hi - lo));
            p[b] = K.c[r][0][k2_terms(r) - 1];
            q[b] = K.c[r][1][k2_terms(r) - 1];
        }
#pragma unroll
        for (int x = k2_terms(r) - 2; x >= 0; --x) {
            if (x % 3 == 0) __builtin_amdgcn_sched_barrier(0);   // no more than three steps' coefficients at once
            const double2 c0 = K.c[r][0][x], c1 = K.c[r][1][x];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                p[b].x = fma(p[b].x, tau[b], c0.x);
                p[b].y = fma(p[b].y, tau[b], c0.y);
                q[b].x = fma(q[b].x, tau[b], c1.x);
                q[b].y = fma(q[b].y, tau[b], c1.y);
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (!select || t[b] > lo) {
                G[b] = p[b];
                D[b] = q[b];
            }
    };
    if (__any(large)) {
        range(std::integral_constant<int, 0>{}, false);
        if (__any(beyond)) {
            bool b1 = false, b2 = false;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                b1 |= t[b] > k2_hi(1);
                b2 |= t[b] > k2_hi(2);
            }
            range(std::integral_constant<int, 1>{}, true);
            if (__any(b1)) range(std::integral_constant<int, 2>{}, true);
            if (__any(b2)) range(std::integral_constant<int, 3>{}, true);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const double R = R2[b] * rinv[b];
            double s, c;
            sincos_quarter(R, K.ph.khi, K.ph.klo, s, c);
            double f = rsqrt_fast(R);
            if (CK) f *= exp2_scaled(R, K.ph.ehi, K.ph.elo);
            c *= f;
            s *= f;
            G[b] = make_double2(G[b].x * c + G[b].y * s, G[b].y * c - G[b].x * s);
            D[b] = make_double2(D[b].x * c + D[b].y * s, D[b].y * c - D[b].x * s);
        }
    }
    if (__any(small)) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (!(t[b] > k2_hi(K2_RANGES - 1))) continue;
            const Small2d v = green2d_small(K, R2[b], rinv[b]);
            G[b] = v.g;
            D[b] = v.d;
        }
    }
}

// G + ln(R) / 2 pi, the regular part on a segment with itself (its limit at R = 0)
template <bool CK>
__device__ __forceinline__ double2 green2d_reg(const Kern2d& K, double R) {
    constexpr double I2P = 0.15915494309189533577;
    if (R == 0.0) return make_double2(-I2P * K.lnc.x, -I2P * K.lnc.y);
    const double lr = log(R);
    if (K.inv_abs <= 0.5 * R) {   // |kappa| R >= 2
        const double R2[1] = {R * R};
        double2 g[1], d[1];
        double ri[1];
        green2d<1, CK>(K, R2, g, d, ri);
        return make_double2(g[0].x + I2P * lr, g[0].y);
    }
    const Series2dSums o = series2d(K, R * R);
    const double2 l = K.lnc;
    return make_double2(I2P * (o.b0.x - (l.x * (1.0 + o.a0m1.x) - l.y * o.a0m1.y) - lr * o.a0m1.x),
                        I2P * (o.b0.y - (l.x * o.a0m1.y + l.y * (1.0 + o.a0m1.x)) - lr * o.a0m1.y));
}

}  // namespace efie
