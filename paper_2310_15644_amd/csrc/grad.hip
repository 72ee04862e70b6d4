// Adjoint vertex gradient of a far-field objective.
//
// For J = sum_{d,c} |F_dc|^2 with F = R(x) j, Z(x) j = V(x) and the adjoint
// Z lambda = R^T conj(F) (Z = Z^T), the gradient with respect to the vertex
// positions x is
//   dJ/dx = 2 Re[ sum_dc w_dc (dR_dc/dx) j + lambda^T dV/dx - lambda^T (dZ/dx) j ],
// w = conj(F).  This file evaluates the three terms for given j, lambda, w:
//
//  * operator term: lambda^T Z j = sum_{p,q} lambda_p^T B_pq j_q over triangle-pair
//    blocks B_pq, and B_pq(x) = B_qp(x)^T as functions of all vertex positions
//    (the pair integral is symmetric; near blocks are symmetrised).  Hence the
//    derivative with respect to the vertices of triangle t is the sum over q of
//    the derivatives of  lambda_t^T B_tq j_q + j_t^T B_tq lambda_q  taken with
//    respect to t's vertices only (t as test triangle).  One block owns one test
//    triangle t and 256 source triangles: its lanes' derivatives reduce to the 9
//    coordinates of t, added with 9 atomics.
//      far pairs, and the smooth part of the near ones: analytic chain rule through
//      G(R), the quadrature points r_a = sum_k l^a_k P_k and the edge lengths in the
//      RWG coefficients;
//      singular part of the near pairs: forward-mode dual numbers (value + one
//      directional derivative) through the closed forms, a lane per test coordinate
//      and point.
//  * excitation and radiation terms: per triangle, same chain rule.
// Per-triangle-vertex accumulators (T x 3 x 3) are finally scattered to vertices.
#include <hip/hip_runtime.h>

#include <cmath>

#include "efie_internal.h"
#include "linalg.h"
#include "pair_kernels.h"

namespace efie {

struct Rule {
    double bary[7][3];   // Radon degree-5 rule: barycentric coordinates and weights (sum 1)
    double w[7];
};

struct C {
    double r, i;
};
__device__ __forceinline__ C cm(C a, C b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__device__ __forceinline__ C cs(C a, double s) { return {a.r * s, a.i * s}; }
__device__ __forceinline__ C ca(C a, C b) { return {a.r + b.r, a.i + b.i}; }

// ------------------------------------------------------------ dual numbers
// a value and its derivative with respect to one coordinate of the test triangle
struct Dual {
    double v, d;
};
__device__ __forceinline__ Dual operator+(Dual a, Dual b) { return {a.v + b.v, a.d + b.d}; }
__device__ __forceinline__ Dual operator-(Dual a, Dual b) { return {a.v - b.v, a.d - b.d}; }
__device__ __forceinline__ Dual operator-(Dual a) { return {-a.v, -a.d}; }
__device__ __forceinline__ Dual operator*(Dual a, Dual b) { return {a.v * b.v, a.d * b.v + a.v * b.d}; }
__device__ __forceinline__ Dual operator+(Dual a, double b) { return {a.v + b, a.d}; }
__device__ __forceinline__ Dual operator-(Dual a, double b) { return {a.v - b, a.d}; }
__device__ __forceinline__ Dual operator-(double a, Dual b) { return {a - b.v, -b.d}; }
__device__ __forceinline__ Dual operator*(Dual a, double b) { return {a.v * b, a.d * b}; }
__device__ __forceinline__ Dual operator*(double a, Dual b) { return b * a; }
__device__ __forceinline__ Dual operator/(Dual a, Dual b) {
    const double i = rcp_fast(b.v), r = a.v * i;
    return {r, (a.d - r * b.d) * i};
}
__device__ __forceinline__ Dual inverse(Dual a) {
    const double i = rcp_fast(a.v);
    return {i, -i * i * a.d};
}
__device__ __forceinline__ double inverse(double a) { return 1.0 / a; }
__device__ __forceinline__ Dual root(Dual a) {
    const double y = rsqrt_fast(fmax(a.v, 1e-300));   // 0 at 0, where a.d = 0 too
    return {a.v * y, 0.5 * y * a.d};
}
__device__ __forceinline__ double root(double a) { return sqrt(a); }
// calls: inlined, their polynomials' constants fill the registers of the whole kernel
__device__ __noinline__ double log_call(double x) { return log(x); }
__device__ __noinline__ double atan_call(double x) { return atan(x); }
__device__ __forceinline__ Dual dlog(Dual a) { return {log_call(a.v), a.d * rcp_fast(a.v)}; }
__device__ __forceinline__ Dual datan(Dual a) { return {atan_call(a.v), a.d * rcp_fast(1.0 + a.v * a.v)}; }
__device__ __forceinline__ Dual dabs(Dual a) { return a.v >= 0.0 ? a : -a; }

// 3-vectors of duals or plain numbers; the products of the two kinds are duals
template <typename T>
struct V3 {
    T x, y, z;
};
template <typename A, typename B>
__device__ __forceinline__ auto sub(const V3<A>& a, const V3<B>& b) -> V3<decltype(a.x - b.x)> {
    return {a.x - b.x, a.y - b.y, a.z - b.z};
}
template <typename A, typename B>
__device__ __forceinline__ auto add(const V3<A>& a, const V3<B>& b) -> V3<decltype(a.x + b.x)> {
    return {a.x + b.x, a.y + b.y, a.z + b.z};
}
template <typename A, typename B>
__device__ __forceinline__ auto dot(const V3<A>& a, const V3<B>& b) {
    return a.x * b.x + a.y * b.y + a.z * b.z;
}
template <typename A, typename B>
__device__ __forceinline__ auto crs(const V3<A>& a, const V3<B>& b) -> V3<decltype(a.y * b.z)> {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <typename A, typename S>
__device__ __forceinline__ auto scl(const V3<A>& a, const S& s) -> V3<decltype(a.x * s)> {
    return {a.x * s, a.y * s, a.z * s};
}
template <typename A>
__device__ __forceinline__ A nrm(const V3<A>& a) { return root(dot(a, a)); }

// Closed-form I0 = int 1/R and I1 = int r'/R (Wilton et al. 1984) over the source triangle u[3]
// (counter-clockwise, positions relative to any common origin, unit normal n) and the
// observation point r, one of the two dual.  Where r lies in the triangle's plane, up to
// rounding, the slope of |d| is one of two, whose mean is taken: none.  (It counts on the
// triangle alone, for its own points or those of a body that touches it: off the triangle
// the angles of the edges add up to zero.)
template <typename TR, typename TU>
__device__ __forceinline__ void potentials_d(const V3<TR>& r, V3<TU> (&u)[3], const V3<TU>& n, double h, Dual& I0,
                                             V3<Dual>& I1) {
    const Dual d = dot(sub(r, u[0]), n);
    const Dual ad = fabs(d.v) <= 1e-14 * h ? Dual{0, 0} : dabs(d);
    const V3<Dual> rho = sub(r, scl(n, d));
    I0 = Dual{0, 0};
    I1 = {I0, I0, I0};
#pragma unroll 1
    for (int e = 0; e < 3; ++e) {
        const V3<TU> rm = u[0], rp = u[1];
        V3<TU> lt = sub(rp, rm);
        lt = scl(lt, inverse(nrm(lt)));
        const V3<TU> uu = crs(lt, n);
        const Dual lp = dot(sub(rp, rho), lt), lm = dot(sub(rm, rho), lt);
        const Dual P0 = dot(sub(rm, rho), uu);
        const Dual R02 = P0 * P0 + d * d;
        const Dual Rp = nrm(sub(r, rp)), Rm = nrm(sub(r, rm));
        Dual lg = {0, 0}, at = {0, 0};
        if (sqrt(R02.v) >= 1e-12 * h) {
            const Dual fp = lp.v >= 0.0 ? Rp + lp : R02 / (Rp - lp);
            const Dual fm = lm.v >= 0.0 ? Rm + lm : R02 / (Rm - lm);
            lg = dlog(fp / fm);
            at = datan(P0 * lp / (R02 + ad * Rp)) - datan(P0 * lm / (R02 + ad * Rm));
        }
        I0 = I0 + P0 * lg - ad * at;
        I1 = add(I1, scl(uu, 0.5 * (R02 * lg + lp * Rp - lm * Rm)));
        u[0] = rp;   // rotated in place, back in order after the three edges
        u[1] = u[2];
        u[2] = rm;
    }
    I1 = add(I1, scl(rho, I0));
}

// ---------------------------------------------------------- operator term
// acc[t][k][x] += -2 Re d/dP_k^x (lambda_t^T B_tq j_q + j_t^T B_tq lambda_q): every
// far pair, and the smooth part (exp(-jkR) - 1)/R of the near ones (the same rule with
// another kernel; its value and slope at R = 0 drop out of the derivative).
//
// With the offsets d_a, d'_b of the points and u_i, u'_j of the vertices from the
// centroids, and alpha_i = s_i l_i lambda_i (or j_i) on t, beta_j likewise on q, the pair's
// sum is sum_ab w_a w_b Phi_ab G_ab, and Phi, the two contractions together, is bilinear:
//   Phi_ab = alpha0 - H . d_a + (E d_a - F) . d'_b
// with constants of the pair.  So a point pair costs its Green's function, six
// multiply-adds for Phi and the folds of w G and w G' Phi / R over b into barycentric
// moments (Bary in pair_kernels.h); the points are multiples of the vertex offsets (0,
// D1 u_k, D2 u_k); the test sums M_kl = sum w l_k w' l'_l G and P_k = sum w l_k (gradient
// vector) carry all nine coordinates.  About 85 FP64 operations per point pair, where
// the vectors U_a, V_b and the library's sincos took four times as many.
// Bound by the vector ALU; N = 7680 (26.2 M ordered pairs): 19.1 ms
// before, 5.2 ms now.
__global__ __launch_bounds__(256, 2) void grad_far_kernel(DevMesh m, double kr, Scale sc, const double2* __restrict__ lam,
                                                       const double2* __restrict__ jv, double* __restrict__ acc,
                                                       int nqblk) {
    __shared__ double red[4][9];
    const int T = m.T;
    const int t = blockIdx.x / nqblk;
    const int q = (blockIdx.x - t * nqblk) * 256 + threadIdx.x;
    double out[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) out[k] = 0.0;
    if (q < T) {
        const bool near = is_near(m, t, q);
        const double smooth = near ? 0.0 : 1.0;   // 1 of the far kernel's cosine
        // Points of near triangles that coincide (of one triangle, or where two bodies touch) are
        // rounded apart here, by some 6 units of the last place of h; and below R = 2 eps / k
        // the rounding of the slope passes the slope itself, k^2 / 2.  R = 0 up to there.
        const double r0 = 2e-15 * (m.hm[t] + 1.0 / kr), zero2 = near ? r0 * r0 : -1.0;
        const Phase<double> ph = make_phase<double>(0.5 * kr, 0.0);
        // a triangle's vertex offsets, s_i l_i and the two weighted coefficients
        auto corners = [&](int tri, double (&u)[3][3], double (&len)[3], C (&wl)[3], C (&wj)[3]) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                u[i][0] = m.vx[i * T + tri];
                u[i][1] = m.vy[i * T + tri];
                u[i][2] = m.vz[i * T + tri];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
                const double dx = u[i1][0] - u[i2][0], dy = u[i1][1] - u[i2][1], dz = u[i1][2] - u[i2][2];
                len[i] = sqrt(dx * dx + dy * dy + dz * dz);
                const double w = m.cf[i * T + tri] > 0.0 ? len[i] : -len[i];
                const double2 l = lam[m.te[i * T + tri]], j = jv[m.te[i * T + tri]];
                wl[i] = {l.x * w, l.y * w};
                wj[i] = {j.x * w, j.y * w};
            }
        };
        const C c1 = {0.25 * sc.ar, 0.25 * sc.ai}, c2 = {sc.pr, sc.pi};
        double ut[3][3], uq[3][3];
        C alpha0, E, H[3], F[3];
        {
            double lt[3], lq[3];
            C aL[3], aJ[3], bL[3], bJ[3];
            corners(t, ut, lt, aL, aJ);
            corners(q, uq, lq, bL, bJ);
            const C A0L = ca(ca(aL[0], aL[1]), aL[2]), A0J = ca(ca(aJ[0], aJ[1]), aJ[2]);
            const C B0J = ca(ca(bJ[0], bJ[1]), bJ[2]), B0L = ca(ca(bL[0], bL[1]), bL[2]);
            const C ab = ca(cm(A0L, B0J), cm(A0J, B0L));
            E = cm(c1, ab);
            C hg = {0, 0};
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const C hL = ca(ca(cs(aL[0], ut[0][x]), cs(aL[1], ut[1][x])), cs(aL[2], ut[2][x]));
                const C hJ = ca(ca(cs(aJ[0], ut[0][x]), cs(aJ[1], ut[1][x])), cs(aJ[2], ut[2][x]));
                const C gL = ca(ca(cs(bL[0], uq[0][x]), cs(bL[1], uq[1][x])), cs(bL[2], uq[2][x]));
                const C gJ = ca(ca(cs(bJ[0], uq[0][x]), cs(bJ[1], uq[1][x])), cs(bJ[2], uq[2][x]));
                F[x] = cm(c1, ca(cm(hL, B0J), cm(hJ, B0L)));
                H[x] = cm(c1, ca(cm(A0L, gJ), cm(A0J, gL)));
                hg = ca(hg, ca(cm(hL, gJ), cm(hJ, gL)));
            }
            alpha0 = ca(cm(c1, hg), cm(c2, ab));
        }
        const double D[3] = {m.cx[t] - m.cx[q], m.cy[t] - m.cy[q], m.cz[t] - m.cz[q]};
        C M[3][3];        // [k][l]
        double P[3][3];   // [k][x], real part
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int l = 0; l < 3; ++l) M[k][l] = {0, 0}, P[k][l] = 0.0;
#pragma unroll 1
        for (int a = 0; a < 7; ++a) {
            const double da[3] = {m.qx[a * T + t], m.qy[a * T + t], m.qz[a * T + t]};
            double o[3];
            C al = alpha0, be[3];
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                o[x] = D[x] + da[x];
                al.r -= H[x].r * da[x];
                al.i -= H[x].i * da[x];
                be[x] = {E.r * da[x] - F[x].r, E.i * da[x] - F[x].i};
            }
            double gr[7], gi[7], hr[7];
#pragma unroll
            for (int b = 0; b < 7; ++b) {
                // d'_b: 0, D1 u'_k, D2 u'_k
                const double f = b == 0 ? 0.0 : (b < 4 ? Bary<7>::D1 : Bary<7>::D2);
                const double* u = uq[b == 0 ? 0 : (b - 1) % 3];
                const double dx = o[0] - f * u[0], dy = o[1] - f * u[1], dz = o[2] - f * u[2];
                const double R2 = dx * dx + dy * dy + dz * dz;
                const bool zero = R2 <= zero2;
                const double Ri = zero ? 0.0 : rsqrt_fast(R2);
                double s2, c2_;
                sincos_quarter(R2 * Ri, ph.khi, ph.klo, s2, c2_);   // of k R / 2
                const double sn = 2.0 * s2 * c2_, cm1 = -2.0 * s2 * s2;
                // G = ((1 +) cos - 1 - j sin)/R;  G'/R = -(G + j k exp(-jkR))/R^2
                const double g_r = (smooth + cm1) * Ri, g_i = zero ? -kr : -sn * Ri;
                const double R2i = -Ri * Ri;
                const double p_r = (g_r + kr * sn) * R2i, p_i = (g_i + kr * (1.0 + cm1)) * R2i;
                double F_r = al.r, F_i = al.i;   // Phi_ab
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    F_r += f * (be[x].r * u[x]);
                    F_i += f * (be[x].i * u[x]);
                }
                gr[b] = g_r;
                gi[b] = g_i;
                hr[b] = p_r * F_r - p_i * F_i;
            }
            double sr[3], si[3], tr[3];
            Bary<7>::fold(gr, sr);
            Bary<7>::fold(gi, si);
            Bary<7>::fold(hr, tr);
            const double(&ck)[3] = bary_table<7, double>.c[a];
            // gradient vector sum_b w_b G'/R Phi (r_a - r_b)
            const double T0 = tr[0] + tr[1] + tr[2];
            double g[3];
#pragma unroll
            for (int x = 0; x < 3; ++x)
                g[x] = o[x] * T0 - (tr[0] * uq[0][x] + tr[1] * uq[1][x] + tr[2] * uq[2][x]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int l = 0; l < 3; ++l) {
                    M[k][l].r += ck[k] * sr[l];
                    M[k][l].i += ck[k] * si[l];
                    P[k][l] += ck[k] * g[l];
                }
        }
        // dS/dP_k^x = P_k + E m1_k - H m0_k - (p_k m1 - r_k m0) + the edge lengths' terms,
        // m0_k = sum_l M_kl, m1_k = sum_l M_kl u'_l, m0, m1 their sums over k
        double lt[3], lq[3];
        C aL[3], aJ[3], bL[3], bJ[3];
        corners(t, ut, lt, aL, aJ);
        corners(q, uq, lq, bL, bJ);
        const C B0J = ca(ca(bJ[0], bJ[1]), bJ[2]), B0L = ca(ca(bL[0], bL[1]), bL[2]);
        C m0k[3], m1k[3][3], m0 = {0, 0}, m1[3] = {{0, 0}, {0, 0}, {0, 0}}, theta = {0, 0}, psi[3], gL[3], gJ[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            m0k[k] = ca(ca(M[k][0], M[k][1]), M[k][2]);
            m0 = ca(m0, m0k[k]);
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                m1k[k][x] = ca(ca(cs(M[k][0], uq[0][x]), cs(M[k][1], uq[1][x])), cs(M[k][2], uq[2][x]));
                m1[x] = ca(m1[x], m1k[k][x]);
                theta = ca(theta, cs(m1k[k][x], ut[k][x]));
            }
        }
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            psi[x] = ca(ca(cs(m0k[0], ut[0][x]), cs(m0k[1], ut[1][x])), cs(m0k[2], ut[2][x]));
            gL[x] = ca(ca(cs(bL[0], uq[0][x]), cs(bL[1], uq[1][x])), cs(bL[2], uq[2][x]));
            gJ[x] = ca(ca(cs(bJ[0], uq[0][x]), cs(bJ[1], uq[1][x])), cs(bJ[2], uq[2][x]));
        }
        double edge[3];   // Re of the factor of dl_i / l_i
        C p[3], r[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            p[i] = ca(cm(aL[i], B0J), cm(aJ[i], B0L));
            C um = {0, 0}, rt = {0, 0};
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                r[i][x] = ca(cm(aL[i], gJ[x]), cm(aJ[i], gL[x]));
                um = ca(um, cs(m1[x], ut[i][x]));
                rt = ca(rt, cm(r[i][x], ca(psi[x], cs(m0, -ut[i][x]))));
            }
            const C y = ca(cm(p[i], ca(theta, cs(um, -1.0))), cs(rt, -1.0));
            edge[i] = ca(cm(c1, y), cm(c2, cm(m0, p[i]))).r;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                C g = ca(cm(E, m1k[k][x]), cs(cm(H[x], m0k[k]), -1.0));
                g = ca(g, cs(cm(c1, ca(cm(p[k], m1[x]), cs(cm(r[k][x], m0), -1.0))), -1.0));
                out[3 * k + x] = P[k][x] + g.r;
            }
        // l_i depends on P_(i+1) (along +e_i) and P_(i+2) (along -e_i), e_i from i+2 to i+1
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
            const double f = edge[i] / (lt[i] * lt[i]);
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const double v = f * (ut[i1][x] - ut[i2][x]);
                out[3 * i1 + x] += v;
                out[3 * i2 + x] -= v;
            }
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) out[k] *= -2.0;
    }
    // reduce over the block: 9 values for triangle t
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) out[k] += __shfl_xor(out[k], o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0)
        for (int k = 0; k < 9; ++k) red[w][k] = out[k];
    __syncthreads();
    if (threadIdx.x < 9) {
        const double s = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
        atomicAdd(&acc[size_t(t) * 9 + threadIdx.x], s);
    }
}

// The singular parts 1/R of the ordered near pairs (t, q), symmetrised: half of t's
// points against the closed form over q and half of q's points against that over t.
// A wave per pair, lane 9 a + c at point a of both triangles and coordinate c of t, both
// contractions together: no lane holds more than one point's duals, and the roots and
// logarithms of a pair run side by side.  sc.ar = sc.pr = 0 (real k), so only the
// imaginary parts of the contractions enter.  Bound by the vector ALU.  A thread per pair
// with nine passes over the contractions, the smooth part included, took 9.0 ms at
// N = 7680 (182290 pairs); 1.8 ms now (three waves per SIMD spill: 3.5 ms).
__global__ __launch_bounds__(256, 2) void grad_near_kernel(DevMesh m, Scale sc, const double2* __restrict__ lam,
                                                        const double2* __restrict__ jv, double* __restrict__ acc) {
    const int e = int(blockIdx.x * 4u + (threadIdx.x >> 6)), lane = int(threadIdx.x) & 63;
    if (e >= m.n_near) return;   // whole waves
    const int T = m.T;
    const int t = m.near_p[e], q = m.near_q[e];
    const int g = lane / 9, c = lane - 9 * g;
    double out = 0.0;
    if (g < 7) {
        // positions relative to the centroid of q
        const V3<double> D = {m.cx[t] - m.cx[q], m.cy[t] - m.cy[q], m.cz[t] - m.cz[q]};
        V3<double> Pq[3];
        V3<Dual> Pt[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            Pt[i] = {{D.x + m.vx[i * T + t], c == 3 * i ? 1.0 : 0.0},
                     {D.y + m.vy[i * T + t], c == 3 * i + 1 ? 1.0 : 0.0},
                     {D.z + m.vz[i * T + t], c == 3 * i + 2 ? 1.0 : 0.0}};
            Pq[i] = {m.vx[i * T + q], m.vy[i * T + q], m.vz[i * T + q]};
        }
        // S_ij: imaginary part of both contractions' coefficients, without t's edge lengths
        double S[3][3];
        {
            C aL[3], aJ[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double2 l = lam[m.te[i * T + t]], j = jv[m.te[i * T + t]];
                const double s = m.cf[i * T + t] > 0.0 ? 1.0 : -1.0;
                aL[i] = {s * l.x, s * l.y};
                aJ[i] = {s * j.x, s * j.y};
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double2 l = lam[m.te[j * T + q]], v = jv[m.te[j * T + q]];
                double w = nrm(sub(Pq[(j + 1) % 3], Pq[(j + 2) % 3]));
                if (m.cf[j * T + q] < 0.0) w = -w;
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    S[i][j] = w * ((aL[i].r * v.y + aL[i].i * v.x) + (aJ[i].r * l.y + aJ[i].i * l.x));
            }
        }
        // a_i = sum_j S_ij, v_i = sum_j S_ij Q_j; l_i the lengths of t's edges
        double a[3];
        V3<double> v[3];
        Dual l[3], sum = {0, 0};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            l[i] = nrm(sub(Pt[(i + 1) % 3], Pt[(i + 2) % 3]));
            a[i] = S[i][0] + S[i][1] + S[i][2];
            v[i] = add(add(scl(Pq[0], S[i][0]), scl(Pq[1], S[i][1])), scl(Pq[2], S[i][2]));
            sum = sum + l[i] * a[i];
        }
        // point g: 1/3 of the vertices' sum and D1 or D2 of one vertex's offset from it
        const double f = g == 0 ? 0.0 : (g < 4 ? Bary<7>::D1 : Bary<7>::D2), b0 = (1.0 - f) / 3.0;
        const double wa = g == 0 ? Bary<7>::W0 : (g < 4 ? Bary<7>::W1 : Bary<7>::W2);
        const int kv = g == 0 ? -1 : (g - 1) % 3;
        double by[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) by[i] = b0 + (i == kv ? f : 0.0);
        const V3<Dual> rt = add(add(scl(Pt[0], by[0]), scl(Pt[1], by[1])), scl(Pt[2], by[2]));
        const V3<double> rq = add(add(scl(Pq[0], by[0]), scl(Pq[1], by[1])), scl(Pq[2], by[2]));
        Dual z, I0;
        V3<Dual> I1;
        {   // t's point against q: sum_i l_i (r - P_i) . (a_i I1 - v_i I0)
            V3<double> n = crs(sub(Pq[1], Pq[0]), sub(Pq[2], Pq[0]));
            const double i2a = 1.0 / nrm(n);
            n = scl(n, i2a);
            potentials_d(rt, Pq, n, m.hm[q], I0, I1);
            Dual uw = {0, 0};
#pragma unroll
            for (int i = 0; i < 3; ++i) uw = uw + l[i] * dot(sub(rt, Pt[i]), sub(scl(I1, a[i]), scl(v[i], I0)));
            z = (uw * (0.25 * sc.ai) + I0 * sum * sc.pi) * i2a;
        }
        {   // q's point against t: sum_i l_i (I1 - P_i I0) . (a_i r - v_i)
            V3<Dual> n = crs(sub(Pt[1], Pt[0]), sub(Pt[2], Pt[0]));
            const Dual i2a = inverse(nrm(n));
            n = scl(n, i2a);
            potentials_d(rq, Pt, n, m.hm[t], I0, I1);
            Dual uw = {0, 0};
#pragma unroll
            for (int i = 0; i < 3; ++i) uw = uw + l[i] * dot(sub(I1, scl(Pt[i], I0)), sub(scl(rq, a[i]), v[i]));
            z = z + (uw * (0.25 * sc.ai) + I0 * sum * sc.pi) * i2a;
        }
        // -2 Re of j (j sc.. and the half of each side are in z's factors)
        out = 2.0 * wa * z.d;
    }
    const double u = __shfl_down(out, 36, 64);   // points 4, 5, 6 to 0, 1, 2
    if (g < 3) out += u;
    double v = __shfl_down(out, 18, 64);
    const double w = __shfl_down(out, 9, 64), y = __shfl_down(out, 27, 64);
    if (lane < 9) atomicAdd(&acc[size_t(t) * 9 + lane], (out + w) + (v + y));
}

// ------------------------------------------------ excitation and radiation terms
// per triangle t:  S_V = (e0/2) sum_a w_a (U^lambda_a . pol) exp(-j k khat . r_a)
//                  S_R = (1/2) sum_a w_a U^j_a . E(r_a),  E(r) = sum_dc W_dc rho e_dc exp(j k rhat_d . r)
// acc[t][k][x] += 2 Re dS/dP_k^x
__global__ __launch_bounds__(128) void grad_tri_kernel(DevMesh m, double kr, double eta, Rule rule,
                                                       const double2* __restrict__ lam, const double2* __restrict__ jv,
                                                       const double2* __restrict__ W, const double* __restrict__ dirs,
                                                       int ndir, double kx, double ky, double kz, double px, double py,
                                                       double pz, double e0, double* __restrict__ acc) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m.T) return;
    const int T = m.T;
    double u[3][3], e[3][3], l[3];
    C aL[3], aJ[3];
    for (int i = 0; i < 3; ++i) {
        u[i][0] = m.vx[i * T + t];
        u[i][1] = m.vy[i * T + t];
        u[i][2] = m.vz[i * T + t];
    }
    for (int i = 0; i < 3; ++i) {
        const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
        const double ev[3] = {u[i1][0] - u[i2][0], u[i1][1] - u[i2][1], u[i1][2] - u[i2][2]};
        l[i] = sqrt(ev[0] * ev[0] + ev[1] * ev[1] + ev[2] * ev[2]);
        for (int x = 0; x < 3; ++x) e[i][x] = ev[x] / l[i];
        const double s = m.cf[i * T + t] > 0.0 ? 1.0 : -1.0;
        const double2 a = lam[m.te[i * T + t]], b = jv[m.te[i * T + t]];
        aL[i] = {a.x * s * l[i], a.y * s * l[i]};
        aJ[i] = {b.x * s * l[i], b.y * s * l[i]};
    }
    const double c0[3] = {m.cx[t], m.cy[t], m.cz[t]};
    const C AL = ca(ca(aL[0], aL[1]), aL[2]), AJ = ca(ca(aJ[0], aJ[1]), aJ[2]);
    const double rho = kr * eta / (4.0 * 3.14159265358979323846);   // E carries -j rho
    C g[3][3];
    for (int k = 0; k < 3; ++k)
        for (int x = 0; x < 3; ++x) g[k][x] = {0, 0};
    C YL[3] = {{0, 0}, {0, 0}, {0, 0}}, YJ[3] = {{0, 0}, {0, 0}, {0, 0}};
    for (int a = 0; a < 7; ++a) {
        const double da[3] = {m.qx[a * T + t], m.qy[a * T + t], m.qz[a * T + t]};
        const double wa = 0.5 * rule.w[a];
        C UL[3], UJ[3];
        for (int x = 0; x < 3; ++x) {
            UL[x] = UJ[x] = {0, 0};
            for (int i = 0; i < 3; ++i) {
                UL[x] = ca(UL[x], cs(aL[i], da[x] - u[i][x]));
                UJ[x] = ca(UJ[x], cs(aJ[i], da[x] - u[i][x]));
            }
        }
        // excitation field H_V = e0 pol exp(-j k khat . r) and grad_r (U.H_V)
        double sn, csn;
        sincos(-kr * (kx * (c0[0] + da[0]) + ky * (c0[1] + da[1]) + kz * (c0[2] + da[2])), &sn, &csn);
        const C ph = {e0 * csn, e0 * sn};
        C H[3] = {cs(ph, px), cs(ph, py), cs(ph, pz)};
        C UH = ca(ca(cm(UL[0], H[0]), cm(UL[1], H[1])), cm(UL[2], H[2]));
        C gradUH[3];
        const C mjk = {0.0, -kr};
        for (int x = 0; x < 3; ++x) gradUH[x] = cs(cm(UH, mjk), x == 0 ? kx : (x == 1 ? ky : kz));
        // radiation field E(r) = sum_dc W_dc (-j rho) e_dc exp(j k rhat . r): with U = U^j
        C Ef[3] = {{0, 0}, {0, 0}, {0, 0}};
        C gradUE[3] = {{0, 0}, {0, 0}, {0, 0}};
        for (int d = 0; d < ndir; ++d) {
            const double rx = dirs[3 * d], ry = dirs[3 * d + 1], rz = dirs[3 * d + 2];
            const double th = acos(fmin(1.0, fmax(-1.0, rz)));
            const double phv = atan2(ry, rx);
            double sth, cth, sph, cph;
            sincos(th, &sth, &cth);
            sincos(phv, &sph, &cph);
            const double et[3] = {cth * cph, cth * sph, -sth}, ep[3] = {-sph, cph, 0.0};
            double s2, c2;
            sincos(kr * (rx * (c0[0] + da[0]) + ry * (c0[1] + da[1]) + rz * (c0[2] + da[2])), &s2, &c2);
            // coefficient W_dc * (-j rho) * exp(j phase)
            const C ex = cm(C{c2, s2}, C{0.0, -rho});
            const double2 w0 = W[2 * d], w1 = W[2 * d + 1];
            const C wt = cm(C{w0.x, w0.y}, ex), wp = cm(C{w1.x, w1.y}, ex);
            C f[3];
            for (int x = 0; x < 3; ++x) f[x] = ca(cs(wt, et[x]), cs(wp, ep[x]));
            const C UE = ca(ca(cm(UJ[0], f[0]), cm(UJ[1], f[1])), cm(UJ[2], f[2]));
            for (int x = 0; x < 3; ++x) Ef[x] = ca(Ef[x], f[x]);
            const C jkU = cm(UE, C{0.0, kr});
            gradUE[0] = ca(gradUE[0], cs(jkU, rx));
            gradUE[1] = ca(gradUE[1], cs(jkU, ry));
            gradUE[2] = ca(gradUE[2], cs(jkU, rz));
        }
        for (int k = 0; k < 3; ++k) {
            const double lk = rule.bary[a][k];
            for (int x = 0; x < 3; ++x) {
                // (A0 l^a_k - alpha_k) H + l^a_k grad(U.H)
                C t1 = cs(cm(ca(cs(AL, lk), cs(aL[k], -1.0)), H[x]), wa);
                C t2 = cs(gradUH[x], wa * lk);
                C t3 = cs(cm(ca(cs(AJ, lk), cs(aJ[k], -1.0)), Ef[x]), wa);
                C t4 = cs(gradUE[x], wa * lk);
                g[k][x] = ca(g[k][x], ca(ca(t1, t2), ca(t3, t4)));
            }
        }
        for (int i = 0; i < 3; ++i)
            for (int x = 0; x < 3; ++x) {
                YL[i] = ca(YL[i], cs(H[x], wa * (da[x] - u[i][x])));
                YJ[i] = ca(YJ[i], cs(Ef[x], wa * (da[x] - u[i][x])));
            }
    }
    for (int k = 0; k < 3; ++k)
        for (int x = 0; x < 3; ++x) {
            C gg = g[k][x];
            for (int i = 0; i < 3; ++i) {
                double dl = 0.0;
                if (k == (i + 1) % 3) dl = e[i][x];
                else if (k == (i + 2) % 3) dl = -e[i][x];
                if (dl == 0.0) continue;
                gg = ca(gg, cm(YL[i], cs(aL[i], dl / l[i])));
                gg = ca(gg, cm(YJ[i], cs(aJ[i], dl / l[i])));
            }
            atomicAdd(&acc[size_t(t) * 9 + 3 * k + x], 2.0 * gg.r);
        }
}

__global__ void grad_scatter_kernel(DevMesh m, const double* __restrict__ acc, double* __restrict__ out) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m.T) return;
    for (int k = 0; k < 3; ++k) {
        const int v = m.tv[k * m.T + t];
        for (int x = 0; x < 3; ++x) atomicAdd(&out[3 * size_t(v) + x], acc[size_t(t) * 9 + 3 * k + x]);
    }
}

Rule radon_rule() {
    Rule r{};
    radon7(r.bary, r.w);
    return r;
}

}  // namespace efie

using namespace efie;

extern "C" int efie_vertex_grad_workspace_size(efie_mesh mesh, size_t* bytes) {
    return guarded([&]() {
        EFIE_REQUIRE(mesh && bytes, EFIE_ERR_ARG, "vertex_grad_workspace_size: null");
        *bytes = size_t(mesh->T) * 9 * sizeof(double);
        return int(EFIE_OK);
    });
}

extern "C" int efie_vertex_grad(efie_mesh mesh, double k, double eta, const void* J, const void* lambda,
                                const void* W, const double* dirs, int64_t ndir, const double* khat, const double* pol,
                                double e0, double* dxyz, void* ws, size_t ws_bytes, hipStream_t stream) {
    return guarded([&]() {
        EFIE_REQUIRE(mesh && J && lambda && W && dirs && khat && pol && dxyz && ws, EFIE_ERR_ARG,
                     "vertex_grad: null argument");
        EFIE_REQUIRE(mesh->dev != nullptr, EFIE_ERR_STATE, "vertex_grad: mesh tables not uploaded");
        EFIE_REQUIRE(mesh->far3 == 0.0, EFIE_ERR_ARG, "vertex_grad: differentiates the 7x7 rule only (far rule on)");
        EFIE_REQUIRE(k > 0.0 && std::isfinite(k) && ndir >= 1 && ndir < (int64_t(1) << 20), EFIE_ERR_ARG,
                     "vertex_grad: bad k or ndir");
        EFIE_REQUIRE(ws_bytes >= size_t(mesh->T) * 9 * sizeof(double), EFIE_ERR_ARG, "vertex_grad: ws too small");
        const DevMesh& m = mesh->dm;
        double* acc = static_cast<double*>(ws);
        fill_zero_bytes(acc, size_t(m.T) * 9 * sizeof(double), stream);
        fill_zero_bytes(dxyz, size_t(mesh->nv) * 3 * sizeof(double), stream);
        const Rule rule = radon_rule();
        const double f = eta / (4.0 * 3.14159265358979323846);
        Scale sc{};
        sc.ar = 0.0;
        sc.ai = f * k;
        sc.pr = 0.0;
        sc.pi = -f / k;
        const double2* lam = static_cast<const double2*>(lambda);
        const double2* jv = static_cast<const double2*>(J);
        const int nqblk = (m.T + 255) / 256;
        EFIE_REQUIRE(size_t(m.T) * nqblk < (size_t(1) << 31), EFIE_ERR_ARG, "vertex_grad: mesh too large");
        const double tpairs = double(m.T) * double(m.T) - double(m.n_near);
        prof_begin(PROF_GRAD_FAR, stream);
        hipLaunchKernelGGL(grad_far_kernel, dim3(unsigned(size_t(m.T) * nqblk)), dim3(256), 0, stream, m, k, sc, lam,
                           jv, acc, nqblk);
        prof_end(PROF_GRAD_FAR, stream, tpairs);
        if (m.n_near) {
            prof_begin(PROF_GRAD_NEAR, stream);
            hipLaunchKernelGGL(grad_near_kernel, dim3((m.n_near + 3) / 4), dim3(256), 0,
                               stream, m, sc, lam, jv, acc);
            prof_end(PROF_GRAD_NEAR, stream, double(m.n_near));
        }
        prof_begin(PROF_GRAD_TRI, stream);
        hipLaunchKernelGGL(grad_tri_kernel, dim3((m.T + 127) / 128), dim3(128), 0, stream, m, k, eta, rule, lam, jv,
                           static_cast<const double2*>(W), dirs, int(ndir), khat[0], khat[1], khat[2], pol[0], pol[1],
                           pol[2], e0, acc);
        prof_end(PROF_GRAD_TRI, stream, double(m.T));
        hipLaunchKernelGGL(grad_scatter_kernel, dim3((m.T + 127) / 128), dim3(128), 0, stream, m, acc, dxyz);
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}
