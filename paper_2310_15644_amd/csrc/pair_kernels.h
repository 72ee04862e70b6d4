// Device code shared by the single-mesh and the batched assembly kernels:
// Green's function evaluations, the far-pair moment accumulation, the
// closed-form potentials of the singular part and the near-pair blocks.
// (Formulas and readings are described in assemble.hip.)
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "efie_internal.h"
#include "phase_math.h"

namespace efie {

constexpr double PI = 3.14159265358979323846;
constexpr int FAR_BLOCK = 256;
constexpr int FAR_PB = 4;   // test triangles per block of the row-building far kernel

struct Scale {          // Z contribution = A * T_A + P * T_Phi (complex), or parts mode
    double ar, ai, pr, pi;
};

template <typename R>
struct Tables {
    const R *qx, *qy, *qz, *qw, *vx, *vy, *vz, *cf, *dv;
    const R *q3x, *q3y, *q3z;   // 3-point rule of the adaptive far rule (null: not used)
};

// Whether the far pair (p, q) takes the 3x3 rule: D^2 >= (far3 h)^2 with h the
// larger longest edge of the two triangles, all in FP64 without contraction (the
// same decision as the oracle's)
__device__ __forceinline__ bool far3_pair(const DevMesh& m, int p, int q) {
    const double dx = __dsub_rn(m.cx[q], m.cx[p]);
    const double dy = __dsub_rn(m.cy[q], m.cy[p]);
    const double dz = __dsub_rn(m.cz[q], m.cz[p]);
    const double d2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
    const double lim = __dmul_rn(m.far3, fmax(m.hm[p], m.hm[q]));
    return d2 >= __dmul_rn(lim, lim);
}

// Whether the pair (p, q) is near: the triangles share a vertex, or their
// centroids are closer than near_factor times the larger longest edge (decided
// as on the host, so that the device agrees with the ordered near-pair list).
__device__ __forceinline__ bool is_near(const DevMesh& m, int p, int q) {
    const int T = m.T;
    const int a0 = m.tv[p], a1 = m.tv[T + p], a2 = m.tv[2 * T + p];
    const int b0 = m.tv[q], b1 = m.tv[T + q], b2 = m.tv[2 * T + q];
    const bool share = (a0 == b0) | (a0 == b1) | (a0 == b2) | (a1 == b0) | (a1 == b1) | (a1 == b2) | (a2 == b0) |
                       (a2 == b1) | (a2 == b2);
    return share || near_by_distance(m.cx[p], m.cy[p], m.cz[p], m.cx[q], m.cy[q], m.cz[q], m.hm[p], m.hm[q], m.nf);
}

// ------------------------------------------------------------------ helpers
template <typename R>
__device__ __forceinline__ void atomic_add_c(void* Z, size_t idx, R re, R im);

template <>
__device__ __forceinline__ void atomic_add_c<double>(void* Z, size_t idx, double re, double im) {
    double* z = static_cast<double*>(Z) + 2 * idx;
    atomicAdd(z, re);
    atomicAdd(z + 1, im);
}
template <>
__device__ __forceinline__ void atomic_add_c<float>(void* Z, size_t idx, float re, float im) {
    float* z = static_cast<float*>(Z) + 2 * idx;
    atomicAdd(z, re);
    atomicAdd(z + 1, im);
}

// -------------------------------------------------------- far-pair kernel
// The 7-point rule in barycentric form.  Its points are the centroid and two orbits
// (1 - 2 b, b, b) and permutations; the weight times barycentric coordinate k of a
// point is then a constant, and the moments
//   M_kl = sum_ab w_a lambda_k(a) w_b lambda_l(b) G_ab
// take the sums of an orbit first (13 operations per seven Green's functions and
// part, against 28 with Cartesian moments and weights of the triangle).
template <int NP>
struct Bary;
template <>
struct Bary<7> {
    static constexpr double S15 = 3.872983346207417;
    static constexpr double W0 = 9.0 / 40.0, W1 = (155.0 + S15) / 1200.0, W2 = (155.0 - S15) / 1200.0;
    static constexpr double B1 = (6.0 + S15) / 21.0, B2 = (6.0 - S15) / 21.0;
    static constexpr double D1 = (9.0 - 2.0 * S15) / 21.0 - B1, D2 = (9.0 + 2.0 * S15) / 21.0 - B2;
    template <typename R>
    static __device__ __forceinline__ void fold(const R (&g)[7], R (&s)[3]) {
        const R o1 = g[1] + g[2] + g[3], o2 = g[4] + g[5] + g[6];
        const R t = R(W0 / 3.0) * g[0] + R(W1 * B1) * o1 + R(W2 * B2) * o2;
#pragma unroll
        for (int k = 0; k < 3; ++k) s[k] = t + R(W1 * D1) * g[1 + k] + R(W2 * D2) * g[4 + k];
    }
    static constexpr double coef(int a, int k) {   // weight of point a times its coordinate k
        return a == 0 ? W0 / 3.0 : (a < 4 ? W1 * (B1 + (k == a - 1 ? D1 : 0.0)) : W2 * (B2 + (k == a - 4 ? D2 : 0.0)));
    }
};
// the coefficients as a table, read with scalar loads by the (uniform) test point
template <int NP, typename R>
struct BaryTable {
    R c[NP][3];
    constexpr BaryTable() : c{} {
        for (int a = 0; a < NP; ++a)
            for (int k = 0; k < 3; ++k) c[a][k] = R(Bary<NP>::coef(a, k));
    }
};
template <int NP, typename R>
__device__ constexpr BaryTable<NP, R> bary_table{};

// Far pairs of near factor nf: the centroids are nf h apart, h the larger longest edge, and a
// point is up to D2 2/3 h = 0.47 h from its centroid, so that with nf >= 1.5 |o - s| >= 0.57 h and
// (|o| + |s|)^2 <= 6.9 |o - s|^2; with 2, the default, 3.5.  Below, triangles that share no vertex
// may be any fraction of h apart.
inline bool orbit_distances(double nf) { return nf >= 1.5; }

// The pair (p, q) of one mesh (not near): the NP x NP Green's function moments (NP = 7
// in barycentric form, 3) and the nine half-function products.  emit(i, j, zr, zi)
// receives the Z contribution of test edge i of p and source edge j of q (PARTS:
// zr, zi are the T_A part and emit2 gets the T_Phi part).
// (qx, qy, qz): the point offsets of the product rule, [NP][T].
// PRE: the source triangle's points come from pre[3][NP] already in registers
// instead of the tables
template <int NP, typename R, bool CK, bool PARTS, bool PRE = false, bool ORBIT = false, typename Emit, typename Emit2>
__device__ __forceinline__ void far_pair_rule(const DevMesh& m, const Tables<R>& tb, const R* __restrict__ qx,
                                              const R* __restrict__ qy, const R* __restrict__ qz, int p, int q,
                                              const Phase<R>& ph, const Scale& sc, Emit emit, Emit2 emit2,
                                              const R (*pre)[NP] = nullptr) {
    const int T = m.T;
    const R Dx = R(m.cx[p] - m.cx[q]);
    const R Dy = R(m.cy[p] - m.cy[q]);
    const R Dz = R(m.cz[p] - m.cz[q]);
    // ORBIT (7 points): the source points are D1 and D2 times the vertex offsets, so
    // that |o - s|^2 = |o|^2 + |s|^2 - 2 o.s takes 24 operations per test point, not 42.  It
    // loses (|o| + |s|)^2 / |o - s|^2 units of the last place: for meshes whose near factor
    // keeps the points of far pairs apart (orbit_distances).  For the FP64 rows of the Calderon build
    // (build at N = 7680: 153.2 -> 148.0 ms); the longer chain costs a matrix of 480
    // unknowns, which one wave per SIMD computes, 4 %, and FP32 keeps the differences
    static_assert(!ORBIT || NP == 7, "orbits of the 7-point rule");
    R sx[ORBIT ? 1 : NP], sy[ORBIT ? 1 : NP], sz[ORBIT ? 1 : NP], uo[3][3], c1[3], c2[3];
    if constexpr (ORBIT) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            uo[k][0] = tb.vx[k * T + q];
            uo[k][1] = tb.vy[k * T + q];
            uo[k][2] = tb.vz[k * T + q];
            const R u2 = uo[k][0] * uo[k][0] + uo[k][1] * uo[k][1] + uo[k][2] * uo[k][2];
            c1[k] = R(Bary<7>::D1 * Bary<7>::D1) * u2;
            c2[k] = R(Bary<7>::D2 * Bary<7>::D2) * u2;
        }
    } else {
#pragma unroll
        for (int b = 0; b < NP; ++b) {
            sx[b] = PRE ? pre[0][b] : qx[b * T + q];
            sy[b] = PRE ? pre[1][b] : qy[b * T + q];
            sz[b] = PRE ? pre[2][b] : qz[b * T + q];
        }
    }
    // nine half-function products from M0 = sum G, Md = sum G d_a, Md' = sum G d'_b and
    // Mdd' = sum G d_a . d'_b, weighted (d, d' the points' offsets from the centroids)
    R m0r = 0, m0i = 0, mmr = 0, mmi = 0;
    R mdr[3] = {0, 0, 0}, mdi[3] = {0, 0, 0}, mpr[3] = {0, 0, 0}, mpi[3] = {0, 0, 0};
    R up[3][3], uq[3][3], cq[3], gq[3];
    // the areas' product (and the weights, equal, of the 3-point rule)
    const R area2 = (tb.qw[p] * tb.qw[q]) * R((NP == 3 ? 1.0 / 9.0 : 1.0) / (Bary<7>::W0 * Bary<7>::W0));
    auto corners = [&]() {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            uq[j][0] = tb.vx[j * T + q];
            uq[j][1] = tb.vy[j * T + q];
            uq[j][2] = tb.vz[j * T + q];
            cq[j] = tb.cf[j * T + q] * area2;
            gq[j] = tb.dv[j * T + q] * area2;
            up[j][0] = tb.vx[j * T + p];
            up[j][1] = tb.vy[j * T + p];
            up[j][2] = tb.vz[j * T + p];
        }
    };
    if constexpr (NP == 3) {
        // equal weights: sums over a point's row and column of the 3 x 3 table, 111
        // operations where folds into M_kl take 200
        R cr[3] = {0, 0, 0}, ci[3] = {0, 0, 0};
#pragma unroll 1
        for (int a = 0; a < 3; ++a) {
            const R ax = qx[a * T + p], ay = qy[a * T + p], az = qz[a * T + p];
            const R ox = Dx + ax, oy = Dy + ay, oz = Dz + az;
            R rr = 0, ri = 0;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const R dx = ox - sx[b], dy = oy - sy[b], dz = oz - sz[b];
                R gr, gi;
                green_far(ph, CK, dx * dx + dy * dy + dz * dz, gr, gi);
                rr += gr;
                ri += gi;
                cr[b] += gr;
                ci[b] += gi;
                const R dot = ax * sx[b] + ay * sy[b] + az * sz[b];
                mmr += gr * dot;
                mmi += gi * dot;
            }
            m0r += rr;
            m0i += ri;
            const R av[3] = {ax, ay, az};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                mdr[d] += rr * av[d];
                mdi[d] += ri * av[d];
            }
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const R sv[3] = {sx[b], sy[b], sz[b]};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                mpr[d] += cr[b] * sv[d];
                mpi[d] += ci[b] * sv[d];
            }
        }
        corners();
    } else {
        R Mr[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, Mi[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll 1
        for (int a = 0; a < 7; ++a) {
            const R ox = Dx + qx[a * T + p], oy = Dy + qy[a * T + p], oz = Dz + qz[a * T + p];
            R gr[7], gi[7];
            if constexpr (ORBIT) {
                const R o2 = ox * ox + oy * oy + oz * oz;
                green_far(ph, CK, o2, gr[0], gi[0]);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const R t = ox * uo[k][0] + oy * uo[k][1] + oz * uo[k][2];
                    green_far(ph, CK, fma(R(-2.0 * Bary<7>::D1), t, o2 + c1[k]), gr[1 + k], gi[1 + k]);
                    green_far(ph, CK, fma(R(-2.0 * Bary<7>::D2), t, o2 + c2[k]), gr[4 + k], gi[4 + k]);
                }
            } else {
#pragma unroll
                for (int b = 0; b < 7; ++b) {
                    const R dx = ox - sx[b], dy = oy - sy[b], dz = oz - sz[b];
                    green_far(ph, CK, dx * dx + dy * dy + dz * dz, gr[b], gi[b]);
                }
            }
            R sr[3], si[3];
            Bary<7>::fold(gr, sr);
            Bary<7>::fold(gi, si);
            const R(&ca)[3] = bary_table<7, R>.c[a];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int l = 0; l < 3; ++l) {
                    Mr[k][l] += ca[k] * sr[l];
                    Mi[k][l] += ca[k] * si[l];
                }
        }
        corners();
        // offsets as barycentric sums of the vertex offsets
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const R rr = Mr[k][0] + Mr[k][1] + Mr[k][2], ri = Mi[k][0] + Mi[k][1] + Mi[k][2];
            const R cr = Mr[0][k] + Mr[1][k] + Mr[2][k], ci = Mi[0][k] + Mi[1][k] + Mi[2][k];
            m0r += rr;
            m0i += ri;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                mdr[d] += rr * up[k][d];
                mdi[d] += ri * up[k][d];
                mpr[d] += cr * uq[k][d];
                mpi[d] += ci * uq[k][d];
            }
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                const R dot = up[k][0] * uq[l][0] + up[k][1] * uq[l][1] + up[k][2] * uq[l][2];
                mmr += Mr[k][l] * dot;
                mmi += Mi[k][l] * dot;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const R ux = up[i][0], uy = up[i][1], uz = up[i][2];
        const R ci = tb.cf[i * T + p], gi_ = tb.dv[i * T + p];
        // terms that depend on i only
        const R bir = mmr - (ux * mpr[0] + uy * mpr[1] + uz * mpr[2]);
        const R bii = mmi - (ux * mpi[0] + uy * mpi[1] + uz * mpi[2]);
        const R er[3] = {mdr[0] - ux * m0r, mdr[1] - uy * m0r, mdr[2] - uz * m0r};
        const R ei[3] = {mdi[0] - ux * m0i, mdi[1] - uy * m0i, mdi[2] - uz * m0i};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            // Mdd' - u_i.Md' - u'_j.(Md - u_i M0)
            const R tar = ci * cq[j] * (bir - (uq[j][0] * er[0] + uq[j][1] * er[1] + uq[j][2] * er[2]));
            const R tai = ci * cq[j] * (bii - (uq[j][0] * ei[0] + uq[j][1] * ei[1] + uq[j][2] * ei[2]));
            const R gg = gi_ * gq[j];
            const R tpr = gg * m0r, tpi = gg * m0i;
            if (PARTS) {
                emit(i, j, tar * R(sc.ar), tai * R(sc.ar));
                emit2(i, j, tpr * R(sc.ar), tpi * R(sc.ar));
            } else {
                const R zr = R(sc.ar) * tar - R(sc.ai) * tai + R(sc.pr) * tpr - R(sc.pi) * tpi;
                const R zi = R(sc.ar) * tai + R(sc.ai) * tar + R(sc.pr) * tpi + R(sc.pi) * tpr;
                emit(i, j, zr, zi);
            }
        }
    }
}

// The far pair (p, q) by the 7x7 rule, or by the 3x3 rule where the adaptive far
// rule is on (m.far3 > 0) and the pair is far enough.
template <typename R, bool CK, bool PARTS, bool ORBIT = false, typename Emit, typename Emit2>
__device__ __forceinline__ void far_pair_emit(const DevMesh& m, const Tables<R>& tb, int p, int q, const Phase<R>& ph,
                                              const Scale& sc, Emit emit, Emit2 emit2) {
    if (m.far3 > 0.0 && far3_pair(m, p, q))
        far_pair_rule<3, R, CK, PARTS>(m, tb, tb.q3x, tb.q3y, tb.q3z, p, q, ph, sc, emit, emit2);
    else
        far_pair_rule<NQ, R, CK, PARTS, false, ORBIT>(m, tb, tb.qx, tb.qy, tb.qz, p, q, ph, sc, emit, emit2);
}

// The pair (p, q) added to Z (and Z2 in parts mode) with atomics; near pairs skipped.
template <typename R, bool CK, bool PARTS>
__device__ __forceinline__ void far_pair(const DevMesh& m, const Tables<R>& tb, int p, int q, const Phase<R>& ph,
                                         const Scale& sc, void* Z, void* Z2) {
    const int T = m.T;
    if (is_near(m, p, q)) return;
    const size_t N = size_t(m.N);
    auto at = [&](void* dst) {
        return [=, &m](int i, int j, R re, R im) {
            atomic_add_c<R>(dst, size_t(m.te[i * T + p]) * N + size_t(m.te[j * T + q]), re, im);
        };
    };
    far_pair_emit<R, CK, PARTS>(m, tb, p, q, ph, sc, at(Z), at(Z2));
}

// ----------------------------------------------------- closed-form potentials
// I0 = int 1/|r - r'| dS' and I1 = int (rho' - rho)/|r - r'| dS' over the flat
// triangle with vertex positions u[0..2] (counter-clockwise about the unit normal
// n); r, u relative to the same origin.  Edge-sum formulas of Wilton et al. 1984.
static __device__ void potentials(const double r[3], const double u[3][3], const double n[3], double h, double& I0,
                           double I1[3]) {
    const double d = n[0] * (r[0] - u[0][0]) + n[1] * (r[1] - u[0][1]) + n[2] * (r[2] - u[0][2]);
    const double ad = fabs(d);
    const double rho[3] = {r[0] - d * n[0], r[1] - d * n[1], r[2] - d * n[2]};
    I0 = 0.0;
    I1[0] = I1[1] = I1[2] = 0.0;
#pragma unroll 1
    for (int e = 0; e < 3; ++e) {
        const double* rm = u[e];
        const double* rp = u[(e + 1) % 3];
        double lt[3] = {rp[0] - rm[0], rp[1] - rm[1], rp[2] - rm[2]};
        const double il = rsqrt_fast(lt[0] * lt[0] + lt[1] * lt[1] + lt[2] * lt[2]);
        lt[0] *= il; lt[1] *= il; lt[2] *= il;
        const double uu[3] = {lt[1] * n[2] - lt[2] * n[1], lt[2] * n[0] - lt[0] * n[2], lt[0] * n[1] - lt[1] * n[0]};
        const double lp = (rp[0] - rho[0]) * lt[0] + (rp[1] - rho[1]) * lt[1] + (rp[2] - rho[2]) * lt[2];
        const double lm = (rm[0] - rho[0]) * lt[0] + (rm[1] - rho[1]) * lt[1] + (rm[2] - rho[2]) * lt[2];
        const double P0 = (rm[0] - rho[0]) * uu[0] + (rm[1] - rho[1]) * uu[1] + (rm[2] - rho[2]) * uu[2];
        const double R02 = P0 * P0 + d * d;
        const double Rp = root_fast((r[0] - rp[0]) * (r[0] - rp[0]) + (r[1] - rp[1]) * (r[1] - rp[1]) +
                                    (r[2] - rp[2]) * (r[2] - rp[2]));
        const double Rm = root_fast((r[0] - rm[0]) * (r[0] - rm[0]) + (r[1] - rm[1]) * (r[1] - rm[1]) +
                                    (r[2] - rm[2]) * (r[2] - rm[2]));
        double lg = 0.0, at = 0.0;
        if (R02 >= 1e-24 * h * h) {
            // fp / fm, f = R + l, written as R0^2 / (R - l) for l < 0 (same value, no cancellation)
            const double sp = Rp + fabs(lp), sm = Rm + fabs(lm);
            const double num = (lp >= 0.0 ? sp : R02) * (lm >= 0.0 ? 1.0 : sm);
            const double den = (lp >= 0.0 ? 1.0 : sp) * (lm >= 0.0 ? sm : R02);
            lg = log(num * rcp_fast(den));
            at = atan(P0 * lp * rcp_fast(R02 + ad * Rp)) - atan(P0 * lm * rcp_fast(R02 + ad * Rm));
        }
        I0 += P0 * lg - ad * at;
        const double c1 = 0.5 * (R02 * lg + lp * Rp - lm * Rm);
        I1[0] += c1 * uu[0];
        I1[1] += c1 * uu[1];
        I1[2] += c1 * uu[2];
    }
}

// Test point a of the singular block X(i,j) = sum_a W_a f_i(r_a) . int_s f_j(r')/R dS'
// and of the scalar s0 = sum_a W_a int_s 1/R dS' (test triangle t, source triangle
// s): w times that point's terms added to Y[i][j] and to s0.
static __device__ void singular_point(const DevMesh& m, int t, int s, int a, double w, double Y[3][3], double& s0) {
    const int T = m.T;
    // everything relative to the source centroid
    const double D[3] = {m.cx[t] - m.cx[s], m.cy[t] - m.cy[s], m.cz[t] - m.cz[s]};
    double us[3][3];
    for (int k = 0; k < 3; ++k) {
        us[k][0] = m.vx[k * T + s]; us[k][1] = m.vy[k * T + s]; us[k][2] = m.vz[k * T + s];
    }
    const double n[3] = {m.nx[s], m.ny[s], m.nz[s]};
    const double da[3] = {m.qx[a * T + t], m.qy[a * T + t], m.qz[a * T + t]};
    const double wa = w * m.qw[a * T + t];
    const double r[3] = {D[0] + da[0], D[1] + da[1], D[2] + da[2]};
    double I0, I1[3];
    potentials(r, us, n, m.hm[s], I0, I1);
    const double dd = n[0] * (r[0] - us[0][0]) + n[1] * (r[1] - us[0][1]) + n[2] * (r[2] - us[0][2]);
    const double rho[3] = {r[0] - dd * n[0], r[1] - dd * n[1], r[2] - dd * n[2]};
    s0 += wa * I0;
    double inner[3][3];
    for (int j = 0; j < 3; ++j) {
        const double cs = m.cf[j * T + s];
        for (int x = 0; x < 3; ++x) inner[j][x] = cs * (I1[x] + (rho[x] - us[j][x]) * I0);
    }
    for (int i = 0; i < 3; ++i) {
        const double ct = m.cf[i * T + t];
        const double f[3] = {ct * (da[0] - m.vx[i * T + t]), ct * (da[1] - m.vy[i * T + t]),
                             ct * (da[2] - m.vz[i * T + t])};
        for (int j = 0; j < 3; ++j) {
            const double v = wa * (f[0] * inner[j][0] + f[1] * inner[j][1] + f[2] * inner[j][2]);
            Y[i][j] += v;
        }
    }
}

// (exp(-jkR) - 1)/R with exp(z) - 1 = expm1(x) cos y - 2 sin^2(y/2) + j exp(x) sin y,
// z = -j k R = x + j y; value -j k at R = 0.
static __device__ __forceinline__ void green_smooth(const Phase<double>& ph, double kr, double ki, double R2,
                                                    double& gr, double& gi) {
    if (R2 == 0.0) {
        gr = ki;
        gi = -kr;
        return;
    }
    const double rinv = rsqrt_fast(R2);
    const double R = R2 * rinv;
    double s2, c2;
    sincos_quarter(R, -0.5 * ph.khi, -0.5 * ph.klo, s2, c2);   // of y / 2
    const double siny = 2.0 * s2 * c2;
    double nr = -2.0 * s2 * s2, ni = siny;
    if (ki != 0.0) {   // uniform over the launch
        const double x = ki * R;
        nr = expm1(x) * (1.0 + nr) + nr;
        ni *= exp2_scaled(R, ph.ehi, ph.elo);
    }
    gr = nr * rinv;
    gi = ni * rinv;
}

// Near pair e of the ordered list, computed by a group of NEAR_G = 16 consecutive
// lanes (g = 0..15 its lane in the group; every lane of the group calls this with
// the same valid e): lane g with a = g % 8 < 7 takes test point a, the lower half of
// the group p's point in the singular block of p against q and columns 0 to 3 of the
// smooth part's row a of the 7 x 7 rule, the upper half q's point against p and
// columns 4 to 6, so all lanes of a wave run the same code.  The moments are summed
// over the group with a butterfly of lane exchanges (a fixed order: deterministic),
// then lane g < 9 emits entry 3 i + j = g: emit(i, j, zr, zi) receives the FP64 Z
// contribution of test edge i and source edge j (PARTS: T_A part; emit2: T_Phi).
// Bound by memory latency and a lane's chain of dependent operations for small meshes
// (FP64 blocks alone, N = 480: 29 us, of which 18 for a single wave), by the vector ALU
// for large ones (N = 7680: 134 us).  150 registers, three waves per SIMD, where both
// blocks on each of 8 lanes and the library's roots and quotients took 213 (30 and 137 us).
constexpr int NEAR_G = 16;

template <bool PARTS, typename Emit, typename Emit2>
__device__ void near_pair_group(const DevMesh& m, int e, int g, double kr, double ki, const Scale& sc, Emit emit,
                                Emit2 emit2) {
    const int p = m.near_p[e], q = m.near_q[e];
    const int T = m.T;
    // v: the smooth part's moments as in the far kernel (offsets from the centroids)
    //   [0,1] M0, [2..7] Md (re, im per axis), [8..13] Md', [14,15] Mdd';
    // Y = (X_pq + X_qp^T) / 2 of the singular part, and s0 its scalar
    double v[16];
    for (int x = 0; x < 16; ++x) v[x] = 0.0;
    double Y[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    double s0 = 0.0;
    const int a = g & 7;
    const bool upper = g >= 8;
    if (a < NQ) {
        const double D[3] = {m.cx[p] - m.cx[q], m.cy[p] - m.cy[q], m.cz[p] - m.cz[q]};
        const double ax = m.qx[a * T + p], ay = m.qy[a * T + p], az = m.qz[a * T + p], wa = m.qw[a * T + p];
        double s0r = 0, s0i = 0, s1r[3] = {0, 0, 0}, s1i[3] = {0, 0, 0};
        const Phase<double> ph = make_phase<double>(kr, ki);
#pragma unroll 1
        for (int c = 0; c < 4; ++c) {   // the upper half's eighth column repeats the seventh with weight 0
            const int b = min(upper ? 4 + c : c, NQ - 1);
            const double bx = m.qx[b * T + q], by = m.qy[b * T + q], bz = m.qz[b * T + q];
            const double wb = upper && c == 3 ? 0.0 : m.qw[b * T + q];
            const double dx = D[0] + ax - bx, dy = D[1] + ay - by, dz = D[2] + az - bz;
            double gr, gi;
            green_smooth(ph, kr, ki, dx * dx + dy * dy + dz * dz, gr, gi);
            gr *= wb;
            gi *= wb;
            s0r += gr; s0i += gi;
            s1r[0] += gr * bx; s1i[0] += gi * bx;
            s1r[1] += gr * by; s1i[1] += gi * by;
            s1r[2] += gr * bz; s1i[2] += gi * bz;
        }
        const double av[3] = {ax, ay, az};
        v[0] = wa * s0r;
        v[1] = wa * s0i;
        for (int d = 0; d < 3; ++d) {
            v[2 + 2 * d] = wa * av[d] * s0r;
            v[3 + 2 * d] = wa * av[d] * s0i;
            v[8 + 2 * d] = wa * s1r[d];
            v[9 + 2 * d] = wa * s1i[d];
        }
        v[14] = wa * (ax * s1r[0] + ay * s1r[1] + az * s1r[2]);
        v[15] = wa * (ax * s1i[0] + ay * s1i[1] + az * s1i[2]);
        // singular part, symmetrised: (X_pq + X_qp^T) / 2
        double X[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
        singular_point(m, upper ? q : p, upper ? p : q, a, 0.5, X, s0);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) Y[i][j] = upper ? X[j][i] : X[i][j];
    }
#pragma unroll
    for (int o = 1; o < NEAR_G; o <<= 1) {
#pragma unroll
        for (int x = 0; x < 16; ++x) v[x] += __shfl_xor(v[x], o, NEAR_G);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) Y[i][j] += __shfl_xor(Y[i][j], o, NEAR_G);
        s0 += __shfl_xor(s0, o, NEAR_G);
    }
    const double m0r = v[0], m0i = v[1];
    if (g < 9) {
        const int i = g / 3, j = g - 3 * i;
        const double ux = m.vx[i * T + p], uy = m.vy[i * T + p], uz = m.vz[i * T + p];
        const double ci = m.cf[i * T + p], gi_ = m.dv[i * T + p];
        const double vx = m.vx[j * T + q], vy = m.vy[j * T + q], vz = m.vz[j * T + q];
        const double cj = m.cf[j * T + q], gj = m.dv[j * T + q];
        const double br = v[14] - (ux * v[8] + uy * v[10] + uz * v[12]) -
                          (vx * (v[2] - ux * m0r) + vy * (v[4] - uy * m0r) + vz * (v[6] - uz * m0r));
        const double bi = v[15] - (ux * v[9] + uy * v[11] + uz * v[13]) -
                          (vx * (v[3] - ux * m0i) + vy * (v[5] - uy * m0i) + vz * (v[7] - uz * m0i));
        const double tar = ci * cj * br + Y[i][j];
        const double tai = ci * cj * bi;
        const double gg = gi_ * gj;
        const double tpr = gg * (m0r + s0), tpi = gg * m0i;
        if (PARTS) {
            emit(i, j, tar * sc.ar, tai * sc.ar);
            emit2(i, j, tpr * sc.ar, tpi * sc.ar);
        } else {
            const double zr = sc.ar * tar - sc.ai * tai + sc.pr * tpr - sc.pi * tpi;
            const double zi = sc.ar * tai + sc.ai * tar + sc.pr * tpi + sc.pi * tpr;
            emit(i, j, zr, zi);
        }
    }
}

// near pair e added to Z (and Z2 in parts mode) with atomics, in ZT precision (by
// the group of NEAR_G lanes, lane g)
template <typename ZT, bool PARTS>
__device__ void near_pair(const DevMesh& m, int e, int g, double kr, double ki, const Scale& sc, void* Z, void* Z2) {
    const int p = m.near_p[e], q = m.near_q[e];
    const int T = m.T;
    const size_t N = size_t(m.N);
    auto at = [&](void* dst) {
        return [=, &m](int i, int j, double re, double im) {
            atomic_add_c<ZT>(dst, size_t(m.te[i * T + p]) * N + size_t(m.te[j * T + q]), ZT(re), ZT(im));
        };
    };
    near_pair_group<PARTS>(m, e, g, kr, ki, sc, at(Z), at(Z2));
}

}  // namespace efie
