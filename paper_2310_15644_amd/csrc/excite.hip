// Plane-wave excitation and far-field radiation on gfx950.
//
//   V[s][m] = int f_m . E0 pol_s exp(-j k khat_s . r) dS            (7-point rule)
//   F[s][d] = -(j k eta / 4 pi) (I - rhat rhat) . sum_n J[s][n] a_n(rhat_d),
//   a_n(rhat) = int f_n(r') exp(j k rhat . r') dS'                  (7-point rule)
// The far field is formed in two steps: a radiation matrix whose row 2d+c holds
// the (theta, phi)[c] component of -(j k eta/4 pi) a_n(rhat_d) for every n, then
// F = J R^T with the tiled complex GEMM (FP64), so F comes out as (nrhs, ndir, 2).
#include <hip/hip_runtime.h>

#include <cmath>

#include "efie_internal.h"
#include "linalg.h"
#include "pair_kernels.h"
#include "phase_math.h"

namespace efie {

// One triangle of an RWG: centroid c, vertex offsets u from it, the offset ui of the
// vertex opposite the edge, w = s l / (2 A) times the triangle's area.
struct HalfRwg {
    double c[3], u[3][3], ui[3], w;
};
__device__ __forceinline__ HalfRwg half_rwg(const DevMesh& m, int n, int h) {
    const int T = m.T, t = m.et[h * m.N + n], l = m.el[h * m.N + n];
    HalfRwg r;
    r.c[0] = m.cx[t];
    r.c[1] = m.cy[t];
    r.c[2] = m.cz[t];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r.u[k][0] = m.vx[k * T + t];
        r.u[k][1] = m.vy[k * T + t];
        r.u[k][2] = m.vz[k * T + t];
    }
    r.ui[0] = m.vx[l * T + t];
    r.ui[1] = m.vy[l * T + t];
    r.ui[2] = m.vz[l * T + t];
    r.w = m.cf[l * T + t] * m.qw[t] * (1.0 / Bary<7>::W0);   // point 0's weight is W0 times the area
    return r;
}
// E_l = sum_a w_a lambda_l(a) exp(j k d . r_a) over the 7-point rule: the phases of the
// points are the centroid's and D1 or D2 times a vertex's (Bary in pair_kernels.h)
__device__ __forceinline__ void wave_moments(const HalfRwg& r, const Phase<double>& ph, double dx, double dy, double dz,
                                             double (&er)[3], double (&ei)[3]) {
    const double p0 = dx * r.c[0] + dy * r.c[1] + dz * r.c[2];
    double cs[7], sn[7];
    sincos_quarter(p0, ph.khi, ph.klo, sn[0], cs[0]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double pu = dx * r.u[k][0] + dy * r.u[k][1] + dz * r.u[k][2];
        sincos_quarter(p0 + Bary<7>::D1 * pu, ph.khi, ph.klo, sn[1 + k], cs[1 + k]);
        sincos_quarter(p0 + Bary<7>::D2 * pu, ph.khi, ph.klo, sn[4 + k], cs[4 + k]);
    }
    Bary<7>::fold(cs, er);
    Bary<7>::fold(sn, ei);
}
// w sum_l E_l (u_l - ui) . e, added to (ar, ai)
__device__ __forceinline__ void add_component(const HalfRwg& r, const double (&er)[3], const double (&ei)[3], double ex,
                                              double ey, double ez, double& ar, double& ai) {
    double vr = 0.0, vi = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double f = (r.u[k][0] - r.ui[0]) * ex + (r.u[k][1] - r.ui[1]) * ey + (r.u[k][2] - r.ui[2]) * ez;
        vr += er[k] * f;
        vi += ei[k] * f;
    }
    ar += r.w * vr;
    ai += r.w * vi;
}

// A thread takes one RWG and a block's WAVE_ND directions (uniform: scalar loads), so that
// the RWG's tables are read once for all of them; one direction per block where that
// leaves too few blocks (wave_dirs).  Bound by the vector ALU: 14 sines and cosines
// per value, about 550 FP64 operations.  N = 7680, 512 directions: excitation 182 us
// and radiation matrix 200 us with a thread per value, 82 and 90 us now.
constexpr int WAVE_ND = 8;
inline int wave_dirs(int64_t N, int64_t ndir) { return (N + 255) / 256 * (ndir / WAVE_ND) >= 512 ? WAVE_ND : 1; }
// blocks: those of the RWGs for the first nd directions, then for the next
inline dim3 wave_grid(int64_t N, int64_t ndir, int nd) {
    return dim3(unsigned((N + 255) / 256 * ((ndir + nd - 1) / nd)));
}

__global__ __launch_bounds__(256) void excite_kernel(DevMesh m, double k, const double* __restrict__ khat,
                                                     const double* __restrict__ pol, int nrhs, double e0, int nd,
                                                     double2* __restrict__ V) {
    const int N = m.N, nb = (N + 255) / 256;
    const int g = int(blockIdx.x) / nb, n = (int(blockIdx.x) - g * nb) * 256 + int(threadIdx.x);
    if (n >= N) return;
    const Phase<double> ph = make_phase<double>(-k, 0.0);
    const HalfRwg a = half_rwg(m, n, 0), b = half_rwg(m, n, 1);
    const int s1 = min(nrhs, (g + 1) * nd);
    for (int s = g * nd; s < s1; ++s) {
        double vr = 0.0, vi = 0.0, er[3], ei[3];
        wave_moments(a, ph, khat[3 * s], khat[3 * s + 1], khat[3 * s + 2], er, ei);
        add_component(a, er, ei, pol[3 * s], pol[3 * s + 1], pol[3 * s + 2], vr, vi);
        wave_moments(b, ph, khat[3 * s], khat[3 * s + 1], khat[3 * s + 2], er, ei);
        add_component(b, er, ei, pol[3 * s], pol[3 * s + 1], pol[3 * s + 2], vr, vi);
        V[size_t(s) * N + n] = make_double2(e0 * vr, e0 * vi);
    }
}

// radiation matrix R[2d + c][n] = -(j k eta / 4 pi) e_c(rhat_d) . a_n(rhat_d)
__global__ __launch_bounds__(256) void radiation_kernel(DevMesh m, double k, double eta, const double* __restrict__ dirs,
                                                        int ndir, int nd, double2* __restrict__ Rm) {
    __shared__ double sph[WAVE_ND][5];   // theta and phi unit vectors (the last z is 0)
    const int N = m.N, nb = (N + 255) / 256;
    const int g = int(blockIdx.x) / nb, n = (int(blockIdx.x) - g * nb) * 256 + int(threadIdx.x);
    const int d0 = g * nd, d1 = min(ndir, d0 + nd);
    if (d0 + int(threadIdx.x) < d1) {
        const int d = d0 + int(threadIdx.x);
        const double th = acos(fmin(1.0, fmax(-1.0, dirs[3 * d + 2])));
        const double phv = atan2(dirs[3 * d + 1], dirs[3 * d]);
        double st, ct, sp, cp;
        sincos(th, &st, &ct);
        sincos(phv, &sp, &cp);
        double* q = sph[threadIdx.x];
        q[0] = ct * cp;
        q[1] = ct * sp;
        q[2] = -st;
        q[3] = -sp;
        q[4] = cp;
    }
    __syncthreads();
    if (n >= N) return;
    const Phase<double> ph = make_phase<double>(k, 0.0);
    const HalfRwg a = half_rwg(m, n, 0), b = half_rwg(m, n, 1);
    // times -(j k eta / 4 pi): (a_r + j a_i) * (-j c) = c a_i - j c a_r
    const double cc = k * eta / (4.0 * 3.14159265358979323846);
    for (int d = d0; d < d1; ++d) {
        const double* q = sph[d - d0];
        double tr = 0.0, ti = 0.0, pr = 0.0, pi = 0.0, er[3], ei[3];
        wave_moments(a, ph, dirs[3 * d], dirs[3 * d + 1], dirs[3 * d + 2], er, ei);
        add_component(a, er, ei, q[0], q[1], q[2], tr, ti);
        add_component(a, er, ei, q[3], q[4], 0.0, pr, pi);
        wave_moments(b, ph, dirs[3 * d], dirs[3 * d + 1], dirs[3 * d + 2], er, ei);
        add_component(b, er, ei, q[0], q[1], q[2], tr, ti);
        add_component(b, er, ei, q[3], q[4], 0.0, pr, pi);
        Rm[size_t(2 * d) * N + n] = make_double2(cc * ti, -cc * tr);
        Rm[size_t(2 * d + 1) * N + n] = make_double2(cc * pi, -cc * pr);
    }
}

// adjoint source of the far field: G[s][n] = sum_e W[s][e] R[e][n], R the
// radiation matrix (2 ndir x N, row 2d + c) that forms F = J R^T
__global__ __launch_bounds__(256) void radiation_adjoint_kernel(const double2* __restrict__ Rm,
                                                                const double2* __restrict__ W, int ne, int N, int nrhs,
                                                                double2* __restrict__ G) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    const int s = blockIdx.y;
    if (n >= N || s >= nrhs) return;
    double gr = 0.0, gi = 0.0;
    for (int e = 0; e < ne; ++e) {
        const double2 r = Rm[size_t(e) * N + n], w = W[size_t(s) * ne + e];
        gr += r.x * w.x - r.y * w.y;
        gi += r.x * w.y + r.y * w.x;
    }
    G[size_t(s) * N + n] = make_double2(gr, gi);
}

// J = sum_i |F_i|^2 over count far-field values, and W = conj(F) (its derivative
// with respect to F, the weight of the adjoint source).  One block: each thread
// sums a fixed stride of the values, then a fixed tree over the block, so the sum
// is the same on every call.
__global__ __launch_bounds__(256) void farfield_objective_kernel(const double2* __restrict__ F, int64_t count,
                                                                 double* __restrict__ J, double2* __restrict__ W) {
    __shared__ double sh[256];
    double a = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += 256) {
        const double2 f = F[i];
        a += f.x * f.x + f.y * f.y;
        if (W) W[i] = make_double2(f.x, -f.y);
    }
    sh[threadIdx.x] = a;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (int(threadIdx.x) < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *J = sh[0];
}

}  // namespace efie

extern "C" int efie_excite_planewave(efie_mesh mesh, double k, const double* khat, const double* pol, int64_t nrhs,
                                     double e0, void* V, hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(mesh && khat && pol && V, EFIE_ERR_ARG, "excite: null argument");
        EFIE_REQUIRE(mesh->dev != nullptr, EFIE_ERR_STATE, "excite: mesh tables not uploaded");
        EFIE_REQUIRE(nrhs >= 1 && nrhs * mesh->N < (int64_t(1) << 31), EFIE_ERR_ARG, "excite: bad nrhs");
        const int nd = efie::wave_dirs(mesh->N, nrhs);
        efie::prof_begin(efie::PROF_EXCITE, stream);
        hipLaunchKernelGGL(efie::excite_kernel, efie::wave_grid(mesh->N, nrhs, nd), dim3(256), 0, stream, mesh->dm, k,
                           khat, pol, int(nrhs), e0, nd, static_cast<double2*>(V));
        efie::prof_end(efie::PROF_EXCITE, stream);
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}

extern "C" int efie_farfield_workspace_size(efie_mesh mesh, int64_t ndir, size_t* bytes) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(mesh && bytes && ndir >= 1, EFIE_ERR_ARG, "farfield_workspace_size: bad argument");
        *bytes = size_t(2 * ndir) * size_t(mesh->N) * 16;
        return int(EFIE_OK);
    });
}

extern "C" int efie_farfield(efie_mesh mesh, double k, double eta, const void* J, int64_t nrhs, const double* dirs,
                             int64_t ndir, void* F, void* ws, size_t ws_bytes, hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(mesh && J && dirs && F && ws, EFIE_ERR_ARG, "farfield: null argument");
        EFIE_REQUIRE(mesh->dev != nullptr, EFIE_ERR_STATE, "farfield: mesh tables not uploaded");
        EFIE_REQUIRE(nrhs >= 1 && ndir >= 1 && nrhs < 65536 && 2 * ndir * mesh->N < (int64_t(1) << 31),
                     EFIE_ERR_ARG, "farfield: bad sizes");
        EFIE_REQUIRE(ws_bytes >= size_t(2 * ndir) * size_t(mesh->N) * 16, EFIE_ERR_ARG, "farfield: workspace too small");
        const int N = int(mesh->N);
        const int nd = efie::wave_dirs(N, ndir);
        efie::prof_begin(efie::PROF_FARFIELD, stream);
        hipLaunchKernelGGL(efie::radiation_kernel, efie::wave_grid(N, ndir, nd), dim3(256), 0, stream, mesh->dm, k, eta,
                           dirs, int(ndir), nd, static_cast<double2*>(ws));
        efie::prof_end(efie::PROF_FARFIELD, stream);
        // F[s][e] = sum_n J[s][n] R[e][n]
        efie::zgemm_nt(J, EFIE_C128, ws, EFIE_C128, F, EFIE_C128, int(nrhs), int(2 * ndir), N, N, N, int(2 * ndir),
                       1.0, 0.0, false, stream);
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}

extern "C" int efie_farfield_adjoint(efie_mesh mesh, double k, double eta, const void* W, int64_t nrhs,
                                     const double* dirs, int64_t ndir, void* G, void* ws, size_t ws_bytes,
                                     hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(mesh && W && dirs && G && ws, EFIE_ERR_ARG, "farfield_adjoint: null argument");
        EFIE_REQUIRE(mesh->dev != nullptr, EFIE_ERR_STATE, "farfield_adjoint: mesh tables not uploaded");
        EFIE_REQUIRE(nrhs >= 1 && ndir >= 1 && nrhs < 65536 && 2 * ndir * mesh->N < (int64_t(1) << 31),
                     EFIE_ERR_ARG, "farfield_adjoint: bad sizes");
        EFIE_REQUIRE(ws_bytes >= size_t(2 * ndir) * size_t(mesh->N) * 16, EFIE_ERR_ARG,
                     "farfield_adjoint: workspace too small");
        const int N = int(mesh->N);
        const int nd = efie::wave_dirs(N, ndir);
        hipLaunchKernelGGL(efie::radiation_kernel, efie::wave_grid(N, ndir, nd), dim3(256), 0, stream, mesh->dm, k, eta,
                           dirs, int(ndir), nd, static_cast<double2*>(ws));
        hipLaunchKernelGGL(efie::radiation_adjoint_kernel, dim3((N + 255) / 256, unsigned(nrhs)), dim3(256), 0, stream,
                           static_cast<const double2*>(ws), static_cast<const double2*>(W), int(2 * ndir), N, int(nrhs),
                           static_cast<double2*>(G));
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}

extern "C" int efie_farfield_objective(const void* F, int64_t count, void* J, void* W, hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(F && J, EFIE_ERR_ARG, "farfield_objective: null argument");
        EFIE_REQUIRE(count >= 1, EFIE_ERR_ARG, "farfield_objective: need count >= 1");
        EFIE_REQUIRE(W != F, EFIE_ERR_ARG, "farfield_objective: W must not alias F");
        hipLaunchKernelGGL(efie::farfield_objective_kernel, dim3(1), dim3(256), 0, stream,
                           static_cast<const double2*>(F), count, static_cast<double*>(J), static_cast<double2*>(W));
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}
