// Device bodies of the pair rows W[p][i][n][side] of a chunk of test triangles
// (every pair value, the source RWG n and its side 0/1 = the source triangle is
// n's T+ / T-), the first step of the Calderon build, and helpers shared with the
// tile assembly: the operator scale factors and the quadrature tables of a mesh.
#pragma once

#include <hip/hip_runtime.h>

#include "efie_internal.h"
#include "pair_kernels.h"

namespace efie {

template <typename R>
struct Cplx;
template <>
struct Cplx<float> {
    using T = float2;
};
template <>
struct Cplx<double> {
    using T = double2;
};

// Z = A T_A + P T_Phi: A = eta j k / (4 pi), P = eta / (j k) / (4 pi) = -j eta conj(k) / (|k|^2 4 pi)
inline Scale operator_scale(double kr, double ki, double eta) {
    Scale sc{};
    const double f = eta / (4.0 * PI);
    sc.ar = -f * ki;
    sc.ai = f * kr;
    const double k2 = kr * kr + ki * ki;
    sc.pr = -f * ki / k2;
    sc.pi = -f * kr / k2;
    return sc;
}

template <typename R>
__host__ __device__ Tables<R> tables_of(const DevMesh& m);
template <>
__host__ __device__ inline Tables<double> tables_of<double>(const DevMesh& m) {
    return {m.qx, m.qy, m.qz, m.qw, m.vx, m.vy, m.vz, m.cf, m.dv, m.q3x, m.q3y, m.q3z};
}
template <>
__host__ __device__ inline Tables<float> tables_of<float>(const DevMesh& m) {
    return {m.qx32, m.qy32, m.qz32, m.qw32, m.vx32, m.vy32, m.vz32, m.cf32, m.dv32,
            m.q3x32, m.q3y32, m.q3z32};
}

// the far pair rows, one block (FAR_BLOCK threads) of logical index `logical` = (group of
// FAR_PB test triangles of the chunk, 256 source triangles).  A block takes FAR_PB
// test triangles against its source triangles: the source triangles' tables, read
// for the first, are cache hits for the others.  UPPER: only the far pairs with
// source triangle q > p are written; the entries of the pairs q < p are left
// unwritten and those of near pairs to the near rows (the reader takes only the
// entries of triangles q >= p and restores the other half from the symmetry of
// the operator).
// (ORBIT: far_pair_rule.)  KEEP: the source triangle's tables stay in registers over the
// FAR_PB test triangles.
template <typename R, bool CK, bool UPPER, bool ORBIT, bool KEEP>
__device__ __forceinline__ void far_rows_block(const DevMesh& m, const Tables<R>& tb, const Phase<R>& ph, const Scale& sc,
                                               typename Cplx<R>::T* __restrict__ W, int c0, int np, int nqblk,
                                               int logical) {
    using C2 = typename Cplx<R>::T;
    const int pg = logical / nqblk, qb = logical - pg * nqblk;
    const int q0 = qb * FAR_BLOCK + int(threadIdx.x);
    const int T = m.T;
    if (q0 >= T) return;
    const size_t N = size_t(m.N);
    const int pl1 = min(np, (pg + 1) * FAR_PB);
#pragma unroll 1
    for (int pl = pg * FAR_PB; pl < pl1; ++pl) {
        const int p = c0 + pl;
        // the source index is opaque to the compiler in each turn: it would keep the
        // source triangle's tables of both rules in registers across the turns (256
        // VGPRs and one wave per SIMD in FP64; reread, they are cache hits)
        int q = q0;
        if (!KEEP) asm volatile("" : "+v"(q));
        C2* rows = W + size_t(pl) * 3 * 2 * N;
        auto put = [&](int i, int j, R re, R im) {
            const size_t n = size_t(m.te[j * T + q]);
            const int side = tb.cf[j * T + q] > R(0) ? 0 : 1;
            rows[(size_t(i) * N + n) * 2 + side] = C2{re, im};
        };
        if (UPPER && q < p) continue;
        const bool near = is_near(m, p, q);
        if (UPPER && near) continue;
        if (near) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) put(i, j, R(0), R(0));
            continue;
        }
        far_pair_emit<R, CK, false, ORBIT>(m, tb, p, q, ph, sc, put, put);
    }
}

// ------------------------------------------------ Z by pair rows and a gather
// The pair rows W[p][i][n][side] of every pair q >= p (the other half is their
// transpose), each pair evaluated once, and Z gathered from them: entry (m, n), m <= n,
// is the sum of four pair values, each the element of one row.  The gather adds them in
// the order of the tiles (row triangle first, both increasing), which evaluate a pair in
// the same orientation (PairOrder), so that Z does not depend on the way taken.

// Z of complex128 takes this way while the rows (64 N^2 bytes) stay below 4 GiB and the
// caller brings the workspace; the tiles of such orders keep its orientation.  The line is
// what a call may ask for beside Z, four times its bytes, and not where the tiles become the
// faster way (tiles / rows: N = 480 88 / 48 us, 7680 3.7 / 2.6 ms, 12000 8.8 / 6.1 ms with 9 GB of
// rows, 30720 80 / 37 ms with 60 GB).
constexpr size_t PAIR_ROWS_MAX = size_t(4) << 30;
template <typename R>
__host__ __device__ inline bool tile_ordered(int N) {
    return sizeof(R) == 8 && size_t(N) * size_t(N) * 64 <= PAIR_ROWS_MAX;
}

// blocks of the pair kernel for PB test triangles each: the test triangles in bands of
// FAR_BLOCK (a multiple of PB), of which band g needs the source blocks g, g + 1, ...
__host__ __device__ inline long long pair_far_blocks(int T, int pb) {
    const long long nb = (T + FAR_BLOCK - 1) / FAR_BLOCK;
    long long n = 0;
    for (long long g = 0; g < nb; ++g) {
        const long long rows = T - g * FAR_BLOCK < FAR_BLOCK ? T - g * FAR_BLOCK : FAR_BLOCK;
        n += (rows + pb - 1) / pb * (nb - g);
    }
    return n;
}

template <bool CK>
__device__ __forceinline__ void pair_far_block(const DevMesh& m, const Tables<double>& tb, const Phase<double>& ph,
                                               const Scale& sc, double2* __restrict__ W, int pb, int b) {
    const int T = m.T;
    const int nb = (T + FAR_BLOCK - 1) / FAR_BLOCK;
    int g = 0, per;   // band, test triangle groups of it
    for (;; ++g) {
        per = (min(T - g * FAR_BLOCK, FAR_BLOCK) + pb - 1) / pb;
        const int in = per * (nb - g);
        if (b < in) break;
        b -= in;
    }
    const int q0 = (g + b / per) * FAR_BLOCK + int(threadIdx.x);
    if (q0 >= T) return;
    const size_t N = size_t(m.N);
    const int p0 = g * FAR_BLOCK + (b % per) * pb, p1 = min(T, p0 + pb);
#pragma unroll 1
    for (int p = p0; p < p1; ++p) {
        int q = q0;   // opaque, as in far_rows_block
        asm volatile("" : "+v"(q));
        if (q < p || is_near(m, p, q)) continue;
        double2* rows = W + size_t(p) * 6 * N;
        auto put = [&](int i, int j, double re, double im) {
            const size_t n = size_t(m.te[j * T + q]);
            const int side = tb.cf[j * T + q] > 0.0 ? 0 : 1;
            rows[(size_t(i) * N + n) * 2 + side] = make_double2(re, im);
        };
        far_pair_emit<double, CK, false>(m, tb, p, q, ph, sc, put, put);
    }
}

// near pair e = (p, q), q >= p, by the group of NEAR_G lanes (lane g)
__device__ __forceinline__ void pair_near_one(const DevMesh& m, double kr, double ki, const Scale& sc,
                                              double2* __restrict__ W, int e, int g) {
    const int p = m.near_p[e], q = m.near_q[e], T = m.T;
    const size_t N = size_t(m.N);
    double2* rows = W + size_t(p) * 6 * N;
    auto put = [&](int i, int j, double re, double im) {
        const size_t n = size_t(m.te[j * T + q]);
        const int side = m.cf[j * T + q] > 0.0 ? 0 : 1;
        rows[(size_t(i) * N + n) * 2 + side] = make_double2(re, im);
    };
    near_pair_group<false>(m, e, g, kr, ki, sc, put, put);
}

// One GT x GT tile of Z, rows r0.., columns c0.. (r0 <= c0), and its mirror, by 256
// threads.  A value of row triangle p and column triangle q stands in the row of p if
// p <= q, otherwise in the row of q (transposed): both are read along their rows, so
// that lanes read neighbouring 32-byte pairs of sides, and meet in LDS.
constexpr int GATHER = 32;
struct GatherLds {
    double2 v[GATHER][GATHER + 1][4];     // [row][column][2 (row side) + column side]
    int et[2][2][GATHER], el[2][2][GATHER];   // [rows, columns][side]: triangle and local edge
};
__device__ __forceinline__ void gather_tile(const DevMesh& m, const double2* __restrict__ W, double2* __restrict__ Z,
                                            int bi, int bj, GatherLds& L) {
    const int N = m.N, tid = int(threadIdx.x);
    const int r0 = bi * GATHER, c0 = bj * GATHER;
    if (tid < 4 * GATHER) {
        const int w = tid / (2 * GATHER), sd = (tid / GATHER) & 1, x = tid % GATHER;
        const int e = min((w ? c0 : r0) + x, N - 1);
        L.et[w][sd][x] = m.et[sd * N + e];
        L.el[w][sd][x] = m.el[sd * N + e];
    }
    __syncthreads();
    const int c = tid % GATHER, y = tid / GATHER;   // column of the row read, first row
    // rows of W along the columns (w = 0: test RWGs of the tile's rows) and along the
    // tile's rows (w = 1: the columns' RWGs as test RWGs)
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int x0 = w ? r0 : c0;
        const bool ok = x0 + c < N;
#pragma unroll
        for (int sd = 0; sd < 2; ++sd)
#pragma unroll
            for (int u = 0; u < GATHER / 8; ++u) {
                const int r = y + 8 * u;
                const int t = L.et[w][sd][r], i = L.el[w][sd][r];
                const int s0 = L.et[1 - w][0][c], s1 = L.et[1 - w][1][c];
                // the stored orientation: t <= s for the tile's rows, t < s for its columns
                const bool h0 = ok && t + w <= s0, h1 = ok && t + w <= s1;
                const double2* src = W + ((size_t(t) * 3 + size_t(i)) * size_t(N) + size_t(ok ? x0 + c : 0)) * 2;
                double2 a = make_double2(0.0, 0.0), b = a;
                if (h0) a = src[0];
                if (h1) b = src[1];
                if (w == 0) {
                    if (h0) L.v[r][c][2 * sd] = a;
                    if (h1) L.v[r][c][2 * sd + 1] = b;
                } else {
                    if (h0) L.v[c][r][sd] = a;
                    if (h1) L.v[c][r][2 + sd] = b;
                }
            }
    }
    __syncthreads();
    double2 z[GATHER / 8];
#pragma unroll
    for (int u = 0; u < GATHER / 8; ++u) {
        const int r = y + 8 * u;
        const int rs = L.et[0][1][r] < L.et[0][0][r] ? 2 : 0, cs = L.et[1][1][c] < L.et[1][0][c] ? 1 : 0;
        double2 a = make_double2(0.0, 0.0);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const double2 v = L.v[r][c][x ^ rs ^ cs];
            a.x += v.x;
            a.y += v.y;
        }
        z[u] = a;
    }
    const bool diag = bi == bj;
#pragma unroll
    for (int u = 0; u < GATHER / 8; ++u) {
        const int r = y + 8 * u;
        if (r0 + r < N && c0 + c < N && !(diag && r > c)) Z[size_t(r0 + r) * N + (c0 + c)] = z[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GATHER / 8; ++u) L.v[y + 8 * u][c][0] = z[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GATHER / 8; ++u) {
        const int r = y + 8 * u;   // Z row c0 + r, column r0 + c: entry (r0 + c, c0 + r)
        if (c0 + r < N && r0 + c < N && !(diag && c >= r)) Z[size_t(c0 + r) * N + (r0 + c)] = L.v[c][r][0];
    }
}

// the ordered near pair e = (p, q) with p in the chunk [c0, c1), by the group of
// NEAR_G lanes (lane g): its values replace the zeros the far rows wrote (FP64
// arithmetic, all nine entries).  upper: pairs with q < p are not written and the
// diagonal blocks (q = p) are halved.
template <typename R>
__device__ __forceinline__ void near_rows_one(const DevMesh& m, double kr, double ki, const Scale& sc,
                                              typename Cplx<R>::T* __restrict__ W, int c0, int c1, int e, int g,
                                              int upper) {
    using C2 = typename Cplx<R>::T;
    const int p = m.near_p[e], q = m.near_q[e];
    if (p < c0 || p >= c1) return;
    if (upper && q < p) return;
    const double f = upper && q == p ? 0.5 : 1.0;
    const int T = m.T;
    const size_t N = size_t(m.N);
    C2* rows = W + size_t(p - c0) * 3 * 2 * N;
    auto put = [&](int i, int j, double re, double im) {
        const size_t n = size_t(m.te[j * T + q]);
        const int side = m.cf[j * T + q] > 0.0 ? 0 : 1;
        rows[(size_t(i) * N + n) * 2 + side] = C2{R(f * re), R(f * im)};
    };
    near_pair_group<false>(m, e, g, kr, ki, sc, put, put);
}

}  // namespace efie
