// Complex64 Y = X Z^T on the fp16 matrix cores, every operand in two fp16 parts.
//
// Splitting.  A row's chunk of KC complex elements is scaled by the power of two that
// takes its largest real or imaginary part to [2^14, 2^15); each scaled value x is
// h + 2^-11 l with h the nearest fp16 number and l the nearest to 2^11 times the (exact)
// remainder: within 2^-23 |x| down to 2^-27 of the chunk's largest part, and within 2^-50
// of the largest part below that.  A product takes three fp16 products, each exact in the
// matrix core's FP32 accumulator: h l' and l h' of the whole chunk first, then, after a
// factor of 2^-11, h h' on top; l l' is below 2^-22 of the product and left out.
// Non-finite values stay non-finite (an infinity gives NaN).
// Range.  Nonzero elements (or a lane's real or imaginary parts) below 2^-27 of the
// largest are "wide": 64 of them err by at most 2^-42 of the product of both chunks'
// largest.  Where every element of the other chunk is above 2^-20 of its largest, one
// term of sum |x| |z| is 2^-20 of that product and the error is below 2^-22 of the sum.
// Where an element of it is smaller ("thin", a zero among them), the large values may
// meet only those, so a turn with a wide and a thin chunk is multiplied as stored, on
// the FP32 matrix cores (39.6 against 17.6 ms where every turn is).  Share of the turns on
// icospheres, whose symmetry leaves rounding errors for zeros, Z times plane waves: 0.33 at
// N = 1920, 0.05 at 7680, 0.01 at 30720; on a perturbed sphere and on random dipoles, none.
// Accumulation.  The FP32 sums of one chunk (at most 64 complex terms) are scaled back
// and added to FP64 accumulators, for complex64 and complex128 results alike.  Measured
// against the FP64 product of the stored values (2-norm): 1.1e-7 for orders 300 to 30720,
// where the FP32 matrix cores give 1.6e-7 to 2.4e-7 with FP64 flushes and 4.4e-7 to
// 6.0e-6 with FP32 sums; 2.9e-7 of sum |x| |z| at worst for rows of 24 decades.
//
// Why.  The FP32 matrix cores reach 157 TFLOP/s: the planar kernels ran at 0.85 to
// 0.95 of that, 25.8 to 28.8 ms for 30720 x 30720 times 512.  Three fp16 products take
// 3/16 of the time of one FP32 product.  This kernel takes 16.1 ms (240 TFLOP/s of
// complex products, 0.29 of the fp16 peak over three).  Bound by instruction issue:
// matrix instructions take 0.36 of a SIMD's cycles and vector ones (splits, tests of the
// range, scaling back) 0.54, and they hardly overlap.  With l unscaled it took 14.3 ms,
// but held values below 2^-16 of a chunk's largest only to 2^-39 of that, and one large
// value in a chunk against a zero cost all digits of the others' products.
// Three bf16 parts need no scaling but six products: 22.4 ms at 1.9 GHz.
//
// Layout.  Per chunk and group: the rows' h and l planes of the real and imaginary
// parts in LDS, rows padded by 8 values (16-byte reads without bank conflicts), one
// buffer; the next chunk's global loads are in flight during the multiply.  Eight lanes
// hold a row's chunk, so that its maximum takes three lane exchanges.
#pragma once

#include <hip/hip_runtime.h>

#include "efie_internal.h"

namespace efie {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
// two complex64 values, 8-byte aligned (rows of odd order)
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(8)));

// max(m, |a|, |b|) (the compiler's fmaxf adds a canonicalization for each operand)
__device__ __forceinline__ float max3_abs(float m, float a, float b) {
    float r;
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(m), "v"(a), "v"(b));
    return r;
}
// maximum of non-negative floats over aligned groups of 8 lanes (their bits compare
// as unsigned integers)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
    return max(v, uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xf, 0xf, true)));
}
__device__ __forceinline__ uint32_t max8(float m) {
    uint32_t v = dpp_max<0xb1>(__builtin_bit_cast(uint32_t, m));   // quad_perm [1, 0, 3, 2]
    v = dpp_max<0x4e>(v);                                          // quad_perm [2, 3, 0, 1]
    return dpp_max<0x141>(v);                                      // row_half_mirror
}
__device__ __forceinline__ float max_abs(float a, float b) {
    float r;
    asm("v_max_f32 %0, |%1|, |%2|" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float min3_abs(float m, float a, float b) {
    float r;
    asm("v_min3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(m), "v"(a), "v"(b));
    return r;
}
// a sc and b sc (sc a power of two) in two fp16 parts each, packed: the nearest fp16
// values, and those of LSCALE times the exact remainders
constexpr float LSCALE = 2048.f;
__device__ __forceinline__ void split2(float a, float b, float sc, halfx2& h, halfx2& l) {
    h = __builtin_convertvector(floatx2{a * sc, b * sc}, halfx2);
    l = __builtin_convertvector(floatx2{__builtin_fmaf(a, sc, -float(h.x)) * LSCALE, __builtin_fmaf(b, sc, -float(h.y)) * LSCALE},
                                halfx2);
}
// of one row's chunk: an element the two parts do not hold to 2^-23, and one so far below the
// largest that the other operand's WIDE elements may count against it (see above); of X, of Z
enum SplitRange { X_WIDE = 1, X_THIN = 2, Z_WIDE = 4, Z_THIN = 8 };

// where the sums of a tile go: complex64 Y, the rows yrow of complex128 Y, or (a block
// of one of several ranges of K) the workspace that split_sum_kernel adds up
enum SplitOut { OUT_C64, OUT_C128, OUT_PART };

// Block: WK groups of WM x WN waves; a wave owns a 32 x 32 tile of complex outputs
// (rows: right-hand sides, columns: unknowns), the groups share the block's tile and
// take the K chunks of the block's range in turn.
template <int WM, int WN, int WK, int KC, int OUT, int MINW>
__global__ __launch_bounds__(64 * WM * WN * WK, MINW) void cgemm_split_kernel(const float2* __restrict__ X,
                                                                              const float2* __restrict__ Z,
                                                                              void* __restrict__ Yv, int M, int n,
                                                                              const int* __restrict__ yrow, int ranges) {
    constexpr int GT = 64 * WM * WN;                  // threads of a group
    constexpr int BM = 32 * WM, BN = 32 * WN;
    constexpr int RS = KC + 8;                        // fp16 per LDS row
    constexpr int PC = KC / 16;                       // 16-byte pieces of a lane: 8 lanes hold a row's chunk
    constexpr int RP = GT / 8;                        // rows of a pass
    constexpr int NA = BM / RP, NB = BN / RP;
    static_assert(BM % RP == 0 && BN % RP == 0, "tile not divisible by the group");
    constexpr int PLANES = 4 * (BM + BN) * RS;        // fp16 of a group's planes
    constexpr int STAGE = 2 * PLANES + 4 * (BM + BN); // bytes: the planes and the rows' exponents
    constexpr int RED = WK > 1 ? (WK - 1) * GT * 16 * 16 : 0;
    constexpr int LDSB = STAGE * WK > RED ? STAGE * WK : RED;
    __shared__ __attribute__((aligned(16))) char lds[LDSB];
    __shared__ int range_of[2];                       // SplitRange bits of a turn's chunks, of even and odd turns
    const int tid = threadIdx.x % GT;
    const int g = WK > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / GT) : 0;
    const int lane = tid & 63, w = tid >> 6;
    const int wm = w / WN, wn = w % WN;
    const int nbm = (M + BM - 1) / BM;
    const int nblk = int(gridDim.x);
    const int xcd = int(blockIdx.x) & 7, idx = int(blockIdx.x) >> 3;
    const int per = nblk >> 3, rem = nblk & 7;
    const int logical = xcd * per + min(xcd, rem) + idx;
    // the tile, rows of right-hand sides fastest, and the range of K
    const int ntile = nblk / ranges;
    const int range = OUT == OUT_PART ? logical / ntile : 0;
    const int tile = logical - range * ntile;
    const int bm = tile % nbm, bn = tile / nbm;
    const int s0 = bm * BM, i0 = bn * BN;
    _Float16* Xs = reinterpret_cast<_Float16*>(lds + g * STAGE);
    _Float16* Zs = Xs + 4 * BM * RS;
    int* ex = reinterpret_cast<int*>(lds + g * STAGE + 2 * PLANES);
    int* ez = ex + BM;

    double dr[16], di[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) dr[r] = di[r] = 0.0;
    floatx4u ra[NA][PC], rb[NB][PC];
    const int lr = tid >> 3, lc = tid & 7;
    // chunk c into registers (rows past the end: the last row again, never written
    // out); a uniform base and 32-bit byte offsets of the thread's rows
    uint32_t oa[NA], ob[NB];
#pragma unroll
    for (int q = 0; q < NA; ++q) oa[q] = (uint32_t(min(lr + RP * q, M - 1 - s0)) * uint32_t(n) + 2 * lc) * 8u;
#pragma unroll
    for (int q = 0; q < NB; ++q) ob[q] = (uint32_t(min(lr + RP * q, n - 1 - i0)) * uint32_t(n) + 2 * lc) * 8u;
    const char* xb = reinterpret_cast<const char*>(X + size_t(s0) * n);
    const char* zb = reinterpret_cast<const char*>(Z + size_t(i0) * n);
    auto gload = [&](int c) {
        const char *xc = xb + size_t(c) * (KC * 8), *zc = zb + size_t(c) * (KC * 8);
        if (c * KC + KC <= n) {
#pragma unroll
            for (int q = 0; q < NA; ++q)
#pragma unroll
                for (int p = 0; p < PC; ++p) ra[q][p] = *reinterpret_cast<const floatx4u*>(xc + oa[q] + 128 * p);
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int p = 0; p < PC; ++p) rb[q][p] = *reinterpret_cast<const floatx4u*>(zc + ob[q] + 128 * p);
        } else {
            const int j = c * KC + 2 * lc;
            auto tail = [&](const char* row, int jj) {   // columns past the end: zero
                floatx4u v{0.f, 0.f, 0.f, 0.f};
                if (jj < n) {
                    v.x = reinterpret_cast<const float*>(row)[0];
                    v.y = reinterpret_cast<const float*>(row)[1];
                }
                if (jj + 1 < n) {
                    v.z = reinterpret_cast<const float*>(row)[2];
                    v.w = reinterpret_cast<const float*>(row)[3];
                }
                return v;
            };
#pragma unroll
            for (int q = 0; q < NA; ++q)
#pragma unroll
                for (int p = 0; p < PC; ++p) ra[q][p] = tail(xc + oa[q] + 128 * p, j + 16 * p);
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int p = 0; p < PC; ++p) rb[q][p] = tail(zc + ob[q] + 128 * p, j + 16 * p);
        }
    };
    // a row's chunk, scaled by the power of two that takes its largest part to [2^14, 2^15), into the planes
    auto put = [&](_Float16* planes, int* e, int rows, int row, const floatx4u (&v)[PC], bool& wide, bool& thin) {
        float m = 0.f, lo = __builtin_inff();   // the lane's largest and smallest part
#pragma unroll
        for (int p = 0; p < PC; ++p) {
            m = max3_abs(max3_abs(m, v[p].x, v[p].y), v[p].z, v[p].w);
            lo = min3_abs(min3_abs(lo, v[p].x, v[p].y), v[p].z, v[p].w);
        }
        const uint32_t mx = max8(m);
        m = __builtin_bit_cast(float, mx);
        if (lo < m * 0x1p-20f) {   // a part of ordinary data now and then, zeros
            const float tt = m * 0x1p-20f, tw = m * 0x1p-27f;
            auto below = [&](float a) {
                thin |= a < tt;
                wide |= a > 0.f && a < tw;
            };
            float mr = 0.f, mi = 0.f;   // the lane's real and imaginary parts
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                below(max_abs(v[p].x, v[p].y));
                below(max_abs(v[p].z, v[p].w));
                mr = max3_abs(mr, v[p].x, v[p].z);
                mi = max3_abs(mi, v[p].y, v[p].w);
            }
            below(mr);
            below(mi);
        }
        const int b = max(int(mx >> 23), 14);
        const float sc = __builtin_bit_cast(float, uint32_t(268 - b) << 23);
        if (lc == 0) e[row] = (b - 141) * (1 << 20);
#pragma unroll
        for (int p = 0; p < PC; ++p) {
            halfx2 rh, rl, ih, il;
            split2(v[p].x, v[p].z, sc, rh, rl);
            split2(v[p].y, v[p].w, sc, ih, il);
            _Float16* d = planes + row * RS + 2 * lc + 16 * p;
            *reinterpret_cast<halfx2*>(d) = rh;
            *reinterpret_cast<halfx2*>(d + rows * RS) = rl;
            *reinterpret_cast<halfx2*>(d + 2 * rows * RS) = ih;
            *reinterpret_cast<halfx2*>(d + 3 * rows * RS) = il;
        }
    };
    auto lstore = [&](int turn) {
        bool xw = false, xt = false, zw = false, zt = false;
#pragma unroll
        for (int q = 0; q < NA; ++q) put(Xs, ex, BM, lr + RP * q, ra[q], xw, xt);
#pragma unroll
        for (int q = 0; q < NB; ++q) put(Zs, ez, BN, lr + RP * q, rb[q], zw, zt);
        if (__any(xt || zt)) {   // wide elements are thin ones too
            const int f = (__any(xw) ? X_WIDE : 0) | (__any(xt) ? X_THIN : 0) | (__any(zw) ? Z_WIDE : 0) | (__any(zt) ? Z_THIN : 0);
            if (lane == 0) atomicOr(&range_of[turn & 1], f);
        }
    };
    // the same chunk as stored, rows padded by one value, over the planes
    constexpr int RF = KC + 1;
    float2* Xf = reinterpret_cast<float2*>(lds + g * STAGE);
    float2* Zf = Xf + BM * RF;
    auto rstore = [&]() {
        auto raw = [&](float2* row, const floatx4u (&v)[PC]) {
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                row[2 * lc + 16 * p] = make_float2(v[p].x, v[p].y);
                row[2 * lc + 16 * p + 1] = make_float2(v[p].z, v[p].w);
            }
        };
#pragma unroll
        for (int q = 0; q < NA; ++q) raw(Xf + (lr + RP * q) * RF, ra[q]);
#pragma unroll
        for (int q = 0; q < NB; ++q) raw(Zf + (lr + RP * q) * RF, rb[q]);
    };
    const int l32 = lane & 31, kh = lane >> 5;
    const _Float16* xp = Xs + (wm * 32 + l32) * RS + 8 * kh;
    const _Float16* zp = Zs + (wn * 32 + l32) * RS + 8 * kh;
    auto multiply = [&]() {
        floatx16 rr{}, ii{}, ri{};   // sum xr zr, sum xi zi, sum xr zi + xi zr
        // h l' + l h' of every term first, then h h' on top of them
#pragma unroll
        for (int ks = 0; ks < KC / 16; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            halfx8 x[4], z[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                x[s] = *reinterpret_cast<const halfx8*>(xp + s * BM * RS + 16 * ks);
                z[s] = *reinterpret_cast<const halfx8*>(zp + s * BN * RS + 16 * ks);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int j = 1 - i;
                rr = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[i], z[j], rr, 0, 0, 0);
                ri = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[i], z[2 + j], ri, 0, 0, 0);
                ii = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[2 + i], z[2 + j], ii, 0, 0, 0);
                ri = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[2 + i], z[j], ri, 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            rr[r] *= 1.f / LSCALE;
            ii[r] *= 1.f / LSCALE;
            ri[r] *= 1.f / LSCALE;
        }
#pragma unroll
        for (int ks = 0; ks < KC / 16; ++ks) {
            halfx8 x[2], z[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                x[s] = *reinterpret_cast<const halfx8*>(xp + 2 * s * BM * RS + 16 * ks);
                z[s] = *reinterpret_cast<const halfx8*>(zp + 2 * s * BN * RS + 16 * ks);
            }
            rr = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[0], z[0], rr, 0, 0, 0);
            ri = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[0], z[1], ri, 0, 0, 0);
            ii = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[1], z[1], ii, 0, 0, 0);
            ri = __builtin_amdgcn_mfma_f32_32x32x16_f16(x[1], z[0], ri, 0, 0, 0);
        }
        // the chunk's sums, scaled back, into the FP64 accumulators: 2^e as the high
        // word of a double from the exponents kept shifted
        const int c = ez[wn * 32 + l32] + (1023 << 20);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int4 e4 = *reinterpret_cast<const int4*>(ex + wm * 32 + 8 * q + 4 * kh);
            const int e[4] = {e4.x + c, e4.y + c, e4.z + c, e4.w + c};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double s2 = __hiloint2double(e[r], 0);
                dr[4 * q + r] = fma(double(rr[4 * q + r] - ii[4 * q + r]), s2, dr[4 * q + r]);
                di[4 * q + r] = fma(double(ri[4 * q + r]), s2, di[4 * q + r]);
            }
        }
    };
    // the chunk of rstore on the FP32 matrix cores
    auto multiply32 = [&]() {
        floatx16 rr{}, ii{}, ri{};
        const float2* xr = Xf + (wm * 32 + l32) * RF + kh;
        const float2* zr = Zf + (wn * 32 + l32) * RF + kh;
#pragma unroll 4
        for (int k = 0; k < KC; k += 2) {
            const float2 x = xr[k], z = zr[k];
            rr = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, z.x, rr, 0, 0, 0);
            ri = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, z.y, ri, 0, 0, 0);
            ii = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, z.y, ii, 0, 0, 0);
            ri = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, z.x, ri, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            dr[r] += double(rr[r] - ii[r]);
            di[r] += double(ri[r]);
        }
    };
    if (threadIdx.x < 2) range_of[threadIdx.x] = 0;
    const int all = (n + KC - 1) / KC;
    const int c0 = OUT == OUT_PART ? int(int64_t(all) * range / ranges) : 0;
    const int nch = OUT == OUT_PART ? int(int64_t(all) * (range + 1) / ranges) : all;
    const int turns = (nch - c0 + WK - 1) / WK;
    if (c0 + g < nch) gload(c0 + g);
    for (int i = 0; i < turns; ++i) {
        const int c = c0 + g + WK * i;
        __syncthreads();
        if (c < nch) lstore(i);
        __syncthreads();
        const int f = __builtin_amdgcn_readfirstlane(range_of[i & 1]);
        if (threadIdx.x == 0) range_of[(i + 1) & 1] = 0;   // read before this turn's barriers, set after the next one
        const bool full = ((f & X_WIDE) && (f & Z_THIN)) || ((f & Z_WIDE) && (f & X_THIN));
        if (full) {
            if (c < nch) rstore();
            __syncthreads();
        }
        if (c + WK < nch) gload(c + WK);
        if (c < nch) {
            if (full) multiply32();
            else multiply();
        }
    }
    if constexpr (WK > 1) {
        // the groups' sums into group 0, in order
        double2* red = reinterpret_cast<double2*>(lds);
        __syncthreads();
        if (g > 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) red[((g - 1) * 16 + r) * GT + tid] = make_double2(dr[r], di[r]);
        }
        __syncthreads();
        if (g > 0) return;
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int o = 0; o < WK - 1; ++o) {
                const double2 v = red[(o * 16 + r) * GT + tid];
                dr[r] += v.x;
                di[r] += v.y;
            }
    }
    if constexpr (OUT == OUT_PART) {
        double2* part = static_cast<double2*>(Yv) + size_t(logical) * (16 * GT) + tid;
#pragma unroll
        for (int r = 0; r < 16; ++r) part[r * GT] = make_double2(dr[r], di[r]);
        return;
    }
    // D of the 32x32x16 instruction: lane l holds column l % 32, rows 8 (r / 4) + 4 (l / 32) + r % 4
    const int col = i0 + wn * 32 + l32;
    if (col >= n) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = s0 + wm * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
        if (row >= M) continue;
        if constexpr (OUT == OUT_C128)
            reinterpret_cast<double2*>(Yv)[size_t(yrow[row]) * n + col] = make_double2(dr[r], di[r]);
        else
            reinterpret_cast<float2*>(Yv)[size_t(row) * n + col] = make_float2(float(dr[r]), float(di[r]));
    }
}

// Y = the sum over the ranges of K, in order, of the partial tiles of
// cgemm_split_kernel<WM, WN, 1, KC, OUT_PART>: a thread per output, a block per 256
// outputs of a tile (one register index of the tile's threads, or several)
template <int WM, int WN, bool OUT64>
__global__ __launch_bounds__(256) void split_sum_kernel(const double2* __restrict__ part, void* __restrict__ Yv, int M,
                                                        int n, const int* __restrict__ yrow, int ntile, int ranges) {
    constexpr int GT = 64 * WM * WN, TS = 16 * GT;
    const int tile = int(blockIdx.x) / (TS / 256);
    const int e = (int(blockIdx.x) % (TS / 256)) * 256 + int(threadIdx.x);
    const int r = e / GT, tid = e % GT, lane = tid & 63, w = tid >> 6;
    const int nbm = (M + 32 * WM - 1) / (32 * WM);
    const int row = (tile % nbm) * 32 * WM + (w / WN) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int col = (tile / nbm) * 32 * WN + (w % WN) * 32 + (lane & 31);
    if (row >= M || col >= n) return;
    double2 a = make_double2(0.0, 0.0);
    const double2* p = part + size_t(tile) * TS + e;
    const size_t step = size_t(ntile) * TS;
    for (int k = 0; k < ranges; k += 8) {   // eight loads in flight
        double2 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = p[size_t(min(k + q, ranges - 1)) * step];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (k + q < ranges) {
                a.x += v[q].x;
                a.y += v[q].y;
            }
    }
    if constexpr (OUT64)
        static_cast<double2*>(Yv)[size_t(yrow[row]) * n + col] = a;
    else
        static_cast<float2*>(Yv)[size_t(row) * n + col] = make_float2(float(a.x), float(a.y));
}

}  // namespace efie
