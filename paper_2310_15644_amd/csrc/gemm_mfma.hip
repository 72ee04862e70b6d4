// Complex64 Y = X Z^T on matrix cores (MFMA): the dispatch, and the kernels on the
// FP32 matrix cores (the default is the fp16 split kernel of gemm_split.h; these stay
// selectable by efie_gemm_select and the autotuner).
//
// Planar complex form: the K chunks of X (right-hand sides) and Z (the
// symmetric operator, whose rows are the output unknowns) are staged in LDS as
// complex (re, im) rows.  In v_mfma_f32_16x16x4f32 lane l supplies A[l%16][l/16]
// and B[l/16][l%16], and accumulator register r of lane l holds
// D[4*(l/16)+r][l%16]; here a lane's operand element is one complex value,
// fetched with one 8-byte LDS read, and each 16 x 16 complex output block takes
// four real instructions per 4 complex K:
//   Yr += Ar Br + (-Ai) Bi,   Yi += Ar Bi + Ai Br
// (8 M n K real flops in all); the FP64-flush path below takes three (3M).  X and Y keep the ABI's interleaved complex
// layouts; no operand is converted or copied.
//
// Tiling: a block of 256 threads (4 wavefronts, 2 x 2) owns BM right-hand sides
// x BNC unknowns; K is walked in chunks of KC complex elements.
// ACC64: the FP32 matrix-core partial sums are flushed into FP64 accumulators after
// every two K chunks (2 KC terms), and the result is written as complex128 to the
// rows Y[yrow[r]] (the Krylov vectors); this bounds the FP32 accumulation error to
// short partial sums.  Otherwise complex64 is written to Y[r].
//
// Pipeline: two LDS buffers and two register sets of staged global loads (16-byte
// loads when n is even and the operands 16-byte aligned, 8-byte otherwise;
// without per-element bounds tests when the tile lies wholly inside the
// matrices).  While chunk c is multiplied from LDS, chunk c+1 waits in registers
// and the loads of chunk c+2 are in flight: the global latency is hidden behind
// two chunks of matrix work instead of one.  After the multiply, chunk c+1 goes
// to the other LDS buffer; one barrier per chunk.  LDS rows are padded to KC + 2
// complex values, which keeps them 16-byte aligned for the 16-byte stores.  (The
// 8-byte reads still meet some bank conflicts; an odd pad removes them for
// KC = 16 and halves them for KC = 32, but changes the time by under one
// percent: the conflicts overlap with the matrix instructions.)
// Block order: workgroups are dealt to the 8 XCDs round-robin by id, so the ids
// are remapped to give each XCD a contiguous run of tiles, walking the
// right-hand-side tiles of one Z row strip first: the blocks that read the
// same strip of Z share one XCD's L2 and run at about the same time.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "efie_internal.h"
#include "linalg.h"
#include "gemm_split.h"

namespace efie {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Minimum wavefronts per SIMD asked of the register allocator: three for the
// FP64-flush tile with 32-row chunks, whose two-chunk flush interval would
// otherwise take it to 178 registers and two wavefronts.
template <int BM, int BNC, int KC, bool ACC64>
constexpr int gemm_min_waves() {
    return (ACC64 && BM == 64 && BNC == 32 && KC == 32) ? 3 : 1;
}

template <int BM, int BNC, int KC, bool ACC64>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(gemm_min_waves<BM, BNC, KC, ACC64>())))
void cgemm_planar_kernel(const float2* __restrict__ X, const float2* __restrict__ Z,
                                                           void* __restrict__ Yv, int M, int mrows, int n,
                                                           const int* __restrict__ yrow) {
    constexpr int AS = KC + 2;             // float2 per LDS row (16-byte aligned rows)
    constexpr int WM = BM / 2, WN = BNC / 2;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int KV = KC / 2;             // 16-byte groups per row of a chunk
    constexpr int NA = BM * KV / 256, NB = BNC * KV / 256;
    static_assert(TM >= 1 && TN >= 1 && NA >= 1 && NB >= 1, "tile too small for the block");
    static_assert(BM * KV % 256 == 0 && BNC * KV % 256 == 0, "tile not divisible by the block");
    __shared__ float2 As[2][BM * AS];
    __shared__ float2 Bs[2][BNC * AS];

    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int wm = w >> 1, wn = w & 1;
    const int nbm = (M + BM - 1) / BM;
    const int nblk = int(gridDim.x);
    const int xcd = int(blockIdx.x) & 7, idx = int(blockIdx.x) >> 3;
    const int per = nblk >> 3, rem = nblk & 7;
    const int logical = xcd * per + min(xcd, rem) + idx;
    const int bm = logical % nbm, bn = logical / nbm;
    const int s0 = bm * BM, i0 = bn * BNC;
    const bool vec = (n & 1) == 0 && ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Z)) & 15) == 0;
    // X has mrows >= M readable rows (rows M.. are computed and not written): a tile
    // within them takes the unchecked loads
    const bool inside = vec && s0 + BM <= mrows && i0 + BNC <= n;

    // FP32 path: accr, acci = Yr, Yi (four real products per complex block).
    // ACC64 path, 3M form: accr = sum xr zr, acci = sum xi zi, acc3 = sum (xr + xi)(zr + zi)
    // (three real products); Yr = accr - acci and Yi = acc3 - accr - acci are formed
    // in FP64 at every flush.
    floatx4 accr[TM][TN], acci[TM][TN], acc3[ACC64 ? TM : 1][ACC64 ? TN : 1];
    double dr[ACC64 ? TM : 1][ACC64 ? TN : 1][4], di[ACC64 ? TM : 1][ACC64 ? TN : 1][4];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            accr[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
            acci[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
    if constexpr (ACC64) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                acc3[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) dr[a][b][r] = di[a][b][r] = 0.0;
            }
    }

    // two register sets of staged global loads: chunk c goes to set c % 2
    float4 ra[2][NA], rb[2][NB];
    auto load2 = [&](const float2* base, int row, int nrows, int j) -> float4 {
        // complex elements j and j+1 of row `row` (zero outside the matrix)
        if (row >= nrows || j >= n) return make_float4(0.f, 0.f, 0.f, 0.f);
        const float2* p = base + size_t(row) * n + j;
        if (vec) return *reinterpret_cast<const float4*>(p);
        const float2 u = p[0];
        const float2 v = j + 1 < n ? p[1] : make_float2(0.f, 0.f);
        return make_float4(u.x, u.y, v.x, v.y);
    };
    auto gload = [&](int j0, float4* ga, float4* gb) {
        if (inside && j0 + KC <= n) {
#pragma unroll
            for (int q = 0; q < NA; ++q) {
                const int e = tid + 256 * q, r = e / KV, c = e % KV;
                ga[q] = *reinterpret_cast<const float4*>(X + size_t(s0 + r) * n + j0 + 2 * c);
            }
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int e = tid + 256 * q, r = e / KV, c = e % KV;
                gb[q] = *reinterpret_cast<const float4*>(Z + size_t(i0 + r) * n + j0 + 2 * c);
            }
        } else {
#pragma unroll
            for (int q = 0; q < NA; ++q) {
                const int e = tid + 256 * q, r = e / KV, c = e % KV;
                ga[q] = load2(X, s0 + r, mrows, j0 + 2 * c);
            }
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int e = tid + 256 * q, r = e / KV, c = e % KV;
                gb[q] = load2(Z, i0 + r, n, j0 + 2 * c);
            }
        }
    };
    auto lstore = [&](int buf, const float4* ga, const float4* gb) {
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const int e = tid + 256 * q, r = e / KV, c = e % KV;
            *reinterpret_cast<float4*>(&As[buf][r * AS + 2 * c]) = ga[q];
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int e = tid + 256 * q, r = e / KV, c = e % KV;
            *reinterpret_cast<float4*>(&Bs[buf][r * AS + 2 * c]) = gb[q];
        }
    };

    const int kq = lane >> 4;          // 0..3: k within an instruction
    const int l16 = lane & 15;
    const int nch = (n + KC - 1) / KC;
    // one chunk: multiply LDS buffer ch % 2, flush when fl is set (ACC64; odd chunks), store
    // the staged chunk ch + 1 (set SN) into the other buffer; the loads of chunk
    // ch + 2 (set SP, free since its chunk went to LDS) are issued first, two chunks
    // ahead
    auto flush = [&]() {
        if constexpr (ACC64) {
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const double p1 = accr[a][b][r], p2 = acci[a][b][r], p3 = acc3[a][b][r];
                        dr[a][b][r] += p1 - p2;
                        di[a][b][r] += p3 - p1 - p2;
                    }
                    accr[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
                    acci[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
                    acc3[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    auto step = [&](int ch, auto sp, auto sn, auto fl) {
        constexpr int SP = decltype(sp)::value, SN = decltype(sn)::value;
        const int buf = ch & 1;
        if (ch + 2 < nch) gload((ch + 2) * KC, ra[SP], rb[SP]);
        const float2* A_ = As[buf] + (wm * WM + l16) * AS + kq;
        const float2* B_ = Bs[buf] + (wn * WN + l16) * AS + kq;
#pragma unroll
        for (int kk = 0; kk < KC; kk += 4) {
            float2 xa[TM], zb[TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) xa[a] = A_[a * 16 * AS + kk];
#pragma unroll
            for (int b = 0; b < TN; ++b) zb[b] = B_[b * 16 * AS + kk];
            if constexpr (ACC64) {
                float xs[TM], zs[TN];
#pragma unroll
                for (int a = 0; a < TM; ++a) xs[a] = xa[a].x + xa[a].y;
#pragma unroll
                for (int b = 0; b < TN; ++b) zs[b] = zb[b].x + zb[b].y;
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[a].x, zb[b].x, accr[a][b], 0, 0, 0);
                        acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[a].y, zb[b].y, acci[a][b], 0, 0, 0);
                        acc3[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[a], zs[b], acc3[a][b], 0, 0, 0);
                    }
            } else {
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[a].x, zb[b].x, accr[a][b], 0, 0, 0);
                        acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[a].x, zb[b].y, acci[a][b], 0, 0, 0);
                    }
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(-xa[a].y, zb[b].y, accr[a][b], 0, 0, 0);
                        acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[a].y, zb[b].x, acci[a][b], 0, 0, 0);
                    }
            }
        }
        if constexpr (ACC64) {
            if constexpr (decltype(fl)::value) flush();
        }
        if (ch + 1 < nch) lstore(buf ^ 1, ra[SN], rb[SN]);
        __syncthreads();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    gload(0, ra[0], rb[0]);
    lstore(0, ra[0], rb[0]);
    if (nch > 1) gload(KC, ra[1], rb[1]);
    __syncthreads();
    using F0 = std::integral_constant<bool, false>;
    using F1 = std::integral_constant<bool, true>;
    for (int ch = 0; ch < nch; ch += 2) {
        step(ch, I0{}, I1{}, F0{});   // chunk ch is even: ch + 2 goes to set 0, ch + 1 comes from set 1
        if (ch + 1 < nch) step(ch + 1, I1{}, I0{}, F1{});
    }
    if (nch & 1) flush();
    // D layout of the 16x16x4 instruction: lane l holds rows 4 (l / 16) + r, column l % 16
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int col = i0 + wn * WN + b * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = s0 + wm * WM + a * 16 + 4 * kq + r;
                if (row < M && col < n) {
                    if (ACC64)
                        reinterpret_cast<double2*>(Yv)[size_t(yrow[row]) * n + col] =
                            make_double2(dr[ACC64 ? a : 0][ACC64 ? b : 0][r], di[ACC64 ? a : 0][ACC64 ? b : 0][r]);
                    else
                        reinterpret_cast<float2*>(Yv)[size_t(row) * n + col] =
                            make_float2(accr[a][b][r], acci[a][b][r]);
                }
            }
        }
}

bool cgemm_mfma_supported(int M, int n) { return M >= 1 && n >= 1; }

// ------------------------------------------------------------ tile variants
// Block tile BM (right-hand sides) x BN (unknowns), K chunk KC.  The FP64-flush
// path needs 3x the accumulator registers, so smaller wavefront tiles win there;
// efie_gemm_autotune measures and selects per path.
struct Variant {
    int bm, bn, kc;
};
static constexpr Variant kVariants[] = {{64, 32, 32}, {64, 64, 16}, {64, 64, 32}, {128, 32, 16},
                                    {32, 64, 16}, {128, 64, 16}, {64, 32, 16}, {64, 128, 16},
                                    {64, 64, 64}};
static constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
// the last: the fp16 split kernel with the tile of launch_split_rule; the default of
// both paths (complex64 output, FP64-flush output)
static constexpr int kSplitVariant = kNumVariants - 1;
static int g_variant[2] = {kSplitVariant, kSplitVariant};

// X rows readable: mcap >= M; the kernel reads up to the tile's multiple of M
// within them, so that a ragged last tile still takes the unchecked loads
template <int BM, int BN, int KC, bool A64>
static void launch_v(const void* X, const void* Z, void* Y, const int* yrow, int M, int mcap, int n, hipStream_t s) {
    const int nbm = (M + BM - 1) / BM, nbn = (n + BN - 1) / BN;
    const size_t nblk = size_t(nbm) * nbn;
    EFIE_REQUIRE(nblk < (size_t(1) << 31), EFIE_ERR_ARG, "cgemm: problem too large");
    const int mrows = std::max(M, std::min(nbm * BM, mcap));
    hipLaunchKernelGGL((cgemm_planar_kernel<BM, BN, KC, A64>), dim3(unsigned(nblk)), dim3(256), 0, s,
                       static_cast<const float2*>(X), static_cast<const float2*>(Z), Y, M, mrows, n, yrow);
}

template <int WM, int WN, int WK, int KC, bool A64, int MINW>
static void launch_split(const void* X, const void* Z, void* Y, const int* yrow, int M, int n, hipStream_t s) {
    const size_t nblk = size_t((M + 32 * WM - 1) / (32 * WM)) * ((n + 32 * WN - 1) / (32 * WN));
    EFIE_REQUIRE(nblk < (size_t(1) << 31), EFIE_ERR_ARG, "cgemm: problem too large");
    hipLaunchKernelGGL((cgemm_split_kernel<WM, WN, WK, KC, A64 ? OUT_C128 : OUT_C64, MINW>), dim3(unsigned(nblk)),
                       dim3(64 * WM * WN * WK), 0, s, static_cast<const float2*>(X), static_cast<const float2*>(Z), Y, M,
                       n, yrow, 1);
}

// Several blocks per tile, each on a range of K, where the caller has a workspace for
// their partial sums: with 17 to 512 tiles of the in-block split one block per CU, or
// none, is left waiting on its own loads.  The number of ranges is the one that takes
// least by a model of the measured times: a chunk takes full us while two blocks share
// a CU (slots = 512 blocks), last us while at most one is left on each, a partial tile
// tile us to write and to add.  Within 10 % of the times from n = 1920 up; in us, the
// matrix in the last-level cache from the call before where it fits (cold, 4317 x 45
// takes 66), in-block / ranges:
//   n = 4317,  M = 45:  124 /  59 (7 ranges)    n = 1920, M = 100:  55 /  36 (8)
//   n = 7680,  M = 64:  240 / 167 (4)           n =  960, M =  64:  30 /  16 (8)
//   n = 12000, M = 20:  474 / 291 (5)           n =  480, M =  64:  17 /  14 (8)
//   n = 12000, M = 200: 1421 / 1353 (2)         n = 30720, M = 512: one range
struct RangePlan {
    int kind = 0, ranges = 1;
    size_t bytes = 0;   // workspace; 0: in-block
};
constexpr size_t RANGE_WS_MAX = size_t(128) << 20;

static RangePlan range_plan(int M, int n) {
    // kinds: 64 x 64 tiles; for at most 32 right-hand sides 32 x 128 tiles, and 32 x 32
    // with two K groups (chunks of 128 then) where those would be too few
    struct Kind {
        int bm, bn, kc;
        double full, last;
    };
    static constexpr Kind kinds[] = {{64, 64, 64, 4.7, 3.5}, {32, 128, 32, 3.4, 2.2}, {32, 32, 128, 4.7, 3.5}};
    RangePlan best;
    best.kind = M > 32 ? 0 : (n > 2048 ? 1 : 2);
    const Kind& k = kinds[best.kind];
    const int64_t tiles = ((int64_t(M) + k.bm - 1) / k.bm) * ((int64_t(n) + k.bn - 1) / k.bn);
    const int64_t chunks = (int64_t(n) + k.kc - 1) / k.kc;
    const size_t tile_bytes = size_t(k.bm) * size_t(k.bn) * 16;
    double least = 1e300;
    for (int64_t r = 1; r <= std::min<int64_t>(32, chunks); ++r) {
        const size_t bytes = r > 1 ? size_t(tiles * r) * tile_bytes : 0;
        if (bytes > RANGE_WS_MAX) break;
        const int64_t blocks = tiles * r, rest = blocks % 512;
        const double rounds = double(blocks / 512) * k.full + (rest == 0 ? 0.0 : rest <= 256 ? k.last : k.full);
        // and half a microsecond a range in the sum's own chain
        const double t = double((chunks + r - 1) / r) * rounds + double(bytes) / 2.4e6 + 0.5 * double(r);
        if (t < least) {
            least = t;
            best.ranges = int(r);
            best.bytes = bytes;
        }
    }
    return best;
}

size_t cgemm_ranges_bytes(int M, int n) { return range_plan(M, n).bytes; }

template <int WM, int WN, int WK, int KC, bool A64, int MINW>
static void launch_ranges(const void* X, const void* Z, void* Y, const int* yrow, int M, int n, int ranges, void* ws,
                          hipStream_t s) {
    const int ntile = ((M + 32 * WM - 1) / (32 * WM)) * ((n + 32 * WN - 1) / (32 * WN));
    hipLaunchKernelGGL((cgemm_split_kernel<WM, WN, WK, KC, OUT_PART, MINW>), dim3(unsigned(ntile) * unsigned(ranges)),
                       dim3(64 * WM * WN * WK), 0, s, static_cast<const float2*>(X), static_cast<const float2*>(Z), ws, M,
                       n, nullptr, ranges);
    hipLaunchKernelGGL((split_sum_kernel<WM, WN, A64>), dim3(unsigned(ntile) * (4 * WM * WN)), dim3(256), 0, s,
                       static_cast<const double2*>(ws), Y, M, n, yrow, ntile, ranges);
}

// The tile of the split kernel by the number of blocks (256 CUs; times in us with
// 32 x 32 tiles and 4 K groups / 64 x 32 and 4 groups / 64 x 64 / 32 x 32 and 2 groups of
// 64-term chunks):
//   n = 1920,  M = 100:   57 /  57 /  99 /  78        n =  1920, M = 16:  52 /  55 /  98 /  77
//   n = 4317,  M = 45:   241 / 124 / 221 / 174        n =  4320, M = 64: 230 / 121 / 218 / 174
//   n = 12000, M = 33:   986 / 681 / 611 / 942        n = 12000, M = 20: 652 / 679 / 608 / 473
//   n = 7679,  M = 200: 1500 / 873 / 573 / 1188       n = 30720, M = 512: 49.4 / 27.3 / 17.2 / 35.3 ms
// A matrix that gives at most one block per CU is split over K inside the block, by the
// smallest tile that still does; otherwise the widest tile converts the least.
template <bool A64>
static void launch_split_rule(const void* X, const void* Z, void* Y, const int* yrow, int M, int n, hipStream_t s) {
    const int64_t m32 = (M + 31) / 32, m64 = (M + 63) / 64, n32 = (int64_t(n) + 31) / 32;
    if (m32 * n32 <= 256)
        launch_split<1, 1, 4, 32, A64, 2>(X, Z, Y, yrow, M, n, s);
    else if (M <= 32)
        launch_split<1, 1, 2, 64, A64, 2>(X, Z, Y, yrow, M, n, s);
    else if (m64 * n32 <= 256)
        launch_split<2, 1, 4, 32, A64, 2>(X, Z, Y, yrow, M, n, s);
    else
        launch_split<2, 2, 1, 64, A64, 2>(X, Z, Y, yrow, M, n, s);
}

// the split product, over several ranges of K where ws holds their partial sums
template <bool A64>
static void launch_split_ws(const void* X, const void* Z, void* Y, const int* yrow, int M, int n, void* ws,
                            size_t ws_bytes, hipStream_t s) {
    const RangePlan p = range_plan(M, n);
    if (p.bytes == 0 || p.bytes > ws_bytes)
        launch_split_rule<A64>(X, Z, Y, yrow, M, n, s);
    else if (p.kind == 0)
        launch_ranges<2, 2, 1, 64, A64, 2>(X, Z, Y, yrow, M, n, p.ranges, ws, s);
    else if (p.kind == 1)
        launch_ranges<1, 4, 1, 32, A64, 2>(X, Z, Y, yrow, M, n, p.ranges, ws, s);
    else
        launch_ranges<1, 1, 2, 64, A64, 2>(X, Z, Y, yrow, M, n, p.ranges, ws, s);
}

template <bool A64>
static void launch_variant(int v, const void* X, const void* Z, void* Y, const int* yrow, int M, int mcap, int n,
                           hipStream_t s) {
    switch (v) {
        case 0: launch_v<64, 32, 32, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 1: launch_v<64, 64, 16, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 2: launch_v<64, 64, 32, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 3: launch_v<128, 32, 16, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 4: launch_v<32, 64, 16, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 5: launch_v<128, 64, 16, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 6: launch_v<64, 32, 16, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        case 7: launch_v<64, 128, 16, A64>(X, Z, Y, yrow, M, mcap, n, s); break;
        default: launch_split_rule<A64>(X, Z, Y, yrow, M, n, s); break;
    }
}

// the tile of 32 right-hand sides: for few columns it leaves half the matrix-core
// work of the 64-row tiles undone (about 2.5 ms against 4.1 ms at 32 columns, level 5)
constexpr int kSmallVariant = 4;
static_assert(kVariants[kSmallVariant].bm == 32, "the small-M tile has 32 rows");

void cgemm_mfma(const void* X, const void* Z, void* Y, int M, int n, hipStream_t s, int mcap, void* ws,
                size_t ws_bytes) {
    prof_begin(PROF_MFMA, s);
    if (g_variant[0] == kSplitVariant)
        launch_split_ws<false>(X, Z, Y, nullptr, M, n, ws, ws_bytes, s);
    else
        launch_variant<false>(g_variant[0], X, Z, Y, nullptr, M, std::max(M, mcap), n, s);
    prof_end(PROF_MFMA, s, 8.0 * M * double(n) * n);
}

void cgemm_mfma_acc64(const void* X, const void* Z, double2* Y, const int* yrow, int M, int n, hipStream_t s,
                      int mcap, bool small_tile, void* ws, size_t ws_bytes) {
    const bool small = small_tile && M <= kVariants[kSmallVariant].bm;
    const int v = small && g_variant[1] != kSplitVariant ? kSmallVariant : g_variant[1];
    const ProfId id = small ? PROF_MFMA_SMALL : PROF_MFMA;   // timed apart from the selected tile
    prof_begin(id, s);
    if (v == kSplitVariant)
        launch_split_ws<true>(X, Z, Y, yrow, M, n, ws, ws_bytes, s);
    else
        launch_variant<true>(v, X, Z, Y, yrow, M, std::max(M, mcap), n, s);
    prof_end(id, s, 8.0 * M * double(n) * n);
}

__global__ void iota_rows_kernel(int* idx, int M) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < M; i += gridDim.x * blockDim.x) idx[i] = i;
}

void zx_product(const void* Z, int zdt, int n, const void* X, int xdt, void* Y, int nrhs, hipStream_t s, void* ws,
                size_t ws_bytes) {
    if (nrhs == 1) {
        gemv(Z, zdt, n, X, xdt, Y, xdt, s);
    } else if (zdt == EFIE_C64 && xdt == EFIE_C64) {
        cgemm_mfma(X, Z, Y, nrhs, n, s, 0, ws, ws_bytes);
    } else {
        zgemm_nt(X, xdt, Z, zdt, Y, xdt, nrhs, n, n, n, n, n, 1.0, 0.0, false, s);
    }
}

}  // namespace efie

extern "C" int efie_gemm_variants(int* count) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(count != nullptr, EFIE_ERR_ARG, "gemm_variants: null");
        *count = efie::kNumVariants;
        return int(EFIE_OK);
    });
}

extern "C" int efie_gemm_variant_info(int v, int* bm, int* bn, int* kc) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(v >= 0 && v < efie::kNumVariants && bm && bn && kc, EFIE_ERR_ARG, "gemm_variant_info: bad argument");
        *bm = efie::kVariants[v].bm;
        *bn = efie::kVariants[v].bn;
        *kc = efie::kVariants[v].kc;
        return int(EFIE_OK);
    });
}

extern "C" int efie_zx_flush64_workspace_size(int64_t n, int64_t nrhs, size_t* bytes) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(bytes && n >= 1 && n < (int64_t(1) << 31) && nrhs >= 1 && nrhs < 65536, EFIE_ERR_ARG,
                     "zx_flush64_workspace_size: bad argument");
        *bytes = ((size_t(n) * size_t(nrhs) * 8 + 255) & ~size_t(255)) + size_t(nrhs) * sizeof(int);
        return int(EFIE_OK);
    });
}

extern "C" int efie_zx_flush64(const void* Z, int64_t n, const void* X, void* Y, int64_t nrhs, void* ws,
                               size_t ws_bytes, hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(Z && X && Y && ws, EFIE_ERR_ARG, "zx_flush64: null argument");
        EFIE_REQUIRE(n >= 1 && n < (int64_t(1) << 31) && nrhs >= 1 && nrhs < 65536, EFIE_ERR_ARG,
                     "zx_flush64: bad sizes");
        EFIE_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 15) == 0, EFIE_ERR_ARG, "zx_flush64: ws not 16-byte aligned");
        const size_t xbytes = (size_t(n) * size_t(nrhs) * 8 + 255) & ~size_t(255);
        EFIE_REQUIRE(ws_bytes >= xbytes + size_t(nrhs) * sizeof(int), EFIE_ERR_ARG, "zx_flush64: workspace too small");
        float2* x32 = static_cast<float2*>(ws);
        int* idx = reinterpret_cast<int*>(static_cast<char*>(ws) + xbytes);
        hipLaunchKernelGGL(efie::iota_rows_kernel, dim3(int((nrhs + 255) / 256)), dim3(256), 0, stream, idx, int(nrhs));
        efie::gather_cast(static_cast<const double2*>(X), idx, int(nrhs), int(n), x32, stream);
        efie::cgemm_mfma_acc64(x32, Z, static_cast<double2*>(Y), idx, int(nrhs), int(n), stream);
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}

extern "C" int efie_gemm_select(int acc64, int variant, int* previous) {
    return efie::guarded([&]() {
        EFIE_REQUIRE((acc64 == 0 || acc64 == 1) && variant >= 0 && variant < efie::kNumVariants, EFIE_ERR_ARG,
                     "gemm_select: bad argument");
        if (previous) *previous = efie::g_variant[acc64];
        efie::g_variant[acc64] = variant;
        return int(EFIE_OK);
    });
}

extern "C" int efie_gemm_autotune(const void* Z, int64_t n, const void* X, int64_t M, int acc64, void* ws,
                                  size_t ws_bytes, int reps, double* ms, int* best, hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(Z && X && ws && ms && best && reps >= 1, EFIE_ERR_ARG, "gemm_autotune: bad argument");
        EFIE_REQUIRE(n >= 1 && n < (int64_t(1) << 31) && M >= 1 && M < 65536, EFIE_ERR_ARG, "gemm_autotune: bad sizes");
        const size_t ybytes = size_t(M) * size_t(n) * (acc64 ? 16 : 8);
        const size_t need = ((ybytes + 255) & ~size_t(255)) + size_t(M) * sizeof(int);
        EFIE_REQUIRE(ws_bytes >= need, EFIE_ERR_ARG, "gemm_autotune: workspace too small");
        void* Y = ws;
        // the split product as efie_zx_ws and the solves run it, where the rest of ws holds its partial sums
        const size_t after = (need + 255) & ~size_t(255);
        char* part = ws_bytes > after ? static_cast<char*>(ws) + after : nullptr;
        if (reinterpret_cast<uintptr_t>(part) & 15) part = nullptr;
        const size_t part_bytes = part ? ws_bytes - after : 0;
        int* idx = reinterpret_cast<int*>(static_cast<char*>(ws) + ((ybytes + 255) & ~size_t(255)));
        hipLaunchKernelGGL(efie::iota_rows_kernel, dim3(int((M + 255) / 256)), dim3(256), 0, stream, idx, int(M));
        hipEvent_t e0, e1;
        EFIE_HIP_CHECK(hipEventCreate(&e0));
        EFIE_HIP_CHECK(hipEventCreate(&e1));
        double best_ms = 1e300;
        *best = 0;
        for (int v = 0; v < efie::kNumVariants; ++v) {
            auto run = [&]() {
                if (v == efie::kSplitVariant && acc64)
                    efie::launch_split_ws<true>(X, Z, Y, idx, int(M), int(n), part, part_bytes, stream);
                else if (v == efie::kSplitVariant)
                    efie::launch_split_ws<false>(X, Z, Y, nullptr, int(M), int(n), part, part_bytes, stream);
                else if (acc64)
                    efie::launch_variant<true>(v, X, Z, Y, idx, int(M), int(M), int(n), stream);
                else
                    efie::launch_variant<false>(v, X, Z, Y, nullptr, int(M), int(M), int(n), stream);
            };
            run();   // warm-up
            EFIE_HIP_CHECK(hipEventRecord(e0, stream));
            for (int r = 0; r < reps; ++r) run();
            EFIE_HIP_CHECK(hipEventRecord(e1, stream));
            EFIE_HIP_CHECK(hipEventSynchronize(e1));
            float t = 0.f;
            EFIE_HIP_CHECK(hipEventElapsedTime(&t, e0, e1));
            ms[v] = double(t) / reps;
            best_ms = std::min(best_ms, ms[v]);
        }
        // the first variant (in table order) within 2 % of the fastest: near-equal
        // tiles are not swapped by timing noise from one run to the next
        for (int v = efie::kNumVariants - 1; v >= 0; --v)
            if (ms[v] <= 1.02 * best_ms) *best = v;
        EFIE_HIP_CHECK(hipEventDestroy(e0));
        EFIE_HIP_CHECK(hipEventDestroy(e1));
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}

extern "C" int efie_zx(const void* Z, int dtype, int64_t n, const void* X, void* Y, int64_t nrhs,
                       hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(Z && X && Y, EFIE_ERR_ARG, "zx: null argument");
        EFIE_REQUIRE(dtype == EFIE_C128 || dtype == EFIE_C64, EFIE_ERR_ARG, "zx: bad dtype");
        EFIE_REQUIRE(n >= 1 && n < (int64_t(1) << 31) && nrhs >= 1 && nrhs < 65536, EFIE_ERR_ARG, "zx: bad sizes");
        efie::zx_product(Z, dtype, int(n), X, dtype, Y, int(nrhs), stream);
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}

extern "C" int efie_zx_workspace_size(int64_t n, int64_t nrhs, int dtype, size_t* bytes) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(bytes && n >= 1 && n < (int64_t(1) << 31) && nrhs >= 1 && nrhs < 65536, EFIE_ERR_ARG,
                     "zx_workspace_size: bad argument");
        EFIE_REQUIRE(dtype == EFIE_C128 || dtype == EFIE_C64, EFIE_ERR_ARG, "zx_workspace_size: bad dtype");
        *bytes = dtype == EFIE_C64 && nrhs > 1 ? efie::cgemm_ranges_bytes(int(nrhs), int(n)) : 0;
        return int(EFIE_OK);
    });
}

extern "C" int efie_zx_ws(const void* Z, int dtype, int64_t n, const void* X, void* Y, int64_t nrhs, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
    return efie::guarded([&]() {
        EFIE_REQUIRE(Z && X && Y, EFIE_ERR_ARG, "zx_ws: null argument");
        EFIE_REQUIRE(dtype == EFIE_C128 || dtype == EFIE_C64, EFIE_ERR_ARG, "zx_ws: bad dtype");
        EFIE_REQUIRE(n >= 1 && n < (int64_t(1) << 31) && nrhs >= 1 && nrhs < 65536, EFIE_ERR_ARG, "zx_ws: bad sizes");
        EFIE_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 15) == 0, EFIE_ERR_ARG, "zx_ws: ws not 16-byte aligned");
        efie::zx_product(Z, dtype, int(n), X, dtype, Y, int(nrhs), stream, ws, ws ? ws_bytes : 0);
        EFIE_HIP_CHECK(hipGetLastError());
        return int(EFIE_OK);
    });
}
