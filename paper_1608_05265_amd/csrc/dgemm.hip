// Double-precision GEMM (the paper's dgemm variants, Section IV-B).
//
//   * FP64: v_mfma_f64_16x16x4_f64 on FP64 matrix cores, FP64 accumulation,
//     the same blocked scheme as the FP32 tiles (K blocks staged into LDS in
//     one canonical layout, double-buffered, alpha/beta fused into the
//     store).
//   * FP32 compute ("false dgemm"): op(A), op(B) rounded to FP32, the product
//     on the FP32 path with FP32 accumulation, alpha and beta applied in FP64
//     to the widened result -- the paper's workaround of sending FP64 data
//     through the single-precision kernel, here as two conversion passes
//     around the sgemm path.
#include "dgemm.hpp"
#include "registry.hpp"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace misgemm {

typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex2u __attribute__((ext_vector_type(2), aligned(8)));  // at any double address
typedef double doublex4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// FP64 staging: LDS holds X as Xs[kk][r] (r contiguous, row length LD
// doubles).  A chunk is two consecutive elements along the stored
// contiguous direction (one 16-byte load).  Row length: R + 16 (even, for
// the 16-byte stores) when r is the stored contiguous direction; R + 17 when
// the slice is transposed on the way in, so that the 8-byte stores of 16
// lanes (eight k values times two rows) hit 16 distinct bank pairs.
// ---------------------------------------------------------------------------
template <int R, int BK, int NT, bool KC>
struct StageF64 {
    static constexpr int CH = R * BK / 2;            // 2-element chunks per tile
    static constexpr int S = (CH + NT - 1) / NT;
    static constexpr int LD = KC ? R + 17 : R + 16;
    static constexpr int ELEMS = BK * LD;
    doublex2 v[S];

    __device__ __forceinline__ static void chunk(int c, int &r, int &kk)
    {
        if (KC) { kk = (c % (BK / 2)) * 2; r = c / (BK / 2); }
        else    { r = (c % (R / 2)) * 2;   kk = c / (R / 2); }
    }

    static constexpr int MIN_ROWS = KC ? 1 : 2;  // rows an EDGE load needs

    // MODE: see LoadMode.  EDGE, two rows at one k: the 16-byte load starts
    // at most at row rows - 2 and store() shifts a chunk that straddles the
    // last row.
    template <LoadMode MODE>
    __device__ __forceinline__ void load(const double *X, int64_t ld, int64_t r0, int64_t k0,
                                         int64_t rows, int64_t kdim, int tid)
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int c = tid + s * NT;
            if (CH % NT != 0 && c >= CH) break;
            int r, kk;
            chunk(c, r, kk);
            int64_t gr = r0 + r;
            const int64_t gk = k0 + kk;
            if (MODE == MASKED) {
                const double *p = KC ? X + gk + gr * ld : X + gr + gk * ld;
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    v[s][e] = (KC ? gr < rows && gk + e < kdim : gk < kdim && gr + e < rows)
                                  ? p[e] : 0.0;
            } else {
                if (MODE == EDGE) gr = min64(gr, rows - MIN_ROWS);
                v[s] = *reinterpret_cast<const doublex2u *>(KC ? X + gk + gr * ld
                                                               : X + gr + gk * ld);
            }
        }
    }

    template <LoadMode MODE>
    __device__ __forceinline__ void store(double *Xs, int64_t r0, int64_t rows, int tid) const
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int c = tid + s * NT;
            if (CH % NT != 0 && c >= CH) break;
            int r, kk;
            chunk(c, r, kk);
            if (KC) {
                Xs[kk * LD + r] = v[s][0];
                Xs[(kk + 1) * LD + r] = v[s][1];
            } else {
                doublex2 x = v[s];
                if (MODE == EDGE && r0 + r + 1 == rows) x[0] = x[1];
                *reinterpret_cast<doublex2 *>(Xs + kk * LD + r) = x;
            }
        }
    }
};

struct DArgs {
    int64_t m, n, k;
    const double *A;
    const double *B;
    double *C;
    int64_t lda, ldb, ldc;
    double alpha, beta;
};

// ---------------------------------------------------------------------------
// FP64 tile: BM x BN per workgroup, waves of WM x WN made of 16x16 MFMA
// blocks.  Operand layout of v_mfma_f64_16x16x4_f64 for lane l: A element
// (row l%16, k l/16), B element (k l/16, column l%16); result element e of
// lane l is row l/16 + 4e of column l%16 (measured on the device with
// one-hot operands: unlike the FP32 16x16 layout, a lane's four rows are
// spaced by four).
//
// KW: the waves of a workgroup are KW groups that each cover the whole tile
// and take 1/KW of the K steps of every block; their sums are added through
// LDS at the end, in the order of the groups.
//
// What bounds it: the matrix cores (64 cycles per 16x16x4, 76.5 TFLOP/s over
// the card), as long as nothing else of a wave stands between two of its
// MFMAs for longer than one of them takes.  A wave issues in order, so
// whatever comes in one lump -- the fragment reads of a K step, the LDS
// stores and the loads of the next blocks -- leaves its matrix core idle.
// Therefore every other instruction is dealt out between the MFMAs
// (sched_group_barrier); the loads run two blocks ahead of their LDS stores
// (two register sets), the stores one block ahead of their reads and the
// reads one K step ahead of their MFMAs, across the barrier too, which
// stands before the last K step of a block.  With two register sets, but
// stores, barrier and reads in lumps at the ends of a block, 2048^3 took
// 259-271 us; with one set 287-316 us; now 248-252 us (69 TFLOP/s).
// ---------------------------------------------------------------------------
template <int BM_, int BN_, int BK_, int WM_, int WN_, int KW_, int OCC_>
struct DShape {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, KW = KW_, OCC = OCC_;
    static constexpr int NWM = BM / WM, NWN = BN / WN, NT = 64 * NWM * NWN * KW;
    static_assert(BM % WM == 0 && BN % WN == 0 && BK % (4 * KW) == 0, "whole waves and K steps");
    static_assert(WM % 16 == 0 && WN % 16 == 0, "wave tile is made of 16x16 blocks");
};

template <class SH, bool TA, bool TB>
struct F64Tile {
    static constexpr int RM = SH::WM / 16, RN = SH::WN / 16;
    using SA = StageF64<SH::BM, SH::BK, SH::NT, TA>;   // A is K-contiguous when transposed
    using SB = StageF64<SH::BN, SH::BK, SH::NT, !TB>;  // B is K-contiguous when not transposed
    static constexpr int STAGE = SA::ELEMS + SB::ELEMS;
    static constexpr int SUMS = (SH::KW - 1) * SH::BM * SH::BN;
    static constexpr int LDS_BYTES = (2 * STAGE > SUMS ? 2 * STAGE : SUMS) * 8;

    struct Frags {
        double a[RM], b[RN];
        __device__ __forceinline__ void read(const double *As, const double *Bs, int kr)
        {
#pragma unroll
            for (int i = 0; i < RM; ++i) a[i] = As[kr * SA::LD + i * 16];
#pragma unroll
            for (int j = 0; j < RN; ++j) b[j] = Bs[kr * SB::LD + j * 16];
        }
        __device__ __forceinline__ void multiply(doublex4 (&acc)[RM][RN]) const
        {
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };

    __device__ __forceinline__ static void epilogue(const DArgs &g, const doublex4 (&acc)[RM][RN],
                                                    int64_t row0, int64_t col0, int lane)
    {
        const int q = lane >> 4, c16 = lane & 15;
        const bool use_c0 = g.beta != 0.0;
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            const int64_t col = col0 + j * 16 + c16;
            if (col >= g.n) continue;
            double *cc = g.C + col * g.ldc;
#pragma unroll
            for (int i = 0; i < RM; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // lanes q = 0..3 of a column hold rows 4e + q: each store
                    // instruction writes 32 contiguous bytes per column
                    const int64_t row = row0 + i * 16 + 4 * e + q;
                    if (row < g.m) {
                        double o = g.alpha * acc[i][j][e];
                        if (use_c0) o += g.beta * cc[row];
                        cc[row] = o;
                    }
                }
            }
        }
    }

    __device__ __forceinline__ static void run(const DArgs &g, int64_t m0, int64_t n0, char *smem)
    {
        if (m0 + SH::BM <= g.m && n0 + SH::BN <= g.n) run_impl<INTERIOR>(g, m0, n0, smem);
        else if (g.m >= SA::MIN_ROWS && g.n >= SB::MIN_ROWS) run_impl<EDGE>(g, m0, n0, smem);
        else run_impl<MASKED>(g, m0, n0, smem);
    }

    template <LoadMode MODE>
    __device__ __forceinline__ static void run_impl(const DArgs &g, int64_t m0, int64_t n0,
                                                    char *smem)
    {
        double *lds = reinterpret_cast<double *>(smem);
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int wm = wave % SH::NWM, wn = wave / SH::NWM % SH::NWN, wk = wave / (SH::NWM * SH::NWN);
        const int kq = lane >> 4, r16 = lane & 15;

        doublex4 acc[RM][RN];
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};

        const KBlocks<SH::BK> kb(g.k);
        const int blocks = (int)kb.count;  // op(A) alone would fill the memory before 2^31
        SA sa[2];  // block b + 1 is in set b & 1
        SB sb[2];
        if (blocks > 0) load_first<MODE>(sa[0], sb[0], g, m0, n0, kb, lds, lds + SA::ELEMS, tid);
        auto load = [&](int set, int b) {
            sa[set].template load<MODE>(g.A, g.lda, m0, kb.at(b), g.m, g.k, tid);
            sb[set].template load<MODE>(g.B, g.ldb, n0, kb.at(b), g.n, g.k, tid);
        };
        if (blocks > 1) load(0, 1);
        if (blocks > 2) load(1, 2);
        __syncthreads();
        constexpr int KS = SH::BK / 4 / SH::KW;  // K steps of this wave
        static_assert(KS % 2 == 0, "a block starts with the fragments in f[0]");
        const int kr = wk * KS * 4 + kq;
        const int ao = wm * SH::WM + r16, bo = SA::ELEMS + wn * SH::WN + r16;
        Frags f[2];
        if (blocks > 0) f[0].read(lds + ao, lds + bo, kr);
        // Block b of the K loop, in LDS stage `set`.  whole: blocks b + 1 to
        // b + 3 exist, so the step is straight-line code.
        auto step = [&](auto whole, int b, int set) {
            constexpr bool WHOLE = decltype(whole)::value;
            const double *cur = lds + set * STAGE;
            double *nxt = lds + (set ^ 1) * STAGE;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks + 1 < KS) {
                    f[(ks + 1) & 1].read(cur + ao, cur + bo, kr + (ks + 1) * 4);
                } else {
                    // every wave has stored its part of block b + 1 and has
                    // read the last of block b
                    __syncthreads();
                    if (WHOLE || b + 1 < blocks) f[0].read(nxt + ao, nxt + bo, kr);
                }
                f[ks & 1].multiply(acc);
                if (ks == 0 && (WHOLE || b + 1 < blocks)) {
                    sa[set].template store<MODE>(nxt, m0, g.m, tid);
                    sb[set].template store<MODE>(nxt + SA::ELEMS, n0, g.n, tid);
                }
                if (ks == (KS > 2 ? 1 : 0) && (WHOLE || b + 3 < blocks)) load(set, b + 3);
#pragma unroll
                for (int q = 0; q < RM * RN; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // an MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // an LDS write
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // a load
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int b = 0;
        for (; b + 4 < blocks; b += 2) {
            step(std::true_type{}, b, 0);
            step(std::true_type{}, b + 1, 1);
        }
        for (; b + 1 < blocks; b += 2) {
            step(std::false_type{}, b, 0);
            step(std::false_type{}, b + 1, 1);
        }
        if (b < blocks) step(std::false_type{}, b, 0);
        if (SH::KW > 1) {
            __syncthreads();
            doublex4 *sums = reinterpret_cast<doublex4 *>(lds) +
                             (wm + wn * SH::NWM) * (RM * RN * 64) + lane;
            constexpr int GROUP = SH::NWM * SH::NWN * RM * RN * 64;
            if (wk > 0) {
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RN; ++j)
                        sums[(wk - 1) * GROUP + (i * RN + j) * 64] = acc[i][j];
            }
            __syncthreads();
            if (wk > 0) return;
#pragma unroll
            for (int w = 0; w < SH::KW - 1; ++w)
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RN; ++j) acc[i][j] += sums[w * GROUP + (i * RN + j) * 64];
        }
        epilogue(g, acc, m0 + wm * SH::WM, n0 + wn * SH::WN, lane);
    }
};

template <class TILE, class SH>
__global__ __launch_bounds__(SH::NT, SH::OCC) void dgemm_kernel(DArgs g, int64_t tiles_m,
                                                                int64_t tiles_n, int group_m)
{
    __shared__ __attribute__((aligned(16))) char smem[TILE::LDS_BYTES];
    const int64_t t = xcd_remap(blockIdx.x, gridDim.x);
    int64_t tm, tn;
    tile_coords(t, tiles_m, tiles_n, group_m, tm, tn);
    TILE::run(g, tm * SH::BM, tn * SH::BN, smem);
}

template <class SH>
hipError_t launch_dgemm_shape(int ta, int tb, const DArgs &g, hipStream_t s)
{
    const int64_t tm = (g.m + SH::BM - 1) / SH::BM, tn = (g.n + SH::BN - 1) / SH::BN;
    const dim3 grid((unsigned)(tm * tn)), block(SH::NT);
    const int gm = GROUP_M_DEFAULT;
    if (!ta && !tb) hipLaunchKernelGGL((dgemm_kernel<F64Tile<SH, false, false>, SH>), grid, block, 0, s, g, tm, tn, gm);
    else if (!ta && tb) hipLaunchKernelGGL((dgemm_kernel<F64Tile<SH, false, true>, SH>), grid, block, 0, s, g, tm, tn, gm);
    else if (ta && !tb) hipLaunchKernelGGL((dgemm_kernel<F64Tile<SH, true, false>, SH>), grid, block, 0, s, g, tm, tn, gm);
    else hipLaunchKernelGGL((dgemm_kernel<F64Tile<SH, true, true>, SH>), grid, block, 0, s, g, tm, tn, gm);
    return hipGetLastError();
}

// Tile choice.  A call takes as long as its fullest CU: the tiles on it times
// the operations of one, over the share of the matrix rate that the shape
// reaches.  Measured shares, alone on a CU and with others on it: 64x64 0.87
// and 0.93 (larger tiles are no faster: 128x64 237-264 us and 128x128
// 241-252 us against 239-259 us at 2048^3); 32x32 in two K groups 0.67 and
// 0.83; 32x32 in four K groups 0.7; 16x16 in eight K groups 0.4, eight waves
// on a tile that one MFMA covers.  Both sides of the lines, in us:
//   1024^3            64x64 36.6   32x32 40.7
//   768^3             64x64 28.6   32x32 24.8
//   1511x777x1003     64x64 69.9   32x32 50.7
//   512x512x2048      32x32 27.9   in four groups 24.0   16x16 29.5
//   256x256x4096      64x64 122    32x32 in four groups 39.9   16x16 21.9
//   64x64x4096        64x64 122    32x32 in four groups 38.6   16x16 15.8
// A launch holds less than 2^32 threads: a tile shape that would need more
// (16x16 on 16 rows by 2^27 columns) is left out, and a call too large for
// 64x64 tiles is cut along its longer side, up to the size that 128x128 tiles
// of 256 threads could take.
hipError_t launch_dgemm_fp64(int ta, int tb, int64_t m, int64_t n, int64_t k, double alpha,
                             const double *A, int64_t lda, const double *B, int64_t ldb,
                             double beta, double *C, int64_t ldc, int cus, hipStream_t s)
{
    DArgs g;
    g.m = m; g.n = n; g.k = k;
    g.A = A; g.B = B; g.C = C;
    g.lda = lda; g.ldb = ldb; g.ldc = ldc;
    g.alpha = alpha; g.beta = beta;
    auto tiles = [&](int64_t edge) { return ((m + edge - 1) / edge) * ((n + edge - 1) / edge); };
    if ((double)((m + 127) / 128) * (double)((n + 127) / 128) * 256 > UINT32_MAX)
        return hipErrorInvalidConfiguration;
    if (tiles(64) * 256 > UINT32_MAX) {
        const int64_t half = (std::max(m, n) / 2 + 63) / 64 * 64;
        const bool rows = m > n;
        const hipError_t e = launch_dgemm_fp64(ta, tb, rows ? half : m, rows ? n : half, k, alpha, A,
                                               lda, B, ldb, beta, C, ldc, cus, s);
        if (e != hipSuccess) return e;
        if (rows)
            return launch_dgemm_fp64(ta, tb, m - half, n, k, alpha, A + (ta ? half * lda : half), lda,
                                     B, ldb, beta, C + half, ldc, cus, s);
        return launch_dgemm_fp64(ta, tb, m, n - half, k, alpha, A, lda, B + (tb ? half : half * ldb),
                                 ldb, beta, C + half * ldc, ldc, cus, s);
    }
    auto cost = [&](int edge, int threads, double share) {
        const int64_t t = tiles(edge);
        return t * threads > UINT32_MAX ? INFINITY
                                        : (double)((t + cus - 1) / cus) * edge * edge / share;
    };
    const bool alone = tiles(32) <= cus;  // a 32x32 tile per CU
    const double c64 = cost(64, 256, 0.9), mid = cost(32, 256, alone ? 0.7 : 0.78),
                 c16 = cost(16, 512, 0.4);
    if (c16 < mid && c16 < c64) return launch_dgemm_shape<DShape<16, 16, 64, 16, 16, 8, 2>>(ta, tb, g, s);
    if (c64 <= mid) return launch_dgemm_shape<DShape<64, 64, 16, 32, 32, 1, 2>>(ta, tb, g, s);
    if (alone) return launch_dgemm_shape<DShape<32, 32, 64, 32, 16, 4, 2>>(ta, tb, g, s);
    return launch_dgemm_shape<DShape<32, 32, 32, 32, 16, 2, 2>>(ta, tb, g, s);
}

// ---------------------------------------------------------------------------
// FP32-compute path helpers.
// ---------------------------------------------------------------------------
// y[i] = (float)x[i], round to nearest even, for i < count.
__global__ __launch_bounds__(256) void narrow_kernel(const double *__restrict__ x, int64_t count,
                                                    float *__restrict__ y)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * 256)
        y[i] = (float)x[i];
}

hipError_t launch_narrow(const double *x, int64_t count, float *y, hipStream_t s)
{
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(narrow_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, count, y);
    return hipGetLastError();
}

// C[i + j*ldc] = alpha * P[i + j*m] + beta * C[i + j*ldc] in FP64 (C not
// read when beta == 0).
__global__ __launch_bounds__(256) void widen_kernel(const float *__restrict__ P, int64_t m,
                                                   int64_t n, double alpha, double beta,
                                                   double *__restrict__ C, int64_t ldc)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    for (int64_t j = blockIdx.y; j < n; j += gridDim.y) {
        double v = alpha * (double)P[i + j * m];
        if (beta != 0.0) v += beta * C[i + j * ldc];
        C[i + j * ldc] = v;
    }
}

hipError_t launch_widen(const float *P, int64_t m, int64_t n, double alpha, double beta,
                        double *C, int64_t ldc, hipStream_t s)
{
    const int64_t gx = (m + 255) / 256;
    const int64_t gy = n < 65535 ? n : 65535;
    hipLaunchKernelGGL(widen_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s, P, m, n,
                       alpha, beta, C, ldc);
    return hipGetLastError();
}

// C = beta * C for FP64 (alpha == 0 or k == 0; beta == 0 writes zeros).
__global__ __launch_bounds__(256) void dscale_kernel(double beta, double *__restrict__ C,
                                                    int64_t m, int64_t n, int64_t ldc)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    for (int64_t j = blockIdx.y; j < n; j += gridDim.y) {
        double *p = C + i + j * ldc;
        *p = beta == 0.0 ? 0.0 : beta * *p;
    }
}

hipError_t launch_dscale(double beta, double *C, int64_t m, int64_t n, int64_t ldc,
                         hipStream_t s)
{
    const int64_t gx = (m + 255) / 256;
    const int64_t gy = n < 65535 ? n : 65535;
    hipLaunchKernelGGL(dscale_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s, beta, C,
                       m, n, ldc);
    return hipGetLastError();
}

}  // namespace misgemm
