// LU factorization with partial pivoting and the solve that uses it: the
// Linpack (HPL) workload of the paper's Section IV-C, on the sgemm path.
//
// Recursive right-looking LU: factor the left half of the column range,
// L11^{-1} A12 (recursive triangular solve), A22 -= A21 A12 (one sgemm --
// the rank-k trailing update), factor A22.  Almost all flops land in sgemm
// calls of decreasing size.  The leaves are panels of 64 columns that one
// launch factors with their rows in the registers of several workgroups
// (lu.panel.hpp); panels of more rows than those hold are factored in memory
// by one workgroup, 8 columns at a time.  Each panel's row interchanges are
// applied to every other column of the matrix right after it, which gives
// the same result as swapping at each level of the recursion (a column
// receives the interchanges in pivot order either way, and the columns right
// of a range are not touched before its left half is done).  The solve
// applies the interchanges to the right-hand sides and then the two
// triangular solves; with few right-hand sides the interchanges run in LDS
// and the triangular recursion stops at 1024-row diagonal blocks that one
// workgroup solves.
#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

#include "../../include/misgemm.h"
#include "lu.panel.hpp"

namespace {

constexpr int LEAF = 64;            // rows of a leaf triangular solve (one per lane)
constexpr int TALL_PANEL = 8;       // columns of a panel factored in memory
constexpr int TALL_THREADS = 1024;
constexpr int SWAP_BLOCK = 32;      // interchanges composed into one permutation
constexpr int SWAP_THREADS = 256;   // laswp workgroup: four wavefronts
constexpr int SWAP_COLS_PER_WAVE = 16;
// One-workgroup triangular solve for a few right-hand sides (the solve
// after the factorization): up to TRSV_ROWS rows per launch, used when the
// right-hand sides number at most TRSV_MAX_RHS.
constexpr int TRSV_ROWS = 1024;
constexpr int64_t TRSV_MAX_RHS = 16;
// Rows of a column whose interchanges are applied in LDS (the column and
// the pivot list: 8 bytes per row).
constexpr int LASWP_LDS_ROWS = 16384;

__device__ inline uint64_t readlane64(uint64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Panels taller than the register kernel takes.
__global__ __launch_bounds__(TALL_THREADS) void lu_panel_tall_kernel(float *__restrict__ P,
                                                                    int64_t lda, int64_t m, int w,
                                                                    int64_t *__restrict__ ipiv,
                                                                    int64_t row0,
                                                                    int *__restrict__ info)
{
    panel_in_memory<TALL_THREADS>(P, lda, m, w, ipiv, row0, info);
}

// Row interchanges k0..k1-1, in order (row k with row ipiv[k]; an entry
// outside [0, nrows) is skipped), on ncols columns of C (row 0 of the
// matrix, leading dimension ldc).  Column index c is matrix column c below
// gap0 and c + gapw from there on, so that a band of gapw columns is left
// alone.  The interchanges are taken SWAP_BLOCK at a time and each block is
// composed into one permutation of at most 2 * SWAP_BLOCK rows ("slots":
// slot i < nb is row k + i, a row outside the block takes slot nb + i for
// the first i that names it).  Each wavefront composes the permutation with
// lane s tracking slot s, then moves SWAP_COLS_PER_WAVE columns: S lanes
// per column (S = the power of two >= 2 nb), lane s loading the row of
// slot s, receiving the value its slot ends up with from the lane that
// loaded it, and storing it -- one load and one store per moved element,
// no chain of dependent swaps.
template <int S>
__device__ inline void laswp_move(float *__restrict__ C, int64_t ldc, int64_t ncols, int64_t gap0,
                                  int64_t gapw, int64_t cbase, int lane, int64_t row, int content)
{
    constexpr int CPP = 64 / S;                       // columns per pass
    constexpr int PASSES = SWAP_COLS_PER_WAVE / CPP;
    const int s = lane & (S - 1), g = lane / S;
    const int64_t rs = __shfl(row, s);
    const int fs = __shfl(content, s);
    const bool moved = rs >= 0 && fs != s;
    float val[PASSES];
    float *colp[PASSES];
#pragma unroll
    for (int q = 0; q < PASSES; ++q) {
        int64_t c = cbase + q * CPP + g;
        const bool act = moved && c < ncols;
        if (c >= gap0) c += gapw;
        colp[q] = act ? C + c * ldc : nullptr;
        val[q] = act ? colp[q][rs] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < PASSES; ++q) {
        const float nv = __shfl(val[q], g * S + fs);
        if (colp[q]) colp[q][rs] = nv;
    }
}

// One wavefront's share of the interchanges: columns cbase ..
// cbase + SWAP_COLS_PER_WAVE - 1 (those below ncols) of C, lane t.
__device__ inline void laswp_wave(float *__restrict__ C, int64_t ldc, int64_t nrows, int64_t ncols,
                                  int64_t gap0, int64_t gapw, const int64_t *__restrict__ ipiv,
                                  int64_t k0, int64_t k1, int64_t cbase, int t)
{
    for (int64_t kb = k0; kb < k1; kb += SWAP_BLOCK) {
        const int nb = (int)(k1 - kb < SWAP_BLOCK ? k1 - kb : SWAP_BLOCK);
        int64_t p = -1;
        if (t < nb) {
            p = ipiv[kb + t];
            if (p < 0 || p >= nrows) p = kb + t;
        }
        // the composition reads uniform lanes: scalar readlanes, not the
        // LDS-routed lane shuffles (it is the dependent chain of a launch)
        int first = t;
        for (int i = 0; i < nb; ++i) {
            const int64_t q = (int64_t)readlane64((uint64_t)p, i);
            if (i < t && q == p && first == t) first = i;
        }
        int pslot = -1;
        if (t < nb) pslot = (p >= kb && p < kb + nb) ? (int)(p - kb) : nb + first;
        // row of slot t
        const int src = t >= nb ? t - nb : 0;
        const int64_t q = __shfl(p, src);
        const int qs = __shfl(pslot, src);
        int64_t row = -1;
        if (t < nb) row = kb + t;
        else if (t < 2 * nb && qs == t) row = q;
        // compose: content = slot whose original value ends in slot t
        int content = t;
        for (int i = 0; i < nb; ++i) {
            const int b = __builtin_amdgcn_readlane(pslot, i);
            const int ca = __builtin_amdgcn_readlane(content, i);
            const int cb = __builtin_amdgcn_readlane(content, b);
            if (t == i) content = cb;
            else if (t == b) content = ca;
        }
        if (nb <= 8)
            laswp_move<16>(C, ldc, ncols, gap0, gapw, cbase, t, row, content);
        else if (nb <= 16)
            laswp_move<32>(C, ldc, ncols, gap0, gapw, cbase, t, row, content);
        else
            laswp_move<64>(C, ldc, ncols, gap0, gapw, cbase, t, row, content);
    }
}

__global__ __launch_bounds__(SWAP_THREADS) void laswp_kernel(
    float *__restrict__ C, int64_t ldc, int64_t nrows, int64_t ncols, int64_t gap0, int64_t gapw,
    const int64_t *__restrict__ ipiv, int64_t k0, int64_t k1)
{
    const int t = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t cbase =
        ((int64_t)blockIdx.x * (SWAP_THREADS / 64) + wave) * SWAP_COLS_PER_WAVE;
    if (cbase >= ncols) return;  // whole wavefront past the last column
    laswp_wave(C, ldc, nrows, ncols, gap0, gapw, ipiv, k0, k1, cbase, t);
}

// The interchanges k0 .. k1-1 on column blockIdx.x of C (nrows <=
// LASWP_LDS_ROWS rows, k1 - k0 <= nrows), for the solve's few right-hand
// sides: the column and the pivot list are staged in LDS, one lane applies
// the interchanges one by one in order (each an LDS round trip, with the
// pivot reads independent of the column), and the column is written back.
// Entries outside [0, nrows) are skipped.
__global__ __launch_bounds__(SWAP_THREADS) void laswp_lds_kernel(float *__restrict__ C,
                                                                int64_t ldc, int nrows,
                                                                const int64_t *__restrict__ ipiv,
                                                                int64_t k0, int64_t k1)
{
    __shared__ float col[LASWP_LDS_ROWS];
    __shared__ int piv[LASWP_LDS_ROWS];
    float *c = C + (int64_t)blockIdx.x * ldc;
    for (int i = threadIdx.x; i < nrows; i += SWAP_THREADS) col[i] = c[i];
    for (int64_t k = k0 + threadIdx.x; k < k1; k += SWAP_THREADS) {
        const int64_t p = ipiv[k];
        piv[k - k0] = (int)((p < 0 || p >= nrows) ? k : p);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int n = (int)(k1 - k0), base = (int)k0;
        for (int i = 0; i < n; ++i) {
            const int r = base + i, p = piv[i];
            const float a = col[r], b = col[p];
            col[r] = b;
            col[p] = a;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nrows; i += SWAP_THREADS) c[i] = col[i];
}

// B (n x ncols, n <= N) := T^{-1} B for T the n x n lower unit (UPPER
// false) or upper (UPPER true) triangle at T.  N lanes per column (lane i
// holds row i of T and x_i), 64 / N columns per wavefront; x_k reaches the
// other rows once it is final, by a lane shuffle (a scalar broadcast when
// the wavefront holds one column).  The lower solve takes
// the terms of x_i in the order k = 0, 1, ..., i-1; the upper one in the
// order k = n-1, ..., i+1, then divides by the diagonal.
template <bool UPPER, int N>
__global__ __launch_bounds__(256) void trsm_leaf_kernel(const float *__restrict__ T, int64_t ldt,
                                                       float *__restrict__ B, int64_t ldb, int n,
                                                       int64_t ncols)
{
    constexpr int CPW = 64 / N;
    const int lane = threadIdx.x & 63, i = lane % N, g = lane / N;
    const int64_t c = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * CPW + g;
    const bool act = c < ncols && i < n;
    float trow[N];
#pragma unroll
    for (int k = 0; k < N; ++k) trow[k] = (i < n && k < n) ? T[i + (int64_t)k * ldt] : 0.0f;
    float x = act ? B[c * ldb + i] : 0.0f;
    if (!UPPER) {
#pragma unroll
        for (int k = 0; k < N - 1; ++k) {
            const float xk = N == 64 ? lane_value(x, k) : __shfl(x, g * N + k);
            if (i > k) x -= trow[k] * xk;
        }
    } else {
#pragma unroll
        for (int k = N - 1; k >= 0; --k) {
            if (i == k && k < n) x = x / trow[k];
            const float xk = N == 64 ? lane_value(x, k) : __shfl(x, g * N + k);
            if (i < k) x -= trow[k] * xk;
        }
    }
    if (act) B[c * ldb + i] = x;
}

// B (n x 1, n <= TRSV_ROWS, column blockIdx.x of B) := T^{-1} B for T the
// lower unit (UPPER false) or upper (UPPER true) triangle, one workgroup per
// right-hand side: wave w holds rows 64w .. 64w+63 (lane = row) in a
// register, and the 64-row blocks are taken in the solve's order (lower:
// first to last, upper: last to first).  The wave that owns block k
// finishes its rows, each final value broadcast from its lane through a
// scalar register (the terms in the triangular leaves' order), and posts
// them to LDS; after one barrier every wave whose rows
// still depend on block k subtracts its contribution, with the entries of T
// it needs loaded before the barrier.  No row reads another row's value
// before that row is final, so the sums are those of substitution by
// blocks.
template <bool UPPER>
__global__ __launch_bounds__(TRSV_ROWS) void trsv_block_kernel(const float *__restrict__ T,
                                                              int64_t ldt, float *__restrict__ B,
                                                              int64_t ldb, int n)
{
    __shared__ float xs[TRSV_ROWS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = wave * 64 + lane;
    const bool live = r < n;
    float *b = B + (int64_t)blockIdx.x * ldb;
    float x = live ? b[r] : 0.0f;
    const int nb = (n + 63) / 64;
    for (int step = 0; step < nb; ++step) {
        const int k = UPPER ? nb - 1 - step : step;
        const bool needs = UPPER ? wave <= k : wave >= k;  // rows that depend on block k
        float tv[64];
        const float *tc = T + (int64_t)k * 64 * ldt;      // column 64k of T
#pragma unroll
        for (int q = 0; q < 64; ++q)
            tv[q] = (needs && live && k * 64 + q < n) ? tc[(int64_t)q * ldt + r] : 0.0f;
        if (wave == k) {
            if (!UPPER) {
#pragma unroll
                for (int q = 0; q < 63; ++q) {
                    const float xq = lane_value(x, q);
                    if (lane > q) x -= tv[q] * xq;
                }
            } else {
                // Each row's quotient by its diagonal entry: where every
                // diagonal entry of the block is a normal number, through
                // its reciprocal (computed before the dependent chain) and
                // one correction step, q0 = x d', x = q0 + (x - q0 d) d'
                // with both updates fused (correctly rounded for a correctly
                // rounded d', so exact wherever the quotient is
                // representable); otherwise by division, so that a zero or
                // non-finite diagonal gives what x / d gives.
                float dg = 1.0f;
#pragma unroll
                for (int q = 0; q < 64; ++q) dg = q == lane ? tv[q] : dg;
                const bool normal = !live || (fabsf(dg) >= FLT_MIN && fabsf(dg) <= FLT_MAX);
                if (__all(normal)) {
                    const float rdg = 1.0f / dg;
#pragma unroll
                    for (int q = 63; q >= 0; --q) {
                        if (lane == q && live) {
                            const float q0 = x * rdg;
                            x = fmaf(fmaf(-q0, dg, x), rdg, q0);
                        }
                        const float xq = lane_value(x, q);
                        if (lane < q) x -= tv[q] * xq;
                    }
                } else {
#pragma unroll
                    for (int q = 63; q >= 0; --q) {
                        if (lane == q && live) x = x / tv[q];
                        const float xq = lane_value(x, q);
                        if (lane < q) x -= tv[q] * xq;
                    }
                }
            }
            xs[r] = x;
        }
        __syncthreads();
        if (needs && wave != k) {
            if (!UPPER) {
#pragma unroll
                for (int q = 0; q < 64; ++q) x -= tv[q] * xs[k * 64 + q];
            } else {
#pragma unroll
                for (int q = 63; q >= 0; --q) x -= tv[q] * xs[k * 64 + q];
            }
        }
    }
    if (live) b[r] = x;
}

// info = 0 and ipiv = 0: the panels' messages travel through the entries that
// are not final yet, and a message word that was never written has tag 0.
__global__ __launch_bounds__(256) void lu_init_kernel(int64_t n, int64_t *__restrict__ ipiv,
                                                      int *__restrict__ info)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) *info = 0;
    if (i < n) ipiv[i] = 0;
}

struct Lu {
    float *A;
    int64_t lda, n;
    int64_t *ipiv;
    int *info;
    int mode;
    hipStream_t s;
    // bounds of a panel's start: the first workgroup's wait for the others and
    // the others' for its word
    int wait_polls, word_polls;
    int max_groups;  // workgroups of a panel; taller ones are factored in memory
};

int check(hipError_t e) { return e == hipSuccess ? 0 : (int)e; }

int gemm(const Lu &c, int64_t m, int64_t n, int64_t k, const float *A, int64_t lda,
         const float *B, int64_t ldb, float *C, int64_t ldc)
{
    if (m == 0 || n == 0 || k == 0) return 0;
    return misgemm_sgemm('N', 'N', m, n, k, -1.0f, A, lda, B, ldb, 1.0f, C, ldc, c.mode, c.s);
}

// Interchanges k0..k1-1 on ncols columns of C (all rows of the matrix),
// skipping the band of gapw columns at gap0.
int laswp(const Lu &c, float *C, int64_t ldc, int64_t ncols, int64_t gap0, int64_t gapw,
          int64_t k0, int64_t k1)
{
    constexpr int cols_per_block = SWAP_THREADS / 64 * SWAP_COLS_PER_WAVE;
    const int64_t blocks = k1 > k0 ? (ncols + cols_per_block - 1) / cols_per_block : 0;
    if (blocks <= 0) return 0;
    hipLaunchKernelGGL(laswp_kernel, dim3((unsigned)blocks), dim3(SWAP_THREADS), 0, c.s, C, ldc,
                       c.n, ncols, gap0, gapw, c.ipiv, k0, k1);
    return check(hipGetLastError());
}

template <bool UPPER, int N>
void launch_trsm_leaf_n(const Lu &c, const float *T, int64_t ldt, float *B, int64_t ldb, int n,
                        int64_t ncols)
{
    constexpr int cols_per_block = 4 * (64 / N);
    const dim3 grid((unsigned)((ncols + cols_per_block - 1) / cols_per_block)), block(256);
    hipLaunchKernelGGL((trsm_leaf_kernel<UPPER, N>), grid, block, 0, c.s, T, ldt, B, ldb, n,
                       ncols);
}

template <bool UPPER>
void launch_trsm_leaf(const Lu &c, const float *T, int64_t ldt, float *B, int64_t ldb, int n,
                      int64_t ncols)
{
    if (n <= 8) launch_trsm_leaf_n<UPPER, 8>(c, T, ldt, B, ldb, n, ncols);
    else if (n <= 16) launch_trsm_leaf_n<UPPER, 16>(c, T, ldt, B, ldb, n, ncols);
    else if (n <= 32) launch_trsm_leaf_n<UPPER, 32>(c, T, ldt, B, ldb, n, ncols);
    else launch_trsm_leaf_n<UPPER, LEAF>(c, T, ldt, B, ldb, n, ncols);
}

template <bool UPPER>
void launch_trsv_block(const Lu &c, const float *T, int64_t ldt, float *B, int64_t ldb, int n,
                       int64_t ncols)
{
    hipLaunchKernelGGL((trsv_block_kernel<UPPER>), dim3((unsigned)ncols), dim3(TRSV_ROWS), 0,
                       c.s, T, ldt, B, ldb, n);
}

// B (n x ncols) := T^{-1} B, T lower unit or upper n x n, recursively: the
// off-diagonal block goes through sgemm.  few_rhs (ncols <= TRSV_MAX_RHS)
// ends the recursion at TRSV_ROWS rows with the one-workgroup solve.
int trsm(const Lu &c, bool upper, const float *T, int64_t ldt, float *B, int64_t ldb, int64_t n,
         int64_t ncols, bool few_rhs = false)
{
    if (n == 0 || ncols == 0) return 0;
    if (few_rhs && n <= TRSV_ROWS && ncols <= TRSV_MAX_RHS) {
        if (upper)
            launch_trsv_block<true>(c, T, ldt, B, ldb, (int)n, ncols);
        else
            launch_trsv_block<false>(c, T, ldt, B, ldb, (int)n, ncols);
        return check(hipGetLastError());
    }
    if (n <= LEAF) {
        if (upper)
            launch_trsm_leaf<true>(c, T, ldt, B, ldb, (int)n, ncols);
        else
            launch_trsm_leaf<false>(c, T, ldt, B, ldb, (int)n, ncols);
        return check(hipGetLastError());
    }
    const int64_t h = (n / 2 + LEAF - 1) / LEAF * LEAF;
    int rc;
    if (!upper) {
        if ((rc = trsm(c, false, T, ldt, B, ldb, h, ncols, few_rhs))) return rc;
        if ((rc = gemm(c, n - h, ncols, h, T + h, ldt, B, ldb, B + h, ldb))) return rc;
        return trsm(c, false, T + h + h * ldt, ldt, B + h, ldb, n - h, ncols, few_rhs);
    }
    if ((rc = trsm(c, true, T + h + h * ldt, ldt, B + h, ldb, n - h, ncols, few_rhs))) return rc;
    if ((rc = gemm(c, h, ncols, n - h, T + h * ldt, ldt, B + h, ldb, B, ldb))) return rc;
    return trsm(c, true, T, ldt, B, ldb, h, ncols, few_rhs);
}

// Rows per thread of the panel kernel for an m-row panel.  One row less is
// 0.5 us less of a column's own work, more workgroups cost more to exchange:
// 64 columns of 1024 rows take 106 us as one workgroup of two rows per thread
// and 123 as two of one; 2048 rows 158 and 127 us, 4608 rows 171 and 146, 8192
// rows 165 and 194 (before the block's products were summed apart, which adds
// 1 us to each).
int panel_rpt(int64_t m)
{
    if (m <= 2 * PANEL_THREADS) return m <= PANEL_THREADS ? 1 : 2;
    return m <= (int64_t)NEAR * PANEL_THREADS ? 1 : 2;
}
int64_t panel_groups(int64_t m)
{
    const int64_t rows = (int64_t)PANEL_THREADS * panel_rpt(m);
    return (m + rows - 1) / rows;
}

// Columns of a panel of m rows.
int64_t panel_width(const Lu &c, int64_t m)
{
    return panel_groups(m) <= c.max_groups ? PANEL : TALL_PANEL;
}

// Factor the panel at P (m x w, top-left element A(j0, j0)).
int panel(const Lu &c, float *P, int64_t m, int w, int64_t j0)
{
    const int64_t groups = panel_groups(m);
    if (groups > c.max_groups) {
        hipLaunchKernelGGL(lu_panel_tall_kernel, dim3(1), dim3(TALL_THREADS), 0, c.s, P, c.lda, m,
                           w, c.ipiv, j0, c.info);
        return check(hipGetLastError());
    }
    // The messages take the last entries of ipiv (down to a 128-byte line),
    // which lie past this panel's: every workgroup but the last brings 512 or
    // more rows, i.e. entries, for its 160 words.
    uint64_t *words = reinterpret_cast<uint64_t *>(
        reinterpret_cast<uintptr_t>(c.ipiv + (c.n - groups * MSG_WORDS)) &
        ~(uintptr_t)(MSG_ALIGN * 8 - 1));
    // One XCD while its CUs hold the workgroups twice over (the block index
    // modulo 8 picks the XCD, calls with other matrices another one); all
    // XCDs beyond that.
    const bool one_xcd = groups > 1 && groups <= PANEL_XCD_GROUPS;
    const int stride = one_xcd ? 8 : 1;
    const int first = one_xcd ? (int)((reinterpret_cast<uintptr_t>(c.A) >> 21) & 7) : 0;
    const dim3 grid((unsigned)(groups * stride)), block(PANEL_THREADS);
    if (panel_rpt(m) == 1)
        hipLaunchKernelGGL((lu_panel_kernel<1>), grid, block, 0, c.s, P, c.lda, (int)m, w, c.ipiv,
                           j0, c.info, words, (int)groups, first, stride, c.wait_polls,
                           c.word_polls);
    else
        hipLaunchKernelGGL((lu_panel_kernel<2>), grid, block, 0, c.s, P, c.lda, (int)m, w, c.ipiv,
                           j0, c.info, words, (int)groups, first, stride, c.wait_polls,
                           c.word_polls);
    return check(hipGetLastError());
}

// Factor columns j0 .. j0+w-1 over rows j0 .. n-1.
int getrf(const Lu &c, int64_t j0, int64_t w)
{
    const int64_t m = c.n - j0;
    float *P = c.A + j0 + j0 * c.lda;
    const int64_t pw = panel_width(c, m);
    int rc;
    if (w <= pw) {
        if ((rc = panel(c, P, m, (int)w, j0))) return rc;
        // this panel's interchanges on every other column
        return laswp(c, c.A, c.lda, c.n - w, j0, w, j0, j0 + w);
    }
    const int64_t w1 = (w / 2 + pw - 1) / pw * pw, w2 = w - w1;
    if ((rc = getrf(c, j0, w1))) return rc;
    if ((rc = trsm(c, false, P, c.lda, P + w1 * c.lda, c.lda, w1, w2))) return rc;
    if ((rc = gemm(c, m - w1, w2, w1, P + w1, c.lda, P + w1 * c.lda, c.lda,
                   P + w1 + w1 * c.lda, c.lda)))
        return rc;
    return getrf(c, j0 + w1, w2);
}

bool lu_mode_ok(int mode) { return mode == MISGEMM_FP32 || mode == MISGEMM_BF16X3; }

}  // namespace

extern "C" {

int misgemm_sgetrf_limited(int64_t n, float *A, int64_t lda, int64_t *ipiv, int *info, int mode,
                           int wait_polls, int word_polls, int max_groups, void *stream)
{
    if (n < 0) return -1;
    if (n > 0 && A == nullptr) return -2;
    if (lda < (n > 0 ? n : 1)) return -3;
    if (n > 0 && ipiv == nullptr) return -4;
    if (info == nullptr) return -5;
    if (!lu_mode_ok(mode)) return -6;
    if (n > ((int64_t)1 << 31)) return MISGEMM_E_TOO_LARGE;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(lu_init_kernel, dim3((unsigned)(n / 256 + 1)), dim3(256), 0, s, n, ipiv,
                       info);
    int rc = check(hipGetLastError());
    if (rc != 0 || n == 0) return rc;
    const Lu c{A, lda, n, ipiv, info, mode, s, wait_polls, word_polls,
               max_groups < PANEL_GROUPS ? max_groups : PANEL_GROUPS};
    return getrf(c, 0, n);
}

int misgemm_sgetrf_waiting(int64_t n, float *A, int64_t lda, int64_t *ipiv, int *info, int mode,
                           int wait_polls, void *stream)
{
    return misgemm_sgetrf_limited(n, A, lda, ipiv, info, mode, wait_polls, PANEL_WORD_WAIT,
                                  PANEL_GROUPS, stream);
}

int misgemm_sgetrf(int64_t n, float *A, int64_t lda, int64_t *ipiv, int *info, int mode,
                   void *stream)
{
    return misgemm_sgetrf_limited(n, A, lda, ipiv, info, mode, PANEL_WAIT, PANEL_WORD_WAIT,
                                  PANEL_GROUPS, stream);
}

int misgemm_sgetrs(int64_t n, int64_t nrhs, const float *A, int64_t lda, const int64_t *ipiv,
                   float *B, int64_t ldb, int mode, void *stream)
{
    if (n < 0) return -1;
    if (nrhs < 0) return -2;
    if (n > 0 && A == nullptr) return -3;
    if (lda < (n > 0 ? n : 1)) return -4;
    if (n > 0 && ipiv == nullptr) return -5;
    if (n > 0 && nrhs > 0 && B == nullptr) return -6;
    if (ldb < (n > 0 ? n : 1)) return -7;
    if (!lu_mode_ok(mode)) return -8;
    if (n == 0 || nrhs == 0) return 0;
    const Lu c{const_cast<float *>(A), lda, n, const_cast<int64_t *>(ipiv), nullptr, mode,
               (hipStream_t)stream, 0, 0, 0};
    const bool few = nrhs <= TRSV_MAX_RHS;
    int rc = 0;
    if (few && n <= LASWP_LDS_ROWS) {
        hipLaunchKernelGGL(laswp_lds_kernel, dim3((unsigned)nrhs), dim3(SWAP_THREADS), 0, c.s, B,
                           ldb, (int)n, ipiv, (int64_t)0, n);
        rc = check(hipGetLastError());
    } else {
        rc = laswp(c, B, ldb, nrhs, nrhs, 0, 0, n);
    }
    if (rc == 0) rc = trsm(c, false, A, lda, B, ldb, n, nrhs, few);
    if (rc == 0) rc = trsm(c, true, A, lda, B, ldb, n, nrhs, few);
    return rc;
}

}  // extern "C"
