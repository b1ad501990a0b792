// Device code of the sgemm path for gfx950 (CDNA4).
//
// One workgroup computes one BM x BN tile of C over the whole K range, the
// GPU form of the paper's blocked scheme (Section III-C): K is consumed in
// BK-wide blocks, each block of op(A) and op(B) is staged ("packed") from
// HBM into LDS in one canonical layout that no longer depends on the
// transposes or leading dimensions, the partial products are accumulated in
// registers for all of K (the "accumulator" variant of Section III-C), the
// next block is fetched while the current one is multiplied (the paper's
// double-buffered input transfer), and alpha/beta are applied once at the
// end (the post-processing of Section III-C), fused into the store.
//
// Two arithmetic forms share the staging/epilogue skeleton:
//   * F32:    v_mfma_f32_32x32x2_f32, FP32 in, FP32 accumulate.
//   * BF16X3: every FP32 element is split while it is staged into three
//             bf16 parts x = x0 + x1 + x2 (round to nearest even), and the six
//             part products with index sum <= 2 run on
//             v_mfma_f32_32x32x16_bf16 with FP32 accumulation.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace misgemm {

typedef float floatx4 __attribute__((ext_vector_type(4)));
// The same four floats in memory at any float address: global memory takes
// 16-byte accesses at 4-byte alignment, so neither the base nor the leading
// dimension of a matrix has to be a multiple of 16 bytes.
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Arguments of one GEMM, as seen by a workgroup.
struct GemmArgs {
    int64_t m, n, k;
    const float *A;
    const float *B;
    float *C;
    int64_t lda, ldb, ldc;
    float alpha, beta;
    // Split-K (read only by the split kernels): this workgroup computes the
    // K range of split `split` of `splits` for tile `tile`; its partial sums
    // go to `part`.
    float *part;
    int64_t tile;
    int split, splits;
};

// ---------------------------------------------------------------------------
// Tile shape: BM x BN per workgroup, BK per K block, WM x WN per wave.
// ---------------------------------------------------------------------------
// OCC_: waves per SIMD the register allocation must leave room for
// (a launch bound; 8-wave tiles get two per SIMD by construction).
template <int BM_, int BN_, int BK_, int WM_, int WN_, int OCC_ = 1>
struct Shape {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, OCC = OCC_;
    static constexpr int NWM = BM / WM, NWN = BN / WN, NW = NWM * NWN, NT = 64 * NW;
    static constexpr int RM = WM / 32, RN = WN / 32;  // 32x32 MFMA blocks per wave
    static_assert(BM % WM == 0 && BN % WN == 0, "wave tiles must divide the tile");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile is made of 32x32 blocks");
};

// Element (r, kk) of an op(X) tile lives at X[kk + r*ld] when the stored
// matrix is contiguous along K (KC = true: A transposed, B not transposed)
// and at X[r + kk*ld] otherwise.

// How a K block of an operand is loaded.  A block is MASKED only when it is
// the ragged end of K (taken first, see k_blocks) or the matrix is smaller
// than one vector; every other block of every tile is loaded without a mask,
// so the K loop is straight-line code with 16-byte loads at every size.
// (Masking each element of every block of a tile as soon as k, a leading
// dimension or a base was not a multiple of the block or of 16 bytes ran
// 2047^3 at 70 TFLOP/s and 4095^3 at 83-109, against 104-115 and 133 for the
// next multiple of 64.)
enum LoadMode {
    INTERIOR,  // the whole BM x BN tile is in range
    EDGE,      // rows past the last are loaded from valid ones: an output row
               // or column depends on its own row of op(A) or op(B) only, and
               // those past the end are never stored
    MASKED     // elements outside the matrix read as zero
};

// K blocks in the order they are consumed: when k is no multiple of BK the
// ragged block (the last k % BK of them) comes first, so that it is the
// prologue's load and the loop has whole blocks only.
template <int BK>
struct KBlocks {
    int64_t count;   // blocks in all
    int64_t first;   // k offset of block 0
    int64_t base;    // block b >= 1 starts at base + b * BK
    bool ragged;     // block 0 is the ragged one
    __device__ __forceinline__ explicit KBlocks(int64_t k)
    {
        const int64_t full = k / BK;
        ragged = full * BK != k;
        count = full + (ragged ? 1 : 0);
        first = ragged ? full * BK : 0;
        base = ragged ? -BK : 0;
    }
    __device__ __forceinline__ int64_t at(int64_t b) const { return base + b * BK; }  // b >= 1
};

__device__ __forceinline__ int64_t min64(int64_t a, int64_t b) { return a < b ? a : b; }

// ---------------------------------------------------------------------------
// F32 staging: LDS holds X as Xs[kk][r] (r contiguous, row length LD).
// ---------------------------------------------------------------------------
template <int R, int BK, int NT, bool KC>
struct StageF32 {
    static constexpr int CH = R * BK / 4;            // float4 chunks per tile
    static constexpr int S = (CH + NT - 1) / NT;     // chunks per thread
    static constexpr int LD = R + (KC ? 2 : 4);      // LDS row length (floats)
    static constexpr int FLOATS = BK * LD;
    floatx4 v[S];

    __device__ __forceinline__ void chunk(int c, int &r, int &kk) const
    {
        if (KC) { kk = (c % (BK / 4)) * 4; r = c / (BK / 4); }
        else    { r = (c % (R / 4)) * 4;   kk = c / (R / 4); }
    }

    // Rows (of the stored contiguous direction) an EDGE load needs.
    static constexpr int MIN_ROWS = KC ? 1 : 4;

    // MODE: see LoadMode.  EDGE, four rows at one k: the 16-byte load starts
    // at most at row rows - 4 and store() shifts a chunk that straddles the
    // last row into place.
    template <LoadMode MODE>
    __device__ __forceinline__ void load_chunk(int s, const float *X, int64_t ld, int64_t r0,
                                               int64_t k0, int64_t rows, int64_t kdim, int tid)
    {
        const int c = tid + s * NT;
        if (CH % NT != 0 && c >= CH) return;
        int r, kk;
        chunk(c, r, kk);
        int64_t gr = r0 + r;
        const int64_t gk = k0 + kk;
        if (MODE == MASKED) {
            const float *p = KC ? X + gk + gr * ld : X + gr + gk * ld;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[s][e] = (KC ? gr < rows && gk + e < kdim : gk < kdim && gr + e < rows)
                              ? p[e] : 0.0f;
        } else {
            if (MODE == EDGE) gr = min64(gr, rows - MIN_ROWS);
            v[s] = *reinterpret_cast<const floatx4u *>(KC ? X + gk + gr * ld : X + gr + gk * ld);
        }
    }

    template <LoadMode MODE>
    __device__ __forceinline__ void load(const float *X, int64_t ld, int64_t r0, int64_t k0,
                                         int64_t rows, int64_t kdim, int tid)
    {
#pragma unroll
        for (int s = 0; s < S; ++s) load_chunk<MODE>(s, X, ld, r0, k0, rows, kdim, tid);
    }

    // r0, rows as in the load of the same MODE.
    template <LoadMode MODE>
    __device__ __forceinline__ void store_chunk(int s, float *Xs, int64_t r0, int64_t rows,
                                                int tid) const
    {
        const int c = tid + s * NT;
        if (CH % NT != 0 && c >= CH) return;
        int r, kk;
        chunk(c, r, kk);
        floatx4 x = v[s];
        if (KC) {
#pragma unroll
            for (int e = 0; e < 4; ++e) Xs[(kk + e) * LD + r] = x[e];
        } else {
            if (MODE == EDGE) {
                const int64_t past = r0 + r + 4 - rows;  // 1..3: the load started past rows early
                if (past & 1) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; }
                if (past & 2) { x[0] = x[2]; x[1] = x[3]; }
                if (past <= 0) x = v[s];
            }
            *reinterpret_cast<floatx4 *>(Xs + kk * LD + r) = x;
        }
    }

    template <LoadMode MODE>
    __device__ __forceinline__ void store(float *Xs, int64_t r0, int64_t rows, int tid) const
    {
#pragma unroll
        for (int s = 0; s < S; ++s) store_chunk<MODE>(s, Xs, r0, rows, tid);
    }
};

// ---------------------------------------------------------------------------
// BF16X3 staging: LDS holds, per part t, Xs[t][r][kk] (kk contiguous, row
// length LD bf16), so one 16-byte LDS read gives a lane the eight K values
// a 32x32x16 bf16 MFMA operand needs.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void split3(float x, __bf16 &h0, __bf16 &h1, __bf16 &h2)
{
    h0 = (__bf16)x;            // round to nearest even
    float r = x - (float)h0;   // exact
    h1 = (__bf16)r;
    r = r - (float)h1;         // exact
    h2 = (__bf16)r;
}

template <int R, int BK, int NT, bool KC>
struct StageX3 {
    // Row stride of 16*(BK/8 + 1) bytes: the 16-byte reads and writes of 32
    // consecutive rows fall in distinct LDS banks.
    static constexpr int LD = BK + 8;                  // bf16 per LDS row
    static constexpr int PART = R * LD;                // bf16 per part
    static constexpr int HALVES = 3 * PART;            // bf16 per operand tile
    // A chunk is eight consecutive k of one row; consecutive threads take
    // consecutive rows.
    static constexpr int KS = 8;
    static constexpr int CH = R * BK / KS;
    static constexpr int S = (CH + NT - 1) / NT;
    static constexpr bool UNITS_FULL = CH % NT == 0;
    static constexpr int UNITS = S;
    float v[S][KS];

    __device__ __forceinline__ static void chunk(int c, int &r, int &kk)
    {
        r = c % R;
        kk = (c / R) * KS;
    }

    static constexpr int MIN_ROWS = 1;

    template <LoadMode MODE>
    __device__ __forceinline__ void load(const float *X, int64_t ld, int64_t r0, int64_t k0,
                                         int64_t rows, int64_t kdim, int tid)
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int c = tid + s * NT;
            if (!UNITS_FULL && c >= CH) break;
            int r, kk;
            chunk(c, r, kk);
            int64_t gr = r0 + r;
            const int64_t gk = k0 + kk;
            if (MODE == EDGE) gr = min64(gr, rows - 1);
            const float *p = KC ? X + gk + gr * ld : X + gr + gk * ld;
            if (MODE == MASKED) {
                const bool in_r = gr < rows;
#pragma unroll
                for (int e = 0; e < KS; ++e)
                    v[s][e] = (in_r && gk + e < kdim) ? p[KC ? e : e * ld] : 0.0f;
            } else if (KC) {
                const floatx4 x0 = *reinterpret_cast<const floatx4u *>(p);
                const floatx4 x1 = *reinterpret_cast<const floatx4u *>(p + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[s][e] = x0[e]; v[s][4 + e] = x1[e]; }
            } else {
#pragma unroll
                for (int e = 0; e < KS; ++e) v[s][e] = p[e * ld];
            }
        }
    }

    __device__ __forceinline__ float unit_val(int u, int e) const { return v[u][e]; }

    __device__ __forceinline__ static int unit_offset(int u, int tid)
    {
        int r, kk;
        chunk(tid + u * NT, r, kk);
        return r * LD + kk;
    }

    // Split the eight values of unit u and write the three parts.
    __device__ __forceinline__ void store_unit(__bf16 *Xs, int u, int tid) const
    {
        bf16x8 p0, p1, p2;
#pragma unroll
        for (int e = 0; e < KS; ++e) {
            __bf16 h0, h1, h2;
            split3(v[u][e], h0, h1, h2);
            p0[e] = h0;
            p1[e] = h1;
            p2[e] = h2;
        }
        __bf16 *base = Xs + unit_offset(u, tid);
        *reinterpret_cast<bf16x8 *>(base) = p0;
        *reinterpret_cast<bf16x8 *>(base + PART) = p1;
        *reinterpret_cast<bf16x8 *>(base + 2 * PART) = p2;
    }

    template <LoadMode MODE>
    __device__ __forceinline__ void store(__bf16 *Xs, int64_t, int64_t, int tid) const
    {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (!UNITS_FULL && tid + s * NT >= CH) break;
            store_unit(Xs, s, tid);
        }
    }
};

// ---------------------------------------------------------------------------
// Epilogue: C = alpha * acc + beta * C0 for one wave's 32x32 blocks.
// MFMA 32x32 output layout: lane l, register 4g + e holds row
// 8g + 4*(l/32) + e, column l % 32, so each lane owns four consecutive rows
// of one column (one 16-byte store in column-major C).
// ---------------------------------------------------------------------------
// beta == 0: C0 is not read.  C0 and C are one array, so as far as the
// compiler knows a store may alias any later load, and no load moves above
// an earlier store: loaded one 16-byte group at a time, every group would
// cost the wave a full memory round trip.  The C0 loads of EPI_GROUP groups
// are therefore issued together ahead of their stores (one round trip per
// EPI_GROUP groups, 4 * EPI_GROUP more VGPRs; 4 keeps the 128x128 tiles at
// three waves per SIMD, 8 does not).
constexpr int EPI_GROUP = 4;

template <int RM, int RN>
__device__ __forceinline__ void epilogue(const GemmArgs &g, const floatx16 (&acc)[RM][RN],
                                         int64_t row0, int64_t col0, int lane)
{
    const int half = lane >> 5, l32 = lane & 31;
    const bool use_c0 = g.beta != 0.0f;
    constexpr int NG = RN * RM * 4;                       // 16-byte groups per lane
    constexpr int GG = EPI_GROUP < NG ? EPI_GROUP : NG;
    static_assert(NG % GG == 0, "whole load groups");
#pragma unroll
    for (int g0 = 0; g0 < NG; g0 += GG) {
        floatx4 c0[GG];
#pragma unroll
        for (int q = 0; q < GG; ++q) {
            const int idx = g0 + q, rn = idx / (RM * 4), rm = (idx / 4) % RM, gi = idx % 4;
            const int64_t col = col0 + rn * 32 + l32;
            const int64_t row = row0 + rm * 32 + gi * 8 + half * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) c0[q][e] = 0.0f;
            if (use_c0 && col < g.n && row + 4 <= g.m)
                c0[q] = *reinterpret_cast<const floatx4u *>(g.C + col * g.ldc + row);
        }
#pragma unroll
        for (int q = 0; q < GG; ++q) {
            const int idx = g0 + q, rn = idx / (RM * 4), rm = (idx / 4) % RM, gi = idx % 4;
            const int64_t col = col0 + rn * 32 + l32;
            const int64_t row = row0 + rm * 32 + gi * 8 + half * 4;
            if (col >= g.n || row >= g.m) continue;
            float *p = g.C + col * g.ldc + row;
            floatx4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = g.alpha * acc[rm][rn][gi * 4 + e];
            if (row + 4 <= g.m) {
                if (use_c0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[e] += g.beta * c0[q][e];
                }
                *reinterpret_cast<floatx4u *>(p) = out;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (row + e < g.m) {
                        float o = out[e];
                        if (use_c0) o += g.beta * p[e];
                        p[e] = o;
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// End of a tile.  A whole-K tile applies alpha/beta and stores.  A split-K
// tile (SPLIT) stores its raw partial accumulator instead; a second kernel
// (splitk_reduce) adds the partials of all splits in split order and runs
// the epilogue, so the result does not depend on the order in which the
// splits ran.  Partial layout: for split s of tile t, float4 group q of
// thread x is at part[((t * splits + s) * Q + q) * NT + x] (Q = RM*RN*4
// groups per thread), so each store instruction of a wave writes 1 KB
// contiguously.
// ---------------------------------------------------------------------------
template <int RM, int RN>
__device__ __forceinline__ int64_t partial_index(int64_t tile, int splits, int split, int q,
                                                 int tid, int nt)
{
    return ((tile * splits + split) * (int64_t)(RM * RN * 4) + q) * nt + tid;
}

template <bool SPLIT, int RM, int RN>
__device__ __forceinline__ void finish(const GemmArgs &g, const floatx16 (&acc)[RM][RN],
                                       int64_t row0, int64_t col0, int tid, int nt)
{
    if constexpr (SPLIT) {
        floatx4 *const part = reinterpret_cast<floatx4 *>(g.part);
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    floatx4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[i][j][q4 * 4 + e];
                    part[partial_index<RM, RN>(g.tile, g.splits, g.split, (i * RN + j) * 4 + q4,
                                               tid, nt)] = v;
                }
    } else {
        epilogue<RM, RN>(g, acc, row0, col0, tid & 63);
    }
}

// The first K block of a tile into LDS (masked when it is the ragged one).
template <LoadMode MODE, class SA, class SB, class ARGS, int BK, class T>
__device__ __forceinline__ void load_first(SA &sa, SB &sb, const ARGS &g, int64_t m0,
                                           int64_t n0, const KBlocks<BK> &kb, T *as, T *bs,
                                           int tid)
{
    if (MODE != MASKED && kb.ragged) {
        sa.template load<MASKED>(g.A, g.lda, m0, kb.first, g.m, g.k, tid);
        sb.template load<MASKED>(g.B, g.ldb, n0, kb.first, g.n, g.k, tid);
        sa.template store<MASKED>(as, m0, g.m, tid);
        sb.template store<MASKED>(bs, n0, g.n, tid);
    } else {
        sa.template load<MODE>(g.A, g.lda, m0, kb.first, g.m, g.k, tid);
        sb.template load<MODE>(g.B, g.ldb, n0, kb.first, g.n, g.k, tid);
        sa.template store<MODE>(as, m0, g.m, tid);
        sb.template store<MODE>(bs, n0, g.n, tid);
    }
}

// ---------------------------------------------------------------------------
// Small tiles for grids that leave CUs idle (a 256^3 problem has 16 tiles of
// 64x64): every one of KW waves holds the whole BM x BN tile and takes every
// KW-th K step of each staged block, so a tile's MFMA chain is KW times
// shorter; at the end the waves' accumulators are added in wave order
// through LDS and wave 0 stores.  The partial sums of one element therefore
// run over the k steps s = w (mod KW) of wave w, and the result is the same
// bits for every launch.
// ---------------------------------------------------------------------------
template <int BM_, int BN_, int BK_, int KW_>
struct WShape {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, KW = KW_, OCC = BM_ * BN_ > 1024 ? 2 : 4;
    static constexpr int WM = BM, WN = BN, NWM = 1, NWN = 1, NW = KW, NT = 64 * KW;
    static constexpr int RM = BM / 32, RN = BN / 32;
    static_assert(BM % 32 == 0 && BN % 32 == 0, "the tile is made of 32x32 blocks");
};

// Waves 1..KW-1 post their accumulators to LDS (lane-contiguous, so every
// store and load of a wave is conflict-free), wave 0 adds them in wave
// order.  The caller's K loop ended with a barrier, so the staging buffers
// are free.
template <int KW, int RM, int RN>
__device__ __forceinline__ void wave_sum(floatx16 (&acc)[RM][RN], float *lds, int wave,
                                         int lane)
{
    constexpr int PER = RM * RN * 16 * 64;
    if (wave > 0) {
        float *dst = lds + (wave - 1) * PER;
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) dst[((i * RN + j) * 16 + e) * 64 + lane] = acc[i][j][e];
    }
    __syncthreads();
    if (wave == 0) {
        for (int w = 1; w < KW; ++w) {
            const float *src = lds + (w - 1) * PER;
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        acc[i][j][e] += src[((i * RN + j) * 16 + e) * 64 + lane];
        }
    }
}

template <class SH>
constexpr auto k_waves_of(int) -> decltype(SH::KW) { return SH::KW; }
template <class SH>
constexpr int k_waves_of(...) { return 1; }
template <class SH>
constexpr int k_waves() { return k_waves_of<SH>(0); }

// ---------------------------------------------------------------------------
// The FP32 tile: stage -> multiply -> epilogue for tile (m0, n0).
//
// What bounds it: the matrix cores (64 cycles per 32x32x2), as long as
// nothing else of a wave stands between two of its MFMAs for longer than one
// of them takes.  A wave issues in order: fragment reads, LDS stores, loads
// and barrier in lumps cost a wave with one 32x32 block 550 of every 1575
// cycles, at any number of LDS stages, load distance or waves per SIMD that
// kept the lumps.  So the K loop is straight-line code (but for its last
// blocks) in groups of four MFMAs or more, with everything else dealt out
// between them: the fragments of the next group, across the barrier of a
// block too, which stands before its last group; the LDS stores of the next
// block and the loads of the one after (two after, in a second register set,
// where a set is small).
// TFLOP/s, lumped -> dealt out (NN): 1024x1024x4096 64x64x32 84 -> 109,
// 2048^3 128x128x16 99 -> 132 and 64x64x32 110 -> 120, 4096^3 256x256x16
// 136 -> 147, 8192x8192x256 128x128x16 109 -> 119.
// ---------------------------------------------------------------------------
template <class SH, bool TA, bool TB>
struct F32Tile {
    using SA = StageF32<SH::BM, SH::BK, SH::NT, TA>;   // A is K-contiguous when transposed
    using SB = StageF32<SH::BN, SH::BK, SH::NT, !TB>;  // B is K-contiguous when not transposed
    static constexpr int NT = SH::NT, RM = SH::RM, RN = SH::RN, KW = k_waves<SH>();
    static constexpr int STAGE_FLOATS = SA::FLOATS + SB::FLOATS;
    static constexpr int RED_FLOATS = (KW - 1) * RM * RN * 16 * 64;
    static constexpr int LDS_BYTES =
        (2 * STAGE_FLOATS > RED_FLOATS ? 2 * STAGE_FLOATS : RED_FLOATS) * 4;
    static constexpr int STEPS = SH::BK / 2 / KW;  // K steps of a wave in a block
    static constexpr int G = 4 / (RM * RN) < 1 ? 1 : 4 / (RM * RN) > STEPS / 2 ? STEPS / 2 : 4 / (RM * RN);
    static constexpr int NG = STEPS / G;           // groups of G steps
    static_assert(SH::BK % (2 * KW) == 0 && NG * G == STEPS && NG % 2 == 0, "whole pairs of groups");
    static constexpr int CHUNKS = SA::S + SB::S;
    // Register sets of loads.  Two are faster where they cost few registers
    // (128x128x16 2048^3: 130 us against 140); 256x128x16 is 1-10% faster
    // with one, 128x128x32 up to 20%, and 256x256x32 spills with two.
    static constexpr int SETS = CHUNKS > 4 || RM * RN >= 8 ? 1 : 2;

    struct Frags {
        float a[G][RM], b[G][RN];
        // ks: K step within the block, of k = 2 ks (lanes 0-31) and 2 ks + 1
        __device__ __forceinline__ void read(const float *As, const float *Bs, int group, int half,
                                             int wk)
        {
#pragma unroll
            for (int s = 0; s < G; ++s) {
                const int kr = 2 * ((group * G + s) * KW + wk) + half;
#pragma unroll
                for (int i = 0; i < RM; ++i) a[s][i] = As[kr * SA::LD + i * 32];
#pragma unroll
                for (int j = 0; j < RN; ++j) b[s][j] = Bs[kr * SB::LD + j * 32];
            }
        }
        __device__ __forceinline__ void multiply(floatx16 (&acc)[RM][RN]) const
        {
#pragma unroll
            for (int s = 0; s < G; ++s)
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s][i], b[s][j],
                                                                          acc[i][j], 0, 0, 0);
        }
    };

    // The chunks of the next block are stored, and those of a later one
    // loaded, in the groups before the barrier.
    static constexpr int chunk_group(int c) { return c * (NG - 1) / CHUNKS; }
    static constexpr int chunks_in(int group)
    {
        int n = 0;
        for (int c = 0; c < CHUNKS; ++c) n += chunk_group(c) == group;
        return n;
    }

    template <bool SPLIT = false>
    __device__ __forceinline__ static void run(const GemmArgs &g, int64_t m0, int64_t n0,
                                               char *smem)
    {
        if (m0 + SH::BM <= g.m && n0 + SH::BN <= g.n) run_impl<INTERIOR, SPLIT>(g, m0, n0, smem);
        else if (g.m >= SA::MIN_ROWS && g.n >= SB::MIN_ROWS) run_impl<EDGE, SPLIT>(g, m0, n0, smem);
        else run_impl<MASKED, SPLIT>(g, m0, n0, smem);
    }

    template <LoadMode MODE, bool SPLIT>
    __device__ __forceinline__ static void run_impl(const GemmArgs &g, int64_t m0, int64_t n0,
                                                    char *smem)
    {
        float *lds = reinterpret_cast<float *>(smem);
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int wm = wave % SH::NWM, wn = wave / SH::NWM % SH::NWN;
        const int wk = KW > 1 ? wave / (SH::NWM * SH::NWN) : 0;
        const int half = lane >> 5, l32 = lane & 31;

        floatx16 acc[RM][RN];
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

        const KBlocks<SH::BK> kb(g.k);
        const int64_t blocks = kb.count;
        SA sa[SETS];  // block b + 1 is in set b % SETS
        SB sb[SETS];
        if (blocks > 0) load_first<MODE>(sa[0], sb[0], g, m0, n0, kb, lds, lds + SA::FLOATS, tid);
#pragma unroll
        for (int d = 0; d < SETS; ++d)
            if (blocks > 1 + d) {
                sa[d].template load<MODE>(g.A, g.lda, m0, kb.at(1 + d), g.m, g.k, tid);
                sb[d].template load<MODE>(g.B, g.ldb, n0, kb.at(1 + d), g.n, g.k, tid);
            }
        __syncthreads();
        const int ao = wm * SH::WM + l32, bo = SA::FLOATS + wn * SH::WN + l32;
        Frags f[2];
        if (blocks > 0) f[0].read(lds + ao, lds + bo, 0, half, wk);
        // Block b of the K loop, in LDS stage b & 1 (given as a constant).
        // whole: blocks b + 1 to b + 1 + SETS exist, so the step is
        // straight-line code.
        auto step = [&](auto whole, int64_t b, int stage) {
            constexpr bool WHOLE = decltype(whole)::value;
            const float *cur = lds + stage * STAGE_FLOATS;
            float *nxt = lds + (stage ^ 1) * STAGE_FLOATS;
            const int set = SETS == 2 ? stage : 0;
            const bool store = WHOLE || b + 1 < blocks, load = WHOLE || b + 1 + SETS < blocks;
            const int64_t k0 = kb.at(b + 1 + SETS);
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                if (q + 1 < NG) {
                    f[(q + 1) & 1].read(cur + ao, cur + bo, q + 1, half, wk);
                } else {
                    // every wave has stored its part of block b + 1 and has
                    // read the last of block b
                    __syncthreads();
                    if (store) f[0].read(nxt + ao, nxt + bo, 0, half, wk);
                }
                f[q & 1].multiply(acc);
#pragma unroll
                for (int c = 0; c < CHUNKS; ++c) {
                    if (chunk_group(c) != q) continue;
                    if (c < SA::S) {
                        if (store) sa[set].template store_chunk<MODE>(c, nxt, m0, g.m, tid);
                        if (load) sa[set].template load_chunk<MODE>(c, g.A, g.lda, m0, k0, g.m, g.k, tid);
                    } else {
                        if (store) sb[set].template store_chunk<MODE>(c - SA::S, nxt + SA::FLOATS, n0, g.n, tid);
                        if (load) sb[set].template load_chunk<MODE>(c - SA::S, g.B, g.ldb, n0, k0, g.n, g.k, tid);
                    }
                }
                constexpr int M = G * RM * RN;
                constexpr int READS = (G * (RM + RN) + M - 1) / M;
                const int writes = (chunks_in(q) * 4 + M - 1) / M, loads = (chunks_in(q) + M - 1) / M;
                deal_out<M, READS>(writes, loads);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int64_t b = 0;
        if (MODE != MASKED) {
            for (; b + 2 + SETS < blocks; b += 2) {
                step(std::true_type{}, b, 0);
                step(std::true_type{}, b + 1, 1);
            }
        }
        for (; b + 1 < blocks; b += 2) {
            step(std::false_type{}, b, 0);
            step(std::false_type{}, b + 1, 1);
        }
        if (b < blocks) step(std::false_type{}, b, 0);
        if constexpr (KW > 1) {
            wave_sum<KW, RM, RN>(acc, lds, wave, lane);
            if (wave != 0) return;
        }
        finish<SPLIT, RM, RN>(g, acc, m0 + wm * SH::WM, n0 + wn * SH::WN, tid, NT);
    }

    // sched_group_barrier takes constants only
    template <int M, int READS>
    __device__ __forceinline__ static void deal_out(int writes, int loads)
    {
#pragma unroll
        for (int q = 0; q < M; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // an MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);  // LDS reads
            if (writes == 1) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            else if (writes == 2) __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);
            else if (writes > 2) __builtin_amdgcn_sched_group_barrier(0x200, 4, 0);
            if (loads == 1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            else if (loads > 1) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);      // VALU
        }
    }
};

// The split-form tile.  Its bound is the issue of one wave: per block a thread
// splits 16 or 32 elements (some 90 or 180 VALU instructions) beside 12 or 48
// MFMAs of 32 cycles.  As in the FP32 tile the K loop is straight-line code
// with the splitting, the LDS accesses and the loads dealt out between the
// MFMAs; in lumps behind them, us before -> after: 2048^3 128x128x32 130 ->
// 111 (156 TFLOP/s), 1024x1024x4096 TN 64x64x32 115 -> 97.
template <class SH, bool TA, bool TB, bool ACC2>
struct X3Tile {
    using SA = StageX3<SH::BM, SH::BK, SH::NT, TA>;
    using SB = StageX3<SH::BN, SH::BK, SH::NT, !TB>;
    static_assert(SH::BK % 16 == 0, "bf16 MFMA consumes K in steps of 16");
    static constexpr int STAGE_HALVES = SA::HALVES + SB::HALVES;
    static constexpr int LDS_BYTES = 2 * STAGE_HALVES * 2;
    static constexpr int NT = SH::NT;

    static constexpr int NKS = SH::BK / 16;  // K steps of a block
    static_assert(NKS % 2 == 0, "a block starts with the fragments in f[0]");
    // register sets of loads: two where a set is small
    static constexpr int SETS = SA::S + SB::S > 2 ? 1 : 2;

    struct Frags {
        bf16x8 a[SH::RM][3], b[SH::RN][3];
        __device__ __forceinline__ void read(const __bf16 *As, const __bf16 *Bs, int ks)
        {
#pragma unroll
            for (int i = 0; i < SH::RM; ++i)
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    a[i][t] = *reinterpret_cast<const bf16x8 *>(As + t * SA::PART +
                                                                i * 32 * SA::LD + ks * 16);
#pragma unroll
            for (int j = 0; j < SH::RN; ++j)
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    b[j][t] = *reinterpret_cast<const bf16x8 *>(Bs + t * SB::PART +
                                                                j * 32 * SB::LD + ks * 16);
        }
        __device__ __forceinline__ void
        multiply(floatx16 (&acc)[SH::RM][SH::RN],
                 floatx16 (&lo)[ACC2 ? SH::RM : 1][ACC2 ? SH::RN : 1]) const
        {
#pragma unroll
            for (int i = 0; i < SH::RM; ++i)
#pragma unroll
                for (int j = 0; j < SH::RN; ++j) {
                    // smallest terms first; (0,0) is the leading product
                    floatx16 &small = ACC2 ? lo[ACC2 ? i : 0][ACC2 ? j : 0] : acc[i][j];
                    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][0], b[j][2], small, 0, 0, 0);
                    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][1], b[j][1], small, 0, 0, 0);
                    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][2], b[j][0], small, 0, 0, 0);
                    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][0], b[j][1], small, 0, 0, 0);
                    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][1], b[j][0], small, 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][0], b[j][0], acc[i][j], 0, 0, 0);
                }
        }
    };

    template <bool SPLIT = false>
    __device__ __forceinline__ static void run(const GemmArgs &g, int64_t m0, int64_t n0,
                                               char *smem)
    {
        if (m0 + SH::BM <= g.m && n0 + SH::BN <= g.n) run_impl<INTERIOR, SPLIT>(g, m0, n0, smem);
        else if (g.m >= SA::MIN_ROWS && g.n >= SB::MIN_ROWS) run_impl<EDGE, SPLIT>(g, m0, n0, smem);
        else run_impl<MASKED, SPLIT>(g, m0, n0, smem);
    }

    template <LoadMode MODE, bool SPLIT>
    __device__ __forceinline__ static void run_impl(const GemmArgs &g, int64_t m0, int64_t n0,
                                                    char *smem)
    {
        __bf16 *lds = reinterpret_cast<__bf16 *>(smem);
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int wm = wave % SH::NWM, wn = wave / SH::NWM;
        const int half = lane >> 5, l32 = lane & 31;

        floatx16 acc[SH::RM][SH::RN];
        floatx16 lo[ACC2 ? SH::RM : 1][ACC2 ? SH::RN : 1];
#pragma unroll
        for (int i = 0; i < SH::RM; ++i)
#pragma unroll
            for (int j = 0; j < SH::RN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
        if (ACC2) {
#pragma unroll
            for (int i = 0; i < (ACC2 ? SH::RM : 1); ++i)
#pragma unroll
                for (int j = 0; j < (ACC2 ? SH::RN : 1); ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) lo[i][j][e] = 0.0f;
        }

        const KBlocks<SH::BK> kb(g.k);
        const int64_t blocks = kb.count;
        SA sa[SETS];  // block b + 1 is in set b % SETS
        SB sb[SETS];
        if (blocks > 0) load_first<MODE>(sa[0], sb[0], g, m0, n0, kb, lds, lds + SA::HALVES, tid);
#pragma unroll
        for (int d = 0; d < SETS; ++d)
            if (blocks > 1 + d) {
                sa[d].template load<MODE>(g.A, g.lda, m0, kb.at(1 + d), g.m, g.k, tid);
                sb[d].template load<MODE>(g.B, g.ldb, n0, kb.at(1 + d), g.n, g.k, tid);
            }
        __syncthreads();
        const int ao = (wm * SH::WM + l32) * SA::LD + half * 8;
        const int bo = SA::HALVES + (wn * SH::WN + l32) * SB::LD + half * 8;
        Frags f[2];
        if (blocks > 0) f[0].read(lds + ao, lds + bo, 0);
        // Block b of the K loop, in LDS stage b & 1 (given as a constant).
        auto step = [&](auto whole, int64_t b, int stage) {
            constexpr bool WHOLE = decltype(whole)::value;
            const __bf16 *cur = lds + stage * STAGE_HALVES;
            __bf16 *nxt = lds + (stage ^ 1) * STAGE_HALVES;
            const int set = SETS == 2 ? stage : 0;
            const bool store = WHOLE || b + 1 < blocks, load = WHOLE || b + 1 + SETS < blocks;
#pragma unroll
            for (int q = 0; q < NKS; ++q) {
                if (q + 1 < NKS) {
                    f[(q + 1) & 1].read(cur + ao, cur + bo, q + 1);
                } else {
                    // every wave has stored its part of block b + 1 and has
                    // read the last of block b
                    __syncthreads();
                    if (store) f[0].read(nxt + ao, nxt + bo, 0);
                }
                f[q & 1].multiply(acc, lo);
                if (q == 0) {
                    if (store) {
                        sa[set].template store<MODE>(nxt, m0, g.m, tid);
                        sb[set].template store<MODE>(nxt + SA::HALVES, n0, g.n, tid);
                    }
                    if (load) {
                        const int64_t k0 = kb.at(b + 1 + SETS);
                        sa[set].template load<MODE>(g.A, g.lda, m0, k0, g.m, g.k, tid);
                        sb[set].template load<MODE>(g.B, g.ldb, n0, k0, g.n, g.k, tid);
                    }
                }
#pragma unroll
                for (int e = 0; e < 6 * SH::RM * SH::RN; ++e) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // an MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // an LDS read
                    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);  // VALU
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // an LDS write
                    __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);  // loads
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int64_t b = 0;
        if (MODE != MASKED) {
            for (; b + 2 + SETS < blocks; b += 2) {
                step(std::true_type{}, b, 0);
                step(std::true_type{}, b + 1, 1);
            }
        }
        for (; b + 1 < blocks; b += 2) {
            step(std::false_type{}, b, 0);
            step(std::false_type{}, b + 1, 1);
        }
        if (b < blocks) step(std::false_type{}, b, 0);
        if (ACC2) {
#pragma unroll
            for (int i = 0; i < SH::RM; ++i)
#pragma unroll
                for (int j = 0; j < SH::RN; ++j)
                    acc[i][j] += lo[ACC2 ? i : 0][ACC2 ? j : 0];
        }
        finish<SPLIT, SH::RM, SH::RN>(g, acc, m0 + wm * SH::WM, n0 + wn * SH::WN, tid, NT);
    }
};

// ---------------------------------------------------------------------------
// Software-pipelined split-precision tile.  While the matrix cores work on K
// block kt from LDS, the global loads of block kt+1 are in flight, and once a
// fraction Q0_NUM/Q0_DEN of the block's MFMA instructions are issued the
// split and LDS store of block kt+1 are interleaved between the remaining
// ones.  One workgroup barrier per K block.  HILO: the leading products in one
// accumulator and the five small ones in another: a third of the error.
// ---------------------------------------------------------------------------
template <class SH, bool TA, bool TB, int Q0_NUM = 1, int Q0_DEN = 3, bool FENCED = false,
          bool PF2 = false, bool HILO = false>
struct X3PTile {
    using SA = StageX3<SH::BM, SH::BK, SH::NT, TA>;
    using SB = StageX3<SH::BN, SH::BK, SH::NT, !TB>;
    static_assert(SH::BK == 16, "one bf16 MFMA K step per K block");
    static_assert(SA::UNITS_FULL && SB::UNITS_FULL, "every thread stages whole units");
    static constexpr int STAGE_HALVES = SA::HALVES + SB::HALVES;
    static constexpr int LDS_BYTES = 2 * STAGE_HALVES * 2;
    static constexpr int NT = SH::NT;
    static constexpr int RM = SH::RM, RN = SH::RN;
    static constexpr int NMFMA = RM * RN * 6;
    static constexpr int LM = HILO ? RM : 1, LN = HILO ? RN : 1;
    static constexpr int NELEM = SA::KS * (SA::UNITS + SB::UNITS);
    // first MFMA slot that carries split/store work for the next block
    static constexpr int Q0 = NMFMA * Q0_NUM / Q0_DEN;

    // Split element e (A units first, then B units) of the staged block into
    // the pending part vectors; after the last element of a unit, write the
    // unit's three parts to LDS.
    __device__ __forceinline__ static void split_elem(int e, const SA &sa, const SB &sb,
                                                      __bf16 *dst, int tid, bf16x8 &p0,
                                                      bf16x8 &p1, bf16x8 &p2)
    {
        constexpr int KS = SA::KS;
        const int u = e / KS, q = e % KS;
        __bf16 h0, h1, h2;
        if (u < SA::UNITS) split3(sa.unit_val(u, q), h0, h1, h2);
        else split3(sb.unit_val(u - SA::UNITS, q), h0, h1, h2);
        p0[q] = h0;
        p1[q] = h1;
        p2[q] = h2;
        if (q == KS - 1) {
            __bf16 *base;
            int part;
            if (u < SA::UNITS) { base = dst + SA::unit_offset(u, tid); part = SA::PART; }
            else { base = dst + SA::HALVES + SB::unit_offset(u - SA::UNITS, tid); part = SB::PART; }
            *reinterpret_cast<bf16x8 *>(base) = p0;
            *reinterpret_cast<bf16x8 *>(base + part) = p1;
            *reinterpret_cast<bf16x8 *>(base + 2 * part) = p2;
        }
    }

    template <bool STORE>
    __device__ __forceinline__ static void body(floatx16 (&acc)[RM][RN], floatx16 (&lo)[LM][LN],
                                                const __bf16 *cur,
                                                __bf16 *nxt, const SA &sa, const SB &sb,
                                                int tid, int wm, int wn, int half, int l32)
    {
        const __bf16 *As = cur + (wm * SH::WM + l32) * SA::LD + half * 8;
        const __bf16 *Bs = cur + SA::HALVES + (wn * SH::WN + l32) * SB::LD + half * 8;
        bf16x8 a[RM][3], b[2][3];
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int t = 0; t < 3; ++t)
                a[i][t] = *reinterpret_cast<const bf16x8 *>(As + t * SA::PART + i * 32 * SA::LD);
#pragma unroll
        for (int t = 0; t < 3; ++t)
            b[0][t] = *reinterpret_cast<const bf16x8 *>(Bs + t * SB::PART);
        if constexpr (FENCED) {
            // Explicit order: after slot Q0 every MFMA is followed by the
            // split of a few elements (and the unit's LDS write when its last
            // element is done); sched_barrier keeps the compiler from moving
            // anything across.
            bf16x8 p0, p1, p2;
            int q = 0;
#pragma unroll
            for (int j = 0; j < RN; ++j) {
#pragma unroll
                for (int pr = 0; pr < 6; ++pr) {
#pragma unroll
                    for (int i = 0; i < RM; ++i) {
                        const int sa_i = pr == 0 ? 0 : pr == 1 ? 1 : pr == 2 ? 2 : pr == 3 ? 0 : pr == 4 ? 1 : 0;
                        const int sb_j = pr == 0 ? 2 : pr == 1 ? 1 : pr == 2 ? 0 : pr == 3 ? 1 : pr == 4 ? 0 : 0;
                        floatx16 &c = HILO && pr < 5 ? lo[HILO ? i : 0][HILO ? j : 0] : acc[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][sa_i], b[j & 1][sb_j], c,
                                                                    0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (i == 0 && pr == 0 && j + 1 < RN) {
#pragma unroll
                            for (int t = 0; t < 3; ++t)
                                b[(j + 1) & 1][t] = *reinterpret_cast<const bf16x8 *>(
                                    Bs + t * SB::PART + (j + 1) * 32 * SB::LD);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (STORE && q >= Q0) {
                            const int e0 = (q - Q0) * NELEM / (NMFMA - Q0);
                            const int e1 = (q + 1 - Q0) * NELEM / (NMFMA - Q0);
#pragma unroll
                            for (int e = e0; e < e1; ++e) split_elem(e, sa, sb, nxt, tid, p0, p1, p2);
                            if (e1 > e0) __builtin_amdgcn_sched_barrier(0);
                        }
                        ++q;
                    }
                }
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            // products, smallest first: (0,2) (1,1) (2,0) (0,1) (1,0) (0,0);
            // consecutive MFMAs go to different accumulators (i varies fastest)
#pragma unroll
            for (int pr = 0; pr < 6; ++pr) {
#pragma unroll
                for (int i = 0; i < RM; ++i) {
                    const int sa_i = pr == 0 ? 0 : pr == 1 ? 1 : pr == 2 ? 2 : pr == 3 ? 0 : pr == 4 ? 1 : 0;
                    const int sb_j = pr == 0 ? 2 : pr == 1 ? 1 : pr == 2 ? 0 : pr == 3 ? 1 : pr == 4 ? 0 : 0;
                    floatx16 &c = HILO && pr < 5 ? lo[HILO ? i : 0][HILO ? j : 0] : acc[i][j];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][sa_i], b[j & 1][sb_j], c, 0, 0, 0);
                    if (i == 0 && pr == 0 && j + 1 < RN) {
#pragma unroll
                        for (int t = 0; t < 3; ++t)
                            b[(j + 1) & 1][t] = *reinterpret_cast<const bf16x8 *>(
                                Bs + t * SB::PART + (j + 1) * 32 * SB::LD);
                    }
                }
            }
        }
        if (STORE) {
#pragma unroll
            for (int u = 0; u < SA::UNITS; ++u) sa.store_unit(nxt, u, tid);
#pragma unroll
            for (int u = 0; u < SB::UNITS; ++u) sb.store_unit(nxt + SA::HALVES, u, tid);
        }
        // Issue order: the fragment reads first, then one MFMA at a time;
        // from MFMA slot Q0 on, each slot also carries a share of the split
        // (independent VALU work from several elements, so the in-order issue
        // does not wait on one element's dependency chain) and, every few
        // slots, one 16-byte LDS write.  B fragments of the next column are
        // read right after the first MFMA of the current column.
        constexpr int NWRITE = 3 * (SA::UNITS + SB::UNITS);
        constexpr int NVALU = 8 * NELEM;  // split work plus address arithmetic
        constexpr int SLOTS = NMFMA - Q0;
        constexpr int VPER = (NVALU + SLOTS - 1) / SLOTS;
        __builtin_amdgcn_sched_group_barrier(0x100, 3 * RM + 3, 0);
#pragma unroll
        for (int qq = 0; qq < NMFMA; ++qq) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (qq % (6 * RM) == 0 && qq / (6 * RM) + 1 < RN)
                __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
            if (STORE && qq >= Q0) {
                __builtin_amdgcn_sched_group_barrier(0x002, VPER, 0);
                if ((qq - Q0) * NWRITE / SLOTS != (qq + 1 - Q0) * NWRITE / SLOTS)
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            }
        }
    }

    template <bool SPLIT = false>
    __device__ __forceinline__ static void run(const GemmArgs &g, int64_t m0, int64_t n0,
                                               char *smem)
    {
        if (m0 + SH::BM <= g.m && n0 + SH::BN <= g.n) run_impl<INTERIOR, SPLIT>(g, m0, n0, smem);
        else if (g.m >= SA::MIN_ROWS && g.n >= SB::MIN_ROWS) run_impl<EDGE, SPLIT>(g, m0, n0, smem);
        else run_impl<MASKED, SPLIT>(g, m0, n0, smem);
    }

    template <LoadMode MODE, bool SPLIT>
    __device__ __forceinline__ static void run_impl(const GemmArgs &g, int64_t m0, int64_t n0,
                                                    char *smem)
    {
        __bf16 *lds = reinterpret_cast<__bf16 *>(smem);
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int wm = wave % SH::NWM, wn = wave / SH::NWM;
        const int half = lane >> 5, l32 = lane & 31;

        floatx16 acc[RM][RN], lo[LM][LN];
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = lo[HILO ? i : 0][HILO ? j : 0][e] = 0.0f;
        const auto join = [&] {
            if constexpr (HILO) {
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RN; ++j) acc[i][j] += lo[i][j];
            }
        };

        const KBlocks<SH::BK> kb(g.k);
        const int64_t ktiles = kb.count;
        if constexpr (PF2) {
            // Two register sets: the global loads of block kt+2 go to the
            // second set at the top of block kt, while the first set (block
            // kt+1, loaded a whole block earlier) is split and stored between
            // the MFMAs; at the end of the block the second set moves into
            // the first.  A load thus has a block and a third of MFMA time to
            // arrive instead of a third, and the one body keeps the
            // accumulators in place.
            SA sa, sa2;
            SB sb, sb2;
            if (ktiles > 0) {
                load_first<MODE>(sa, sb, g, m0, n0, kb, lds, lds + SA::HALVES, tid);
            }
            if (ktiles > 1) {
                sa.template load<MODE>(g.A, g.lda, m0, kb.at(1), g.m, g.k, tid);
                sb.template load<MODE>(g.B, g.ldb, n0, kb.at(1), g.n, g.k, tid);
            }
            __syncthreads();
            for (int64_t kt = 0; kt < ktiles; ++kt) {
                const __bf16 *cur = lds + (kt & 1) * STAGE_HALVES;
                __bf16 *nxt = lds + ((kt + 1) & 1) * STAGE_HALVES;
                if (kt + 2 < ktiles) {
                    const int64_t k0 = kb.at(kt + 2);
                    sa2.template load<MODE>(g.A, g.lda, m0, k0, g.m, g.k, tid);
                    sb2.template load<MODE>(g.B, g.ldb, n0, k0, g.n, g.k, tid);
                }
                // a store whose block does not exist rewrites an idle stage
                // that nothing reads again
                body<true>(acc, lo, cur, nxt, sa, sb, tid, wm, wn, half, l32);
                if (kt + 2 < ktiles) {
                    sa = sa2;
                    sb = sb2;
                }
                __syncthreads();
            }
            join();
            finish<SPLIT, RM, RN>(g, acc, m0 + wm * SH::WM, n0 + wn * SH::WN, tid, NT);
            return;
        }
        SA sa;
        SB sb;
        if (ktiles > 0) {
            load_first<MODE>(sa, sb, g, m0, n0, kb, lds, lds + SA::HALVES, tid);
        }
        __syncthreads();
        for (int64_t kt = 0; kt < ktiles; ++kt) {
            const __bf16 *cur = lds + (kt & 1) * STAGE_HALVES;
            __bf16 *nxt = lds + ((kt + 1) & 1) * STAGE_HALVES;
            if (kt + 1 < ktiles) {
                const int64_t k0 = kb.at(kt + 1);
                sa.template load<MODE>(g.A, g.lda, m0, k0, g.m, g.k, tid);
                sb.template load<MODE>(g.B, g.ldb, n0, k0, g.n, g.k, tid);
            }
            // On the last block the store rewrites the idle buffer with the
            // block already consumed; nothing reads it afterwards.  One body
            // for every iteration keeps the accumulators in place.
            body<true>(acc, lo, cur, nxt, sa, sb, tid, wm, wn, half, l32);
            __syncthreads();
        }
        join();
        finish<SPLIT, RM, RN>(g, acc, m0 + wm * SH::WM, n0 + wn * SH::WN, tid, NT);
    }
};

// The split form of the small tile: each K block holds KW steps of 16 k,
// one per wave, split while staged; a wave adds its leading part products into
// one accumulator and the five small ones, smallest first, into another.
template <class SH, bool TA, bool TB>
struct X3WTile {
    using SA = StageX3<SH::BM, SH::BK, SH::NT, TA>;
    using SB = StageX3<SH::BN, SH::BK, SH::NT, !TB>;
    static constexpr int KW = SH::KW, RM = SH::RM, RN = SH::RN, NT = SH::NT;
    static constexpr int STEPS = SH::BK / 16;  // 16 k per v_mfma_f32_32x32x16_bf16
    static_assert(STEPS % KW == 0, "every wave takes the same number of k steps");
    static constexpr int STAGE_HALVES = SA::HALVES + SB::HALVES;
    static constexpr int RED_FLOATS = (KW - 1) * RM * RN * 16 * 64;
    static constexpr int LDS_BYTES =
        (2 * STAGE_HALVES * 2 > RED_FLOATS * 4 ? 2 * STAGE_HALVES * 2 : RED_FLOATS * 4);

    template <bool SPLIT = false>
    __device__ __forceinline__ static void run(const GemmArgs &g, int64_t m0, int64_t n0,
                                               char *smem)
    {
        static_assert(!SPLIT, "no split-K variant");
        if (m0 + SH::BM <= g.m && n0 + SH::BN <= g.n) run_impl<INTERIOR>(g, m0, n0, smem);
        else if (g.m >= SA::MIN_ROWS && g.n >= SB::MIN_ROWS) run_impl<EDGE>(g, m0, n0, smem);
        else run_impl<MASKED>(g, m0, n0, smem);
    }

    template <LoadMode MODE>
    __device__ __forceinline__ static void run_impl(const GemmArgs &g, int64_t m0, int64_t n0,
                                                    char *smem)
    {
        __bf16 *lds = reinterpret_cast<__bf16 *>(smem);
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int half = lane >> 5, l32 = lane & 31;
        floatx16 acc[RM][RN], lo[RM][RN];
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = lo[i][j][e] = 0.0f;
        const KBlocks<SH::BK> kb(g.k);
        const int64_t ktiles = kb.count;
        SA sa;
        SB sb;
        if (ktiles > 0) {
            load_first<MODE>(sa, sb, g, m0, n0, kb, lds, lds + SA::HALVES, tid);
        }
        __syncthreads();
        for (int64_t kt = 0; kt < ktiles; ++kt) {
            __bf16 *cur = lds + (kt & 1) * STAGE_HALVES;
            __bf16 *nxt = lds + ((kt + 1) & 1) * STAGE_HALVES;
            const bool more = kt + 1 < ktiles;
            if (more) {
                const int64_t k0 = kb.at(kt + 1);
                sa.template load<MODE>(g.A, g.lda, m0, k0, g.m, g.k, tid);
                sb.template load<MODE>(g.B, g.ldb, n0, k0, g.n, g.k, tid);
            }
            const __bf16 *As = cur + l32 * SA::LD + half * 8;
            const __bf16 *Bs = cur + SA::HALVES + l32 * SB::LD + half * 8;
#pragma unroll
            for (int s = 0; s < STEPS / KW; ++s) {
                const int ks = s * KW + wave;
                bf16x8 a[RM][3], b[RN][3];
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int t = 0; t < 3; ++t)
                        a[i][t] = *reinterpret_cast<const bf16x8 *>(
                            As + t * SA::PART + i * 32 * SA::LD + ks * 16);
#pragma unroll
                for (int j = 0; j < RN; ++j)
#pragma unroll
                    for (int t = 0; t < 3; ++t)
                        b[j][t] = *reinterpret_cast<const bf16x8 *>(
                            Bs + t * SB::PART + j * 32 * SB::LD + ks * 16);
#pragma unroll
                for (int i = 0; i < RM; ++i)
#pragma unroll
                    for (int j = 0; j < RN; ++j) {
                        floatx16 &c = lo[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][0], b[j][2], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][1], b[j][1], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][2], b[j][0], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][0], b[j][1], c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][1], b[j][0], c, 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][0], b[j][0],
                                                                            acc[i][j], 0, 0, 0);
                    }
            }
            if (more) {
                sa.template store<MODE>(nxt, m0, g.m, tid);
                sb.template store<MODE>(nxt + SA::HALVES, n0, g.n, tid);
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j) acc[i][j] += lo[i][j];
        wave_sum<KW, RM, RN>(acc, reinterpret_cast<float *>(smem), wave, lane);
        if (wave == 0) epilogue<RM, RN>(g, acc, m0, n0, lane);
    }
};

// ---------------------------------------------------------------------------
// Tile order: blocks are dispatched round-robin over the 8 XCDs (block b goes
// to XCD b % 8).  Renumber so that each XCD receives a contiguous range of
// tile ids, then walk tiles in groups of GROUP_M tile-rows so that the tiles
// resident on one XCD share A row-panels and B column-panels in its L2.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nb)
{
    const int64_t q = nb / 8, r = nb % 8;
    const int64_t x = bid % 8, idx = bid / 8;
    const int64_t base = x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q;
    return base + idx;
}

__device__ __forceinline__ void tile_coords(int64_t t, int64_t tiles_m, int64_t tiles_n,
                                            int group_m, int64_t &tm, int64_t &tn)
{
    const int64_t per_group = (int64_t)group_m * tiles_n;
    const int64_t grp = t / per_group;
    const int64_t first_m = grp * group_m;
    const int64_t gsize = tiles_m - first_m < group_m ? tiles_m - first_m : group_m;
    const int64_t in_grp = t - grp * per_group;
    tm = first_m + in_grp % gsize;
    tn = in_grp / gsize;
}

}  // namespace misgemm
