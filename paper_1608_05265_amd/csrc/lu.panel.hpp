// The panel factorization of the LU: up to 64 columns in one launch.
//
// What bounds it is latency: every column needs its pivot, the largest of
// all its entries, before the next column can be updated, so a panel is a
// chain of reductions.  A launch per 8 columns by one workgroup (the form
// before this one) cost 13 us per launch at 4608 rows and, between the
// launches, the interchanges, triangular solves and small products that
// stitch 8-column panels together: 17.1 ms for the 4608 factorization, 3.7 us
// a column.  Here the rows are spread over G workgroups, each row held in
// the registers of one thread for the whole panel, and the workgroups
// exchange one message per column (the pivot search's candidate and its row)
// through memory, so that 64 columns need no other launch.
//
// The exchange.  A message is a set of 8-byte words, each a 32-bit payload
// under a 32-bit tag that names the column (never 0, never the same twice in
// a factorization), written and read with relaxed device-scope atomics: a
// word either carries the tag, and then its payload is whole, or it does
// not, and the reader looks again.  No fence (a device-scope release writes
// back the XCD's whole L2), no counter, no clearing between columns.  Two
// message slots per workgroup alternate: a workgroup writes column q+2's
// message only after it has read everybody's message of column q+1, which
// everybody writes after having read column q's.  The words live in the tail
// of the caller's ipiv array, whose entries are written by later panels
// only, and which the factorization clears first (tag 0): the library keeps
// no buffer that calls on several streams, or graphs, could share.
// Measured per exchange (a kernel that only exchanges, one polling wavefront
// per workgroup): 1.1 us for 5 workgroups of one XCD, 1.6 us over all XCDs, so
// the workgroups are taken from one XCD (blocks go to the 8 XCDs in turn)
// while the rows fit half of its CUs.
//
// Waiting.  Every workgroup waits for messages of the others, so all G must
// be resident at once.  The first column decides it, once for the launch, in
// the start word: the first workgroup waits a bounded time for everybody's
// first message and swaps in "go" or "stop"; the others wait a bounded, longer
// time for its word and swap in "stop" when it does not come.  The first swap
// stands and everybody obeys it, so no workgroup leaves a launch that goes
// on, in whatever order the workgroups were dispatched (the XCDs dispatch
// independently, and another stream's kernel can hold back the first
// workgroup alone).  After "go" every workgroup is resident and has posted,
// and each wait ends.  After "stop" (other streams' kernels hold the CUs for
// long, or several factorizations hold each other's up) the first workgroup
// factors the panel alone, in memory, and the others end.
#pragma once

#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

namespace {

constexpr int PANEL = 64;             // columns of a panel
constexpr int PANEL_THREADS = 512;
constexpr int PANEL_WAVES = PANEL_THREADS / 64;
constexpr int PANEL_GROUPS = 64;      // most workgroups (one lane polls each)
constexpr int PANEL_XCD_GROUPS = 16;  // most workgroups placed on one XCD (half its CUs)
constexpr int NEAR = 12;              // up to so many, one round trip fetches all messages
// Words of a message: the row, then its candidate; whole 128-byte lines, and
// the messages start on one.
constexpr int MSG = PANEL + 16;
constexpr int MSG_MAG = PANEL, MSG_POS = PANEL + 1, MSG_START = PANEL + 3;
constexpr int64_t MSG_WORDS = 2 * MSG;  // words per workgroup (two slots)
constexpr int64_t MSG_ALIGN = 16;       // words
// Polls (about 0.4 us each) that the first workgroup waits for the others and
// the others for its word; and a bound that no wait after "go" reaches, so
// that the kernel ends even when the words are overwritten under it.
constexpr int PANEL_WAIT = 1 << 16;
constexpr int PANEL_WORD_WAIT = 1 << 18;
constexpr int PANEL_HARD_WAIT = 1 << 22;

// v from another lane of the same 16-lane row (DPP control CTRL).
template <int CTRL>
__device__ inline uint32_t dpp32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

__device__ inline uint32_t readlane32(uint32_t v, int lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// x of lane q (wavefront-uniform) in every lane, through a scalar register.
__device__ inline float lane_value(float x, int q)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), q));
}

// Maximum over the first N lanes (N = 8, 16 or 64; all lanes active),
// uniform: exchanges with the neighbour (quad_perm 1,0,3,2), the other pair
// (quad_perm 2,3,0,1), the mirrored quad in the half row and the mirrored
// half row, then the four 16-lane rows through scalar readlanes.
template <int N>
__device__ inline uint32_t lanes_max(uint32_t v)
{
    const auto up = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = up(v, dpp32<0xB1>(v));
    v = up(v, dpp32<0x4E>(v));
    v = up(v, dpp32<0x141>(v));
    if (N > 8) v = up(v, dpp32<0x140>(v));
    const uint32_t r = readlane32(v, 0);
    if (N <= 16) return r;
    return (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)up(up(r, readlane32(v, 16)), up(readlane32(v, 32), readlane32(v, 48))));
}

// A pivot candidate: mag = the magnitude's bits + 2 (bit patterns of
// non-negative floats order as the values do) and the row's position.  The
// best one has the largest magnitude and, among equals, the smallest position
// -- the first row of largest magnitude, as a sequential scan finds it.  NaN
// is never a candidate; where all of a column is NaN its own row stands in
// with mag 1.  mag 0: no row.
constexpr uint32_t MAG_NONE = 1, MAG_ZERO = 2;
struct Candidate {
    uint32_t mag, pos;
};

// The best candidate of the first N lanes (uniform) and a lane that holds it.
// Positions are distinct, and rarely does more than one lane hold the largest
// magnitude.
template <int N>
__device__ inline Candidate lanes_best(Candidate c, int &owner)
{
    Candidate b;
    b.mag = lanes_max<N>(c.mag);
    uint64_t top = __ballot(c.mag == b.mag);
    if (N < 64) top &= (1ull << (N & 63)) - 1;
    if (__builtin_expect((top & (top - 1)) != 0, 0)) {
        const bool in = (top >> (threadIdx.x & 63)) & 1;
        const uint32_t first = ~lanes_max<N>(in ? ~c.pos : 0u);
        top = __ballot(in && c.pos == first);
    }
    owner = (int)__builtin_ctzll(top);  // never empty: some lane holds the maximum
    b.pos = readlane32(c.pos, owner);
    return b;
}

// The multipliers of a pivot column: the entries below the pivot times the
// pivot's reciprocal when the pivot is at least the smallest normal number
// (so that the reciprocal is finite), as LAPACK's sgetf2 and HPL scale the
// column, else divided by the pivot.
__device__ inline bool scale_by_reciprocal(float piv) { return fabsf(piv) >= FLT_MIN; }

__device__ inline void put_word(uint64_t *p, uint32_t tag, uint32_t payload)
{
    __hip_atomic_store(p, ((uint64_t)tag << 32) | payload, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint64_t get_word(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool tagged(uint64_t word, uint32_t tag) { return (uint32_t)(word >> 32) == tag; }

enum PanelState { PANEL_GO = 1, PANEL_STOP = 2, PANEL_LOST = 3 };

// The launch's one decision: `vote` if nobody decided before, else what
// stands in the word, which was `seen` a while ago.  (A swap fails only where
// the word changed, which it does once in a launch.)
__device__ inline int decide(uint64_t *word, uint64_t seen, uint32_t tag, int vote)
{
    while (!tagged(seen, tag))
        if (__hip_atomic_compare_exchange_strong(word, &seen, ((uint64_t)tag << 32) | (uint32_t)vote,
                                                 __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return vote;
    return (int)(uint32_t)seen;
}

// The panel in memory by one workgroup of NT threads, every column pass
// walking it: panels taller than PANEL_GROUPS workgroups hold, and those
// whose workgroups did not come together.  w <= PANEL.  The same operations in
// the same order as lu_panel_kernel's (columns in blocks of eight, a block's
// products summed apart), so that the factors do not depend on which of the
// two a panel took.
template <int NT>
__device__ void panel_in_memory(float *__restrict__ P, int64_t lda, int64_t m, int w,
                                int64_t *__restrict__ ipiv, int64_t row0, int *__restrict__ info)
{
    __shared__ float sbest[NT];
    __shared__ int64_t sidx[NT];
    __shared__ float su[8][PANEL];  // the block's pivot rows in the columns after it
    const int t = threadIdx.x;
    for (int b = 0; b < w; b += 8) {
        const int e = b + 8 < w ? b + 8 : w;
        uint32_t taken = 0;  // bit k: column b + k has multipliers
        for (int j = b; j < e; ++j) {
            float *col = P + (int64_t)j * lda;
            float best = -1.0f;
            int64_t idx = -1;
            for (int64_t r = j + t; r < m; r += NT) {
                const float v = fabsf(col[r]);
                if (v > best) { best = v; idx = r; }
            }
            sbest[t] = best;
            sidx[t] = idx;
            __syncthreads();
            for (int s = NT / 2; s > 0; s >>= 1) {
                if (t < s) {
                    const float b1 = sbest[t + s];
                    const int64_t i1 = sidx[t + s];
                    if (i1 >= 0 && (sidx[t] < 0 || b1 > sbest[t] || (b1 == sbest[t] && i1 < sidx[t]))) {
                        sbest[t] = b1;
                        sidx[t] = i1;
                    }
                }
                __syncthreads();
            }
            const int64_t p = sidx[0] >= 0 ? sidx[0] : j;
            const float pivot_mag = sbest[0];
            __syncthreads();
            if (t == 0) ipiv[row0 + j] = row0 + p;
            if (p != j && t < w) {
                float *c = P + (int64_t)t * lda;
                const float x = c[j];
                c[j] = c[p];
                c[p] = x;
            }
            __syncthreads();
            const float piv = col[j];
            if (pivot_mag > 0.0f && piv != 0.0f) {
                if (scale_by_reciprocal(piv)) {
                    const float rinv = 1.0f / piv;
                    for (int64_t r = j + 1 + t; r < m; r += NT) col[r] = col[r] * rinv;
                } else {
                    for (int64_t r = j + 1 + t; r < m; r += NT) col[r] = col[r] / piv;
                }
                taken |= 1u << (j - b);
                if (t > j && t < e) su[0][t] = P[j + (int64_t)t * lda];
                __syncthreads();
                for (int64_t r = j + 1 + t; r < m; r += NT) {
                    const float l = col[r];
                    for (int c = j + 1; c < e; ++c) {
                        float *x = P + r + (int64_t)c * lda;
                        *x = fmaf(-l, su[0][c], *x);
                    }
                }
            } else if (t == 0 && *info == 0) {
                *info = (int)(row0 + j + 1);
            }
            __syncthreads();
        }
        if (e == w) break;
        // the pivot rows in the later columns, a column per thread
        if (t < w - e) {
            float *c = P + b + (int64_t)(e + t) * lda;
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float s = 0.0f;
#pragma unroll
                for (int k = 0; k < i; ++k)
                    if ((taken >> k) & 1) s = fmaf(-P[b + i + (int64_t)(b + k) * lda], x[k], s);
                x[i] = c[i] + s;
                c[i] = x[i];
                su[i][t] = (taken >> i) & 1 ? x[i] : 0.0f;
            }
        }
        __syncthreads();
        for (int64_t r = e + t; r < m; r += NT) {
            float nl[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                nl[k] = (taken >> k) & 1 ? -P[r + (int64_t)(b + k) * lda] : -0.0f;
            for (int c = e; c < w; ++c) {
                float s = 0.0f;
#pragma unroll
                for (int k = 0; k < 8; ++k) s = fmaf(su[k][c - e], nl[k], s);
                P[r + (int64_t)c * lda] += s;
            }
        }
        __syncthreads();
    }
}

typedef float panel_f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float panel_f4 __attribute__((ext_vector_type(4)));

// v[G] += sum over k of u[k][4G .. 4G+3] nl[k] on every lane's own row, for
// G = G0, G0 + 1 (u[k]: one element per lane): v_mfma_f32_4x4x1, whose 16
// blocks of 4 rows x 4 columns all take block G of u (broadcast controls 4,
// G), so that lane l's result is its row's four columns, each one fused
// multiply-add, bit for bit fmaf.  Four columns in 8 cycles and no broadcast
// of u through scalar registers: with readlanes and vector FMAs the updates
// took over half of the time.  The eight products are summed apart and added
// once: an entry of the last columns is rounded 7 times by block sums, not 56
// times at its own magnitude.
template <int G0>
__device__ __forceinline__ void rank8(panel_f4 (&v)[PANEL / 4], const float (&u)[8],
                                      const float (&nl)[8])
{
    panel_f4 s0 = {0.0f, 0.0f, 0.0f, 0.0f}, s1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        s0 = __builtin_amdgcn_mfma_f32_4x4x1f32(u[k], nl[k], s0, 4, G0, 0);
        s1 = __builtin_amdgcn_mfma_f32_4x4x1f32(u[k], nl[k], s1, 4, G0 + 1, 0);
    }
    v[G0] += s0;
    v[G0 + 1] += s1;
}

// Factor the m x w panel P (w <= PANEL, leading dimension lda; its top-left
// element is A(row0, row0)) with the workgroups g = 0 .. G-1 of the launch:
// block `first + stride g` is workgroup g, other blocks end at once.  Thread
// t of workgroup g holds rows RPT (PANEL_THREADS g + t) .. + RPT - 1 of the
// panel, all columns.
//
// Rows do not move: each row has a position (its index in the panel after
// the interchanges so far), an interchange renames two positions, and a row
// is done once it is a pivot.  Its part of U, which every workgroup learns,
// is stored at once by the first one (all rows were loaded before the first
// message, so nothing is overwritten early), and whatever the later updates
// make of it in its owner's registers is ignored: no update needs a mask.  At
// the end every row's other entries are stored at its position.
//
// Columns are taken in blocks of eight; register column c holds panel column
// 8b + c during block b and the registers are rotated by eight after it, so
// that one body serves every block (eight columns unrolled; all 64 would
// overflow the instruction cache).  Within a block a pivot row is subtracted
// from the block's own columns only; the other columns take the block's eight
// together at its end, on matrix cores.
//
// Order of a column: with the pivot row u of column j known, every thread
// takes its multiplier, updates its entries of the block's later columns and
// looks for the best candidate in column j+1; the wavefronts' candidates meet
// in LDS, and the wavefront that holds the workgroup's posts its row.  (One
// wavefront only: a row leaves its thread through LDS, where a 16-byte write
// takes its 8 cycles however few lanes are active.)  Another wavefront (the
// poster would wait for its own stores first) reads all candidates, takes the
// winner's row and, in the columns after the block, applies the block's
// earlier pivot rows to it with the row's own multipliers, summed in order
// and added once: the next pivot row.
template <int RPT>
__global__ __launch_bounds__(PANEL_THREADS) void lu_panel_kernel(
    float *__restrict__ P, int64_t lda, int m, int w, int64_t *__restrict__ ipiv, int64_t row0,
    int *__restrict__ info, uint64_t *__restrict__ words, int G, int first, int stride,
    int wait_polls, int word_polls)
{
    static_assert(RPT == 1 || RPT == 2, "rows per thread");
    if ((int)blockIdx.x % stride != first) return;
    const int g = (int)blockIdx.x / stride;
    __shared__ __attribute__((aligned(16))) float srow[PANEL];  // the workgroup's candidate row
    __shared__ uint2 skey[PANEL_WAVES];  // the wavefronts' candidates
    __shared__ float su[PANEL];          // the pivot row
    __shared__ uint2 swin;               // its candidate; mag 0: see sstate
    __shared__ int sstate;               // a PanelState
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);  // scalar branches on it
    const int r0 = RPT * (PANEL_THREADS * g + t);
    if (t == 0) sstate = PANEL_GO;

    panel_f4 v[RPT][PANEL / 4];
    int pos[RPT];
    bool act[RPT];  // a row of the panel that is no pivot yet
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        pos[i] = r0 + i;
        act[i] = r0 + i < m;
    }
#pragma unroll
    for (int c = 0; c < PANEL; ++c) {
        const float *pc = P + (int64_t)c * lda;
        if (RPT == 2 && c < w && r0 + 2 <= m) {
            const panel_f2u x = *reinterpret_cast<const panel_f2u *>(pc + r0);
            v[0][c / 4][c % 4] = x[0];
            v[RPT - 1][c / 4][c % 4] = x[1];
        } else {
#pragma unroll
            for (int i = 0; i < RPT; ++i)
                v[i][c / 4][c % 4] = c < w && r0 + i < m ? pc[r0 + i] : 0.0f;
        }
    }

    float ub[8];  // the block's pivot rows, lane c: register column c
    uint32_t taken = 0;  // bit k: the block's column k has multipliers

    // Post the best candidate of panel column q, which is register column
    // `col`, and learn the winner: swin and su (the pivot row).  aside(ow),
    // ow the posting wavefront, runs between the posting and the reading.
    const auto exchange = [&](int q, int col, auto &&aside) __attribute__((always_inline)) {
        Candidate c{0, 0xFFFFFFFFu};
        int ci = 0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const float a = fabsf(v[i][col / 4][col % 4]);
            uint32_t u = a >= 0.0f ? __float_as_uint(a) + MAG_ZERO : pos[i] == q ? MAG_NONE : 0u;
            u = act[i] ? u : 0u;
            if (u > c.mag || (u == c.mag && (uint32_t)pos[i] < c.pos)) {
                c.mag = u;
                c.pos = (uint32_t)pos[i];
                ci = i;
            }
        }
        int owner;
        const Candidate wb = lanes_best<64>(c, owner);
        if (lane == 0) skey[wave] = make_uint2(wb.mag, wb.pos);
        __syncthreads();
        const uint2 key = skey[lane & (PANEL_WAVES - 1)];
        int ow;
        Candidate gb = lanes_best<PANEL_WAVES>(Candidate{key.x, key.y}, ow);
        const uint32_t tag = (uint32_t)(row0 + q + 1);
        float rowv = 0.0f;
        // the pivot row from a candidate row: in the columns after the block,
        // the block's earlier pivot rows with the row's own multipliers (the
        // entries of a column without a pivot, NaN perhaps, are none)
        const auto pivot_row = [&](float r) __attribute__((always_inline)) {
            const float l = __builtin_amdgcn_inverse_ballot_w64(taken | ~0xFFull) ? r : 0.0f;
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k < col; ++k) s = fmaf(-lane_value(l, k), ub[k], s);
            return lane < 8 ? r : r + s;
        };
        if (wave == ow) {
            if (gb.mag != 0) {
                const int oi = __builtin_amdgcn_readlane(ci, owner);
                if (lane == owner) {
#pragma unroll
                    for (int i = 0; i < RPT; ++i)
                        if (RPT == 1 || i == oi) {
#pragma unroll
                            for (int k = 0; k < PANEL / 4; ++k)
                                reinterpret_cast<panel_f4 *>(srow)[k] = v[i][k];
                            // keeps the two rows' stores apart (merged, the
                            // compiler selects all 64 values with moves first)
                            asm volatile("; row %0" ::"i"(i) : "memory");
                        }
                }
                // LDS serves a wavefront's accesses in order
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                rowv = srow[lane];
            }
            if (G > 1) {
                uint64_t *msg = words + ((int64_t)(q & 1) * G + g) * MSG;
                put_word(msg + lane, tag, __float_as_uint(rowv));
                if (lane < 2) put_word(msg + PANEL + lane, tag, lane == 0 ? gb.mag : gb.pos);
            } else {
                su[lane] = pivot_row(rowv);
                if (lane == 0) swin = make_uint2(gb.mag, gb.pos);
            }
        }
        aside(ow);
        if (G > 1 && wave == ((ow + 1) & (PANEL_WAVES - 1))) {
            const uint64_t *slot = words + (int64_t)(q & 1) * G * MSG;
            const uint64_t *mine = slot + (int64_t)(lane < G ? lane : 0) * MSG;
            Candidate x{0, 0xFFFFFFFFu};
            int st = PANEL_GO, bound = PANEL_HARD_WAIT;
            uint64_t start = 0;
            if (q == 0) {
                start = get_word(words + MSG_START);
                if (g == 0) {
                    bound = wait_polls;
                    if (bound < 0) st = PANEL_STOP;
                } else {  // the first workgroup's word
#pragma unroll 1
                    for (int polls = 0; !tagged(start, tag) && polls < word_polls; ++polls)
                        start = get_word(words + MSG_START);
                    if (lane == 0) st = decide(words + MSG_START, start, tag, PANEL_STOP);
                    st = __builtin_amdgcn_readfirstlane(st);
                }
            }
            int win;
            if (G <= NEAR) {
                // few workgroups: all their messages in one round trip (a column
                // 0.17 us less than keys first, then the winner's row, at 5
                // workgroups; 0.23 us more at 16)
                uint64_t row[NEAR];
                uint64_t a = 0, b = 0;
#pragma unroll 1
                for (int polls = 0; st == PANEL_GO; ++polls) {
                    a = get_word(mine + MSG_MAG);
                    b = get_word(mine + MSG_POS);
#pragma unroll
                    for (int k = 0; k < NEAR; ++k) {
                        row[k] = (uint64_t)tag << 32;
                        if (k < G) row[k] = get_word(slot + (int64_t)k * MSG + lane);
                    }
                    bool all = tagged(a, tag) && tagged(b, tag);
#pragma unroll
                    for (int k = 0; k < NEAR; ++k) all = all && tagged(row[k], tag);
                    if (__all(all)) break;
                    if (polls >= bound) st = q == 0 && g == 0 ? PANEL_STOP : PANEL_LOST;
                }
                if (lane < G) x = Candidate{(uint32_t)a, (uint32_t)b};
                gb = lanes_best<NEAR>(x, win);
                uint32_t r = (uint32_t)row[0];
#pragma unroll
                for (int k = 1; k < NEAR; ++k) r = win == k ? (uint32_t)row[k] : r;
                rowv = __uint_as_float(r);
            } else {
#pragma unroll 1
                for (int polls = 0; st == PANEL_GO; ++polls) {
                    const uint64_t a = get_word(mine + MSG_MAG), b = get_word(mine + MSG_POS);
                    if (lane < G) x = Candidate{(uint32_t)a, (uint32_t)b};
                    if (__all(tagged(a, tag) && tagged(b, tag))) break;
                    if (polls >= bound) st = q == 0 && g == 0 ? PANEL_STOP : PANEL_LOST;
                }
                gb = lanes_best<PANEL_GROUPS>(x, win);
                const uint64_t *from = slot + (int64_t)win * MSG;
#pragma unroll 1
                for (int polls = 0; st == PANEL_GO; ++polls) {
                    const uint64_t a = get_word(from + lane);
                    rowv = __uint_as_float((uint32_t)a);
                    if (__all(tagged(a, tag))) break;
                    if (polls >= PANEL_HARD_WAIT) st = q == 0 && g == 0 ? PANEL_STOP : PANEL_LOST;
                }
            }
            if (q == 0 && g == 0) {
                if (lane == 0) st = decide(words + MSG_START, start, tag, st);
                st = __builtin_amdgcn_readfirstlane(st);
            }
            su[lane] = pivot_row(rowv);
            if (lane == 0) {
                if (st != PANEL_GO) sstate = st;
                swin = make_uint2(st == PANEL_GO ? gb.mag : 0u, gb.pos);
            }
        }
        __syncthreads();
    };

    exchange(0, 0, [](int) {});
    int state = sstate;
    bool noted = false;
#pragma unroll 1
    for (int b = 0; b < PANEL / 8 && state == PANEL_GO; ++b) {
        taken = 0;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int j = 8 * b + jj;
            ub[jj] = 0.0f;
            if (j < w) {
                const uint2 winner = swin;
                float u = su[lane];
                asm volatile("" : "+v"(u));  // read beside swin, not after a branch on it
                const uint32_t umag = (uint32_t)__builtin_amdgcn_readfirstlane((int)winner.x);
                const int p = __builtin_amdgcn_readfirstlane((int)winner.y);
                const float piv = lane_value(u, jj), urow = u;
                const bool ok = umag > MAG_ZERO;
                // multipliers, by the rounded reciprocal: the hardware's, an ulp
                // off at most, and one Newton step give what 1.0f / piv does
                // for every significand (all 2^23 compared, at exponents from
                // the least to the largest taken here); lm: as the updates of
                // this column take them
                float l[RPT], lm[RPT];
                float rinv = __builtin_amdgcn_rcpf(piv);
                rinv = fmaf(fmaf(-piv, rinv, 1.0f), rinv, rinv);
#pragma unroll
                for (int i = 0; i < RPT; ++i) lm[i] = l[i] = v[i][jj / 4][jj % 4] * rinv;
                taken |= 1u << jj;
                if (__builtin_expect(!(ok && fabsf(piv) >= FLT_MIN && fabsf(piv) < 0x1p126f), 0)) {
                    rinv = 1.0f / piv;
#pragma unroll
                    for (int i = 0; i < RPT; ++i) {
                        const float x = v[i][jj / 4][jj % 4];
                        l[i] = !ok ? x : scale_by_reciprocal(piv) ? x * rinv : x / piv;
                        lm[i] = ok ? l[i] : 0.0f;
                    }
                    if (!ok) {
                        u = 0.0f;
                        taken &= ~(1u << jj);
                    }
                }
                ub[jj] = u;
                // what the updates make of a row that is done is ignored, save
                // for its multipliers
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const bool is_p = act[i] && pos[i] == p, is_j = act[i] && pos[i] == j;
                    pos[i] = is_p ? j : is_j ? p : pos[i];
                    act[i] = act[i] && !is_p;
                    v[i][jj / 4][jj % 4] = act[i] ? l[i] : v[i][jj / 4][jj % 4];
                }
#pragma unroll
                for (int c = jj + 1; c < 8; ++c) {
                    const float uc = lane_value(u, c);
#pragma unroll
                    for (int i = 0; i < RPT; ++i)
                        v[i][c / 4][c % 4] = fmaf(-lm[i], uc, v[i][c / 4][c % 4]);
                }
                // the pivot and its row of U, by wavefronts that neither post
                // nor read
                const auto record = [&](int ow) __attribute__((always_inline)) {
                    if (g == 0) {
                        if (wave == ((ow + 2) & (PANEL_WAVES - 1))) {
                            if (lane == 0) ipiv[row0 + j] = row0 + p;
                            if (__builtin_expect(!ok, 0) && !noted && lane == 0 && *info == 0)
                                *info = (int)(row0 + j + 1);
                        }
                        if (wave == ((ow + 3) & (PANEL_WAVES - 1)) && lane >= jj &&
                            lane < PANEL - 8 * b && lane < w - 8 * b)
                            P[(int64_t)(8 * b + lane) * lda + j] = urow;
                        noted = noted || !ok;
                    }
                };
                if (jj < 7 && j + 1 < w) exchange(j + 1, jj + 1, record);
                else record(0);
            }
        }
        // the block's eight pivot rows subtracted from the later columns (the
        // finished ones sit in the registers after those)
        float nl[RPT][8];
#pragma unroll
        for (int i = 0; i < RPT; ++i)
#pragma unroll
            for (int k = 0; k < 8; ++k)
                nl[i][k] = (taken >> k) & 1 ? -v[i][k / 4][k % 4] : -0.0f;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            if (b < 7) rank8<2>(v[i], ub, nl[i]);
            if (b < 6) rank8<4>(v[i], ub, nl[i]);
            if (b < 5) rank8<6>(v[i], ub, nl[i]);
            if (b < 4) rank8<8>(v[i], ub, nl[i]);
            if (b < 3) rank8<10>(v[i], ub, nl[i]);
            if (b < 2) rank8<12>(v[i], ub, nl[i]);
            if (b < 1) rank8<14>(v[i], ub, nl[i]);
        }
        // rotate the registers by the block's eight columns
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const panel_f4 x0 = v[i][0], x1 = v[i][1];
#pragma unroll
            for (int c = 0; c < PANEL / 4 - 2; ++c) v[i][c] = v[i][c + 2];
            v[i][PANEL / 4 - 2] = x0;
            v[i][PANEL / 4 - 1] = x1;
        }
        if (8 * (b + 1) < w) exchange(8 * (b + 1), 0, [](int) {});
        state = sstate;  // of this block's exchanges too
    }
    if (state != PANEL_GO) {
        // called off before the first column, or a wait reached its hard bound
        // and nothing of the registers is used
        if (state == PANEL_STOP && g == 0)
            panel_in_memory<PANEL_THREADS>(P, lda, m, w, ipiv, row0, info);
        if (state == PANEL_LOST && t == 0) *info = -1;
        return;
    }
    // store the rows: rows that are done, up to their diagonal
    const bool plain = act[0] && act[RPT - 1] && pos[0] == r0 && pos[RPT - 1] == r0 + RPT - 1;
    if (RPT == 2 && __all(plain)) {
#pragma unroll
        for (int c = 0; c < PANEL; ++c)
            if (c < w) {
                panel_f2u x;
                x[0] = v[0][c / 4][c % 4];
                x[1] = v[RPT - 1][c / 4][c % 4];
                *reinterpret_cast<panel_f2u *>(P + (int64_t)c * lda + r0) = x;
            }
    } else {
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (r0 + i < m) {
                float *pr = P + pos[i];
                const int cols = act[i] ? w : pos[i];
#pragma unroll
                for (int c = 0; c < PANEL; ++c)
                    if (c < cols) pr[(int64_t)c * lda] = v[i][c / 4][c % 4];
            }
    }
}

}  // namespace
