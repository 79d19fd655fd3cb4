// Overlap counts on the matrix cores: the encoding and the pass test that every
// matrix kernel uses, and a tile of 256 queries x 256 rows in a workgroup (the
// blocked search's block bounds; scan_mfma_kernel, eval_kernel and
// objscan_kernel stream one side past the other without it).  For queries and
// rows (database rows or bit summaries) of 4096 bits each, C[i][j] =
// popcount(query i AND row j), the term every weighted distance and every
// node bound of Eq. 1 is built from.  Over the 4096 bit positions this is a
// dense {0,1} matrix product.  It runs as the FP4 (e2m1) matrix instruction
// v_mfma_f32_32x32x64_f8f6f4: every bit becomes one 4-bit element, zero or a
// power of two whose value on the query side is the reciprocal of its value
// on the row side, so every product is 0 or 1 and the fp32 accumulator holds
// the exact count (at most 4096 < 2^24).  The order in which bits become
// elements only has to be the same for both operands, since the sum over K
// does not depend on it.
//
// Which matrix instruction: expanding the bits takes about 17 vector
// instructions per 8 multiplications of the 32 x 32 x 64 form (32 cycles
// each), and they run beside the matrix unit only in the issue slots it
// leaves.  Measured with two waves per SIMD, cycles per 131,072 x 8
// multiply-adds (256 at the unit's rate) with 32 / 48 / 64 vector
// instructions between them: 16 x 16 x 128 with block scales 347 / 417 / 487,
// without scales 264 / 333 / 400; 32 x 32 x 64 with scales 274 / 317 / 380,
// without 267 / 278 / 334.  So: the larger form (half the operand reads per
// multiplication) without scales (the scaled form is two instructions).
//
// A block of 8 waves owns the 256 x 256 tile, and thread t owns input row t
// (queries 0..255, then rows).  The K dimension is streamed in windows of 512
// bits: each thread copies its row's window, still packed, into LDS (rows 72
// bytes apart), three windows deep: window w + 2 is loaded into registers at
// the start of window w and stored at its end, before the one barrier per
// window, so the reads of window w + 1 never wait for a barrier.  Every wave
// multiplies its 128 queries x 64 rows as 4 x 2 tiles of 32 x 32 per 64-bit
// matrix step, two steps at a time.  In double step s of a window, lane l
// reads two 32-bit words, 4s + 2 (l / 32) and the next, of row l % 32 of each
// fragment, one for each step, and expands them in registers to the 32
// elements an instruction takes from it: element 8j + i holds bit 4i + j, so
// a few shift-and-mask operations make the 16 bytes (expand_q, expand_r).
// With rows 18 words apart the lanes of such a read fall on distinct banks in
// each half.  The words of the next double step are read while the current
// one runs, and a step's operands are expanded between the multiplications of
// the step before it, so neither wave of a SIMD ever has only vector work.
//
// Measured with the sequential search on this tile (1M rows x 4,096 queries,
// kernel time; streamed past each other it takes 4.6 ms): 7.5 ms with 16 x 16 x 128,
// scales and each step's expansion before its multiplications; 6.8 ms with
// 32 x 32 x 64 without scales; 5.8 ms with the epilogue's test by row
// (pass_bound below); 5.4 ms with the expansion between the multiplications.
// Without the epilogue it takes 4.6 ms; without expansion and barriers too,
// which is what the matrix units alone reach at the clock they run at, 4.1.
//
// Rows are the instruction's first operand and queries its second, so a lane
// holds one query per fragment (column l % 32) against 16 of its 32 rows:
// entry e is row 8 (e / 4) + 4 (l / 32) + e % 4.  A kernel then tests a query's
// rows against the query's own bound lane by lane, and a minimum over the
// rows needs no exchange until its end.
//
// A missing row reads as zeros.
#pragma once

#include "qd.h"
#include "qd_device.h"

namespace qd {
namespace mt {

constexpr int kThreads = 512;  // 8 waves, one row per thread
constexpr int MA = 256;        // queries per tile
constexpr int MB = 256;        // rows per tile
constexpr int WIN = 512;       // bits per window (four double steps of 128 bits)
constexpr int QF = 4;          // 32-query fragments of a wave
constexpr int RF = 2;          // 32-row fragments of a wave
constexpr int RST = 72;        // packed row stride in LDS (64 bytes + 8 pad)
constexpr int NBUF = 3;        // windows held in LDS

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef v16f Acc[QF][RF];  // a wave's counts

struct Smem {
    uint8_t rw[NBUF][(MA + MB) * RST];  // packed windows
};

// 32 bits -> the 32 e2m1 elements of one lane's operand: element 8j + i
// (nibble i of word j) comes from bit 4i + j.  The query side keeps bits 0..2
// of each nibble where they are (values 0.5, 1 and 2); the row side gives the
// same bits the reciprocal values (2, 1 and 0.5).  Bit 3, the e2m1 sign bit,
// moves to bit 1 (value 1) on both sides, so the product of two set bits is
// exactly 1, three of the query side's four words need no shift, and the row
// side's last two words come from one shift right by 2.
__device__ __forceinline__ v8i expand_q(uint32_t w) {
    constexpr uint32_t M = 0x11111111u;
    return v8i{(int)(w & M), (int)(w & (M << 1)), (int)(w & (M << 2)), (int)((w >> 2) & (M << 1)), 0, 0, 0, 0};
}
__device__ __forceinline__ v8i expand_r(uint32_t w) {
    constexpr uint32_t M = 0x11111111u;
    const uint32_t r2 = w >> 2;
    return v8i{(int)((w << 2) & (M << 2)), (int)(w & (M << 1)), (int)(r2 & M), (int)(r2 & (M << 1)), 0, 0, 0, 0};
}

// 64 bit positions of 32 rows x 32 queries, and 128 of 16 x 16 (formats 4 =
// e2m1 for both operands; with zero scale arguments the instruction without
// scales, every element at its own value).
__device__ __forceinline__ v16f mma32(v8i rows, v8i queries, v16f c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(rows, queries, c, 4, 4, 0, 0, 0, 0);
}
__device__ __forceinline__ v4f mma16(v8i a, v8i b, v4f c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 4, 4, 0, 0, 0, 0);
}

// Workgroups are dispatched to the 8 XCDs round-robin (workgroup x runs on
// XCD x % 8), and each XCD has its own L2.  xcd_tile maps workgroup x to a
// tile index so that every XCD gets one contiguous range of the n tiles: tiles
// that share B rows (consecutive indices) then share one L2.  Returns false
// for the padding workgroups of a grid of xcd_grid(n) workgroups.
constexpr uint32_t kXcds = 8;
// A dispatch packet holds the grid size in work-items as a 32-bit number, so a
// launch of kThreads-thread workgroups stays below 2^32 / kThreads of them;
// kernels take their tiles in a workgroup-stride loop over a grid of at most
// kMaxGrid workgroups (a multiple of kXcds, so a workgroup keeps its XCD).
constexpr uint64_t kMaxGrid = 1ull << 22;
__host__ __device__ inline uint64_t tile_grid(uint64_t n) { return n < kMaxGrid ? n : kMaxGrid; }
__host__ __device__ inline uint64_t xcd_grid(uint64_t n) { return (n + kXcds - 1) / kXcds * kXcds; }
__device__ __forceinline__ bool xcd_tile(uint64_t x, uint64_t n, uint64_t &tile) {
    const uint64_t per = (n + kXcds - 1) / kXcds;
    tile = (x % kXcds) * per + x / kXcds;
    return tile < n;
}

// Input row owned by this thread (0..511; < 256 is a query).
__device__ __forceinline__ int own_row() { return (int)threadIdx.x; }

// Tile coordinates of this lane's accumulators: the query of acc[a][*][*], and
// the row of acc[*][b][4 g + e], e = 0..3, is quad_row(b, g) + e.
__device__ __forceinline__ int acc_query(int a) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    return (w >> 2) * 128 + a * 32 + (lane & 31);
}
__device__ __forceinline__ int quad_row(int b, int g) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    return (w & 3) * 64 + b * 32 + g * 8 + (lane >> 5) * 4;
}
// The pass test of the epilogues.  With wA + wB = sw (4096, or 4097 when |q| is
// 0 or 4096), K = |q|*wB + |t|*wA - C*sw <= K_k exactly when
//   C - |t| * (wA / sw) >= (|q|*wB - K_k) / sw,
// one multiply-add per pair on the left, a constant of the query on the
// right.  In fp32 both sides are within 0.003 of their values (every term is
// below 2^25, so the conversions are off by at most 2, 2 / 4096 after the
// division), so the query's bound is lowered by 0.02: no pair is lost, and
// the exact key test follows for the few that pass.
__device__ __forceinline__ float inv_sw(uint32_t pq) { return pq == 0 || pq == QD_BITS ? 1.f / 4097.f : 1.f / 4096.f; }
__device__ __forceinline__ float pass_bound(uint32_t pq, uint32_t wb, uint32_t kth) {
    return ((float)__umul24(pq, wb) - (float)kth) * inv_sw(pq) - 0.02f;
}
constexpr float kNoBound = 1e38f;  // a missing query: nothing passes
constexpr float kNoRow = 1e30f;    // a missing row's popcount: it never passes

// This lane's four rows `tp` against its query: C - |t| * ratio of each.
struct Quad {
    float v[4];
    __device__ __forceinline__ float max() const { return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])); }
};
__device__ __forceinline__ Quad quad_test(const v16f &acc, int g, const float4 &tp, float nratio) {
    return Quad{{__builtin_fmaf(tp.x, nratio, acc[4 * g]), __builtin_fmaf(tp.y, nratio, acc[4 * g + 1]),
                 __builtin_fmaf(tp.z, nratio, acc[4 * g + 2]), __builtin_fmaf(tp.w, nratio, acc[4 * g + 3])}};
}

// Exact count held by an accumulator entry.
__device__ __forceinline__ uint32_t count(float c) { return (uint32_t)c; }

// Rows: this thread's row (32 x 16 bytes), always a readable global row; when
// the zero flag is set its bits count as 0 (a missing row past the end of
// the input), read from a row of zeros, so the loaded words need no mask.  A
// global-memory pointer: a generic one would make the window loads flat
// loads, which also hold the LDS counter the fragment reads wait on (the row
// of zeros is a global variable, so a choice between it and a row stays
// global).
static __device__ uint4 kZeroRow[32];  // never written: zero-initialised

__device__ __forceinline__ const uint4 *row_or_zero(const uint4 *row, bool zero) { return zero ? kZeroRow : row; }

// LDS offset, inside a window, of the words that this lane reads of fragment
// f: f < QF queries, then rows.
__device__ __forceinline__ int frag_offset(int f) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int row = f < QF ? (w >> 2) * 128 + f * 32 : MA + (w & 3) * 64 + (f - QF) * 32;
    return (row + (lane & 31)) * RST + (lane >> 5) * 8;
}

// The counts of one tile: this thread's row is `row` (zero: a missing one).
// Every wave has read the LDS windows when it returns.
__device__ __forceinline__ void overlap_tile(const uint4 *row, bool zero, Smem &sm, Acc &acc) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int a = 0; a < QF; a++)
#pragma unroll
        for (int b = 0; b < RF; b++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[a][b][e] = 0.f;

    // window v of a row is its 16-byte pieces 4v .. 4v+3, loaded as they
    // are (a missing row from the row of zeros) and stored unchanged, so
    // nothing waits for the loads before then (and no branch skips them).
    const uint4 *const own_src = row_or_zero(row, zero);
    auto stage = [&](uint8_t *dst, uint4 p0, uint4 p1, uint4 p2, uint4 p3) {
        uint2 *d = reinterpret_cast<uint2 *>(dst + tid * RST);  // 8-byte aligned
        d[0] = make_uint2(p0.x, p0.y);
        d[1] = make_uint2(p0.z, p0.w);
        d[2] = make_uint2(p1.x, p1.y);
        d[3] = make_uint2(p1.z, p1.w);
        d[4] = make_uint2(p2.x, p2.y);
        d[5] = make_uint2(p2.z, p2.w);
        d[6] = make_uint2(p3.x, p3.y);
        d[7] = make_uint2(p3.z, p3.w);
    };
    // the first two windows
#pragma unroll
    for (int v = 0; v < 2; v++)
        stage(sm.rw[v], own_src[4 * v], own_src[4 * v + 1], own_src[4 * v + 2], own_src[4 * v + 3]);
    __syncthreads();
    constexpr int kWins = 4096 / WIN;
    int roff[QF + RF];
#pragma unroll
    for (int f = 0; f < QF + RF; f++) roff[f] = frag_offset(f);
    uint64_t r[2][QF + RF];  // the words of this double step and of the next
#pragma unroll
    for (int f = 0; f < QF + RF; f++) r[0][f] = *reinterpret_cast<const uint64_t *>(sm.rw[0] + roff[f]);
    // Operands of the two steps of a double step.  While a step's eight
    // multiplications run, the other step's operands are expanded between
    // them, one fragment after each, so a wave always has a multiplication to
    // issue; sched_barrier keeps that order.
    v8i qv[2][QF], rv[2][RF];
    auto expand = [&](int h, int f, uint32_t x) {  // fragment order: rows first, both are needed first
        if (f < RF)
            rv[h][f] = expand_r(x);
        else
            qv[h][f - RF] = expand_q(x);
    };
    // the words of fragment f (rows first) of a double step: low and high
    auto lo = [&](const uint64_t (&x)[QF + RF], int f) { return (uint32_t)x[f < RF ? QF + f : f - RF]; };
    auto hi = [&](const uint64_t (&x)[QF + RF], int f) { return (uint32_t)(x[f < RF ? QF + f : f - RF] >> 32); };
    auto multiply = [&](int h, auto &&words) {
#pragma unroll
        for (int m = 0; m < QF * RF; m++) {
            acc[m / RF][m % RF] = mma32(rv[h][m % RF], qv[h][m / RF], acc[m / RF][m % RF]);
            if (m < QF + RF) expand(h ^ 1, m, words(m));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int f = 0; f < QF + RF; f++) expand(0, f, lo(r[0], f));
    // Every window runs the same code, so the compiler keeps one loop instead
    // of peeling its end (a peeled end spilled registers in the kernels).
    // (The last two stage the row's first windows again: in bounds, never used.)
    int cur = 0;  // buffer of window win; window win + 1 is in the next, win + 2 goes to the one after
    for (int win = 0; win < kWins; win++) {
        const int nxt = cur == NBUF - 1 ? 0 : cur + 1, stg = nxt == NBUF - 1 ? 0 : nxt + 1;
        const uint8_t *buf = sm.rw[cur];
        const int nb = (4 * win + 8) & 31;  // window win + 2
        const uint4 n0 = own_src[nb], n1 = own_src[nb + 1], n2 = own_src[nb + 2], n3 = own_src[nb + 3];
#pragma unroll
        for (int s = 0; s < 4; s++) {
            // the next step's words: from this window, or the first of the next
            // window (published by the previous window's barrier)
            const uint8_t *from = s < 3 ? buf + (s + 1) * 16 : sm.rw[nxt];
#pragma unroll
            for (int f = 0; f < QF + RF; f++) r[(s + 1) & 1][f] = *reinterpret_cast<const uint64_t *>(from + roff[f]);
            // the next double step's reads go out before this one's work
            __builtin_amdgcn_sched_barrier(0);
            multiply(0, [&](int f) { return hi(r[s & 1], f); });
            multiply(1, [&](int f) { return lo(r[(s + 1) & 1], f); });
            __builtin_amdgcn_sched_barrier(0);
        }
        // the buffer of window win - 1: every wave finished reading it before
        // the previous barrier
        stage(sm.rw[stg], n0, n1, n2, n3);
        __syncthreads();
        cur = nxt;
    }
}

}  // namespace mt
}  // namespace qd
