// Sequential search of query batches on the matrix cores.
//
// For many queries the overlap counts C[q][t] = popcount(q AND t) of Eq. 1
// form a dense {0,1} matrix product C = Q T^T over the 4096 bit positions;
// scan_mfma_kernel computes them in the encoding of mfma_tile.h.
//
// Selection, in three passes of the same kernel: a sample of the rows (spread
// evenly over them, sample_row) gives each query the smallest key of every group of
// 32 sampled rows; the k-th smallest of those bounds the query's k-th key from
// above (k distinct rows reach it).  The matrix pass then keeps every (row,
// key) up to the bound in a per-query candidate buffer; the exact top k are
// all among them.  A long pass runs in parts: after the first (an eighth of the
// rows) the bounds are tightened to the k-th key found so far, so the rest
// lists about 7 k rows per query.  A bound is a full key (K << 32 | row): of
// rows with equal K (repeated or blank descriptors, a blank query) only those
// up to the bound's row are kept, so ties do not fill the buffer.  A final kernel selects each query's k best
// candidates and writes the results.  A query whose buffer overflowed, which
// takes rows whose order meets the sample's, is bounded by the k-th smallest of
// the candidates it holds (rows all the same) and passed over the rows once
// more, with the others like it only; should it overflow again, one workgroup
// reads all rows for it, so the result is exact in every case.
#include <math.h>

#include <algorithm>
#include <vector>

#include "mfma_tile.h"
#include "qd_device.h"
#include "qd_internal.h"
#include "qd_launch.h"

namespace qd {

namespace {

constexpr int kBlock = 256;
constexpr uint32_t kCap = 8192;        // candidate slots per query at most
// A pass takes as many queries as a workspace of 1 GB serves, at least 16,384 (up
// to 96 KB each): so many are bound by the matrix units, and the rows are read
// again for the next ones at no cost that can be seen.
constexpr uint32_t kMinBatch = 16384;
constexpr uint64_t kBatchBytes = 1ull << 30;
constexpr uint32_t kMaxGroups = 8192;  // sample minima per query

// ---------------------------------------------------------------------------
// The matrix pass.  A wave streams 64 rows at a time, straight from memory into
// the matrix instruction's operand registers, against 64 queries that its
// workgroup keeps packed in LDS (a group of up to 256 queries): 2 x 2 fragments
// of 32 rows x 32 queries.  The work is cut into units, (group, 64-row tile,
// 64-query tile of the group), in that order; every workgroup of the
// persistent grid takes an equal run of row tiles and its 8 waves take the
// run's units in turn, so waves that share a row tile read it together.
// Waves share nothing but the queries: the only barriers are around a change
// of group.
// Bits -> K order (the same for rows and queries): line L of a row (128 bytes),
// piece pair i, half h = lane / 32: the lane holds the 16-byte piece 8L + 2i + h
// of row l % 32, and matrix step S = 16 L + 4 i + c takes its word c.  A line's
// 8 loads (4 per fragment) are issued together, a line ahead; the operands of
// a step are expanded between the multiplications of the step before it, over
// the ends of units too.  |t| is counted from the same words.
// kSample: instead of listing the rows that pass, the smallest key of the
// lane's 32 rows of each query goes to minima[(2 i + h) * nq + query], i the
// tile's number in this pass, as (K << 5 | the row's number among the lane's; K < 2^25).
// Bound: the rows' bytes for up to 64 queries (5.8 TB/s), the matrix units above
// (7.2 PFLOP/s at 256 queries; they reach about 8.1 at the clock they run at).
// 10M rows, k = 10, whole calls with 32 / 64 / 128 / 256 queries: 0.97 / 0.99 /
// 1.65 / 3.0 ms.  The row scan's 16-query tiles, which expand every row once per
// 16 queries, took 1.4 / 2.4 / 4.5 ms, and a 256 x 256 tile per block (rows and
// queries staged in LDS, a barrier per 512 bits) 5.8 ms at 256; 4,096 queries x
// 1M rows 4.6 ms against 5.4 on that tile.
constexpr int kMidBlock = 512;
constexpr int kMidWaves = kMidBlock / 64;
constexpr int kMidQ = 64, kMidR = 64;     // queries and rows of a unit
constexpr uint32_t kGroupQ = 4 * kMidQ;   // queries of a group
constexpr uint32_t kMidQueue = 128;       // passing pairs per wave: room for one row's 64 past the flush mark
constexpr int kMidStride = 512 + 16;      // bytes per query in LDS: 16-byte reads of 32 rows on distinct banks

// Row of the sample's entry i: one out of every n / entries rows, at a place
// that a hash of i picks, so that no period of the rows meets the sample's.
// step = n / entries in 32.32 fixed point, at least 1.  The sample's tile t has
// one entry of each 64th of the rows, sample_entry: the 64 rows of a tile lie far
// apart, and near rows (rows of one object, rows in order of distance, repeated
// rows, one view of every object) in different groups, of which each adds one key
// to the bound.  With whole tiles sampled
// a run of tied or similar rows filled few groups, and up to 16,000 of its rows
// passed: 64 queries x 10M rows that are all equal 1.4 ms, 17 then.
__device__ __forceinline__ uint64_t sample_row(uint32_t i, uint64_t step) {
    const uint32_t a = (uint32_t)((i * step) >> 32), b = (uint32_t)(((uint64_t)(i + 1) * step) >> 32);
    uint32_t h = i * 2654435761u;  // multiplicative hashing by the golden ratio, twice
    h = (h ^ (h >> 16)) * 2654435761u;
    return a + __umulhi(h, b - a);
}

// (the same place of the next 64th is 5/8 of the tiles on)
__device__ __forceinline__ uint32_t sample_turn(uint32_t slot, uint32_t tiles) {
    return slot * (tiles * 5 / 8 + 1) % tiles;
}
__device__ __forceinline__ uint32_t sample_entry(uint32_t slot, uint32_t turn, uint32_t tile, uint32_t tiles) {
    const uint32_t x = tile + turn;
    return slot * tiles + (x < tiles ? x : x - tiles);
}

// LDS, sized by the queries of the largest group.
struct MidSmem {
    uint32_t pop[kGroupQ];            // |q|
    u64 thr[kGroupQ];                 // candidate bound
    float bound[kGroupQ];             // pass test's bound
    uint32_t id[kGroupQ];             // kAgain: the query's number
    float tp[kMidWaves][kMidR];       // per wave: its rows' |t|
    uint32_t queue[kMidWaves][kMidQueue][3];  // per wave: passing (query, key, row)
};
inline size_t mid_lds_bytes(uint32_t nq) {
    const uint32_t q = nq < kGroupQ ? (nq + kMidQ - 1) / kMidQ * kMidQ : kGroupQ;
    return sizeof(MidSmem) + (size_t)q * kMidStride;
}

// kAgain: the queries are those of `list`.
enum Pass { kFirst, kSample, kAgain };
template <Pass kPass>
__global__ __launch_bounds__(kMidBlock, 2) void scan_mfma_kernel(const uint4 *__restrict__ db, uint64_t n, uint64_t t0,
                                                                 uint64_t tiles, uint64_t sample_step,
                                                                 const uint4 *__restrict__ q, uint32_t nq,
                                                                 const u64 *__restrict__ thr, uint32_t *__restrict__ cnt,
                                                                 u64 *__restrict__ cand, uint32_t cap,
                                                                 uint32_t *__restrict__ minima,
                                                                 const uint32_t *__restrict__ list,
                                                                 const uint32_t *__restrict__ nq_dev) {
    extern __shared__ __align__(16) uint8_t s_raw[];
    MidSmem &sm = *reinterpret_cast<MidSmem *>(s_raw);
    uint8_t *s_q = s_raw + sizeof(MidSmem);
    static_assert(sizeof(MidSmem) % 16 == 0, "the queries are read 16 bytes at a time");
    const uint32_t nq_given = nq;
    if (nq_dev) nq = min(nq, *nq_dev);  // the batch's size on the device (captured graphs)
    const int lane = threadIdx.x & 63, wv = (int)readfirst(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;
    float *tpw = sm.tp[wv];
    uint32_t (*cq)[3] = sm.queue[wv];
    uint32_t turn[2] = {0, 0};
    if (kPass == kSample) {
#pragma unroll
        for (int b = 0; b < 2; b++) turn[b] = sample_turn(32 * b + li, (uint32_t)tiles);
    }
    // the pass's row tiles: t0 + i, i < tiles (kSample: the sample's)
    const uint32_t nq_max = nq_given, n_qt = (nq + kMidQ - 1) / kMidQ;
    // this workgroup's units [ua, ub) of all groups' (each group: its query
    // tiles x tiles), rounded down to whole row tiles at both ends
    const uint64_t units = tiles * n_qt;
    const uint64_t ua = units / gridDim.x * blockIdx.x + min((uint64_t)blockIdx.x, units % gridDim.x);
    const uint64_t ub = ua + units / gridDim.x + (blockIdx.x < units % gridDim.x ? 1 : 0);

    uint32_t nqe = 0;  // entries in this wave's queue (the same in every lane)
    auto flush = [&](uint32_t q0) {
        for (uint32_t e = lane; e < nqe; e += 64) {
            const uint32_t qs = cq[e][0], qk = kPass == kAgain ? sm.id[qs] : q0 + qs;
            const uint32_t pos = atomicAdd(&cnt[qk], 1u);
            if (pos < cap)
                cand[(uint64_t)qk * cap + pos] = ((u64)cq[e][1] << 32) | cq[e][2];
            else  // the query is searched again: no more of its rows here
                sm.bound[qs] = mt::kNoBound;
        }
        nqe = 0;
    };
    const uint64_t per_group = 4 * tiles;  // units of a full group
    for (uint64_t g0 = ua / per_group * per_group; g0 < ub; g0 += per_group) {
        const uint32_t q0 = (uint32_t)(g0 / per_group) * kGroupQ;               // the group's first query
        const uint32_t gqt = min(4u, n_qt - q0 / kMidQ);                         // its query tiles
        const uint64_t ra = (ua > g0 ? ua - g0 : 0) / gqt;                       // its row tiles here
        const uint64_t rb = min((ub - g0) / gqt, tiles);
        __syncthreads();  // every wave is done with the group before
        for (uint32_t e = threadIdx.x; e < gqt * kMidQ * 32; e += kMidBlock) {
            uint32_t qi = q0 + (e >> 5);
            const bool real = qi < nq;
            if (kPass == kAgain) qi = list[real ? qi : 0];
            const uint4 x = real ? q[(uint64_t)qi * 32 + (e & 31)] : make_uint4(0, 0, 0, 0);
            *reinterpret_cast<uint4 *>(s_q + (size_t)(e >> 5) * kMidStride + (e & 31) * 16) = x;
            const uint32_t pq = sum32_half(popc4(x));  // a half wave holds one query
            if ((e & 31) == 0) {
                const uint32_t wb = (QD_BITS - pq) > 1 ? QD_BITS - pq : 1;
                const u64 th = kPass != kSample && real ? thr[qi] : 0;
                sm.pop[e >> 5] = pq;
                sm.thr[e >> 5] = th;
                if (kPass == kAgain) sm.id[e >> 5] = qi;
                sm.bound[e >> 5] = real ? mt::pass_bound(pq, wb, (uint32_t)(th >> 32)) : mt::kNoBound;
            }
        }
        __syncthreads();
        // the wave's units wv, wv + 8, ... of (rb - ra) row tiles x gqt query tiles
        const uint64_t un = (rb - ra) * gqt;
        uint64_t u = (uint64_t)wv;
        if (u >= un) continue;
        uint32_t qt = (uint32_t)wv % gqt;
        uint64_t rt = ra + (uint32_t)wv / gqt;  // the pass's row tile
        // rows 32 b + li of row tile r (past the end: the last row, masked in the test)
        uint4 v[2][2][4];  // [line parity][fragment][piece pair]
        auto load = [&](uint64_t r, int L, uint4 (&x)[2][4]) {
#pragma unroll
            for (int b = 0; b < 2; b++) {
                uint64_t row = kPass == kSample
                                   ? sample_row(sample_entry(32 * b + li, turn[b], (uint32_t)r, (uint32_t)tiles),
                                                sample_step)
                                   : (t0 + r) * kMidR + 32 * b + li;
                row = row < n ? row : n - 1;
                const uint4 *src = db + row * 32 + 8 * L + lh;
#pragma unroll
                for (int i = 0; i < 4; i++) x[b][i] = src[2 * i];
            }
        };
        auto q_row = [&](uint32_t t) { return s_q + (size_t)(t * kMidQ + li) * kMidStride + lh * 16; };
        auto word = [](const uint4 &x, int c) { return c == 0 ? x.x : c == 1 ? x.y : c == 2 ? x.z : x.w; };
        const uint8_t *qrow = q_row(qt);
        uint4 qw[2][2];         // queries' pieces: [piece pair parity][fragment]
        mt::v8i qv[2][2], rv[2][2];  // operands: [step parity][fragment]
        uint32_t tp[2] = {0, 0};
        auto read_q = [&](const uint8_t *row, int pair) {
#pragma unroll
            for (int a = 0; a < 2; a++)
                qw[pair & 1][a] = *reinterpret_cast<const uint4 *>(row + 32 * a * kMidStride + pair * 32);
        };
        auto expand = [&](int S, int f) {  // fragment f of step S (mod 64): rows 0, 1, then queries
            const int L = (S >> 4) & 3, i = (S >> 2) & 3, c = S & 3;
            if (f < 2) {
                const uint32_t x = word(v[L & 1][f][i], c);
                rv[S & 1][f] = mt::expand_r(x);
                tp[f] += __popc(x);
            } else {
                qv[S & 1][f - 2] = mt::expand_q(word(qw[(4 * L + i) & 1][f - 2], c));
            }
        };
        load(rt, 0, v[0]);
        read_q(qrow, 0);
#pragma unroll
        for (int f = 0; f < 4; f++) expand(0, f);
        for (;;) {
            // the wave's next unit (after the last: this one again, unused)
            const bool more = u + kMidWaves < un;
            uint32_t nqt = qt + kMidWaves % gqt;
            const uint32_t wrap = nqt >= gqt ? 1 : 0;
            nqt -= wrap ? gqt : 0;
            const uint64_t nrt = more ? rt + kMidWaves / gqt + wrap : rt;  // row tile, then query tile
            const uint8_t *nqrow = q_row(more ? nqt : qt);
            mt::v16f acc[2][2];
            uint32_t tcur[2];
#pragma unroll
            for (int L = 0; L < 4; L++) {
                load(L < 3 ? rt : nrt, (L + 1) & 3, v[(L + 1) & 1]);
#pragma unroll
                for (int st = 0; st < 16; st++) {
                    const int S = 16 * L + st;
                    if ((S & 3) == 0) read_q(S < 60 ? qrow : nqrow, (S / 4 + 1) & 15);
                    if (S == 63) {  // from here on the next unit's rows are counted
                        tcur[0] = tp[0];
                        tcur[1] = tp[1];
                        tp[0] = tp[1] = 0;
                    }
#pragma unroll
                    for (int m = 0; m < 4; m++) {
                        const mt::v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                                               0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                        acc[m >> 1][m & 1] =
                            mt::mma32(rv[S & 1][m & 1], qv[S & 1][m >> 1], S == 0 ? zero : acc[m >> 1][m & 1]);
                        expand(S + 1, m);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            // |t| of the tile's rows, to every lane through the wave's LDS
            const uint64_t row0 = (t0 + rt) * kMidR;  // (not the sample's rows, which all exist)
#pragma unroll
            for (int b = 0; b < 2; b++) {
                tcur[b] += (uint32_t)__shfl_xor((int)tcur[b], 32);
                if (lh == b) tpw[32 * b + li] = kPass == kSample || row0 + 32 * b + li < n ? (float)tcur[b] : mt::kNoRow;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int a = 0; a < 2; a++) {
                const uint32_t qs = qt * kMidQ + 32 * a + li;  // this lane's query
                const float bound = sm.bound[qs];
                const uint32_t pq = sm.pop[qs];
                const uint32_t wa = pq > 1 ? pq : 1, wb = (QD_BITS - pq) > 1 ? QD_BITS - pq : 1;
                if (kPass == kSample) {
                    // K = |q|*wB - (C*(wA + wB) - |t|*wA), exact in fp32 (integers
                    // below 2^24, but for C = |q| = 4096: 4096 * 4097 is even)
                    const float sw = (float)(wa + wb), nwa = -(float)wa;
                    int32_t best = INT32_MIN;
#pragma unroll
                    for (int b = 0; b < 2; b++)
#pragma unroll
                        for (int g = 0; g < 4; g++) {
                            const float4 t4 = *reinterpret_cast<const float4 *>(tpw + 32 * b + 8 * g + 4 * lh);
                            const float t[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                const float v = __builtin_fmaf(t[e], nwa, acc[a][b][4 * g + e] * sw);
                                best = max(best, (int32_t)v * 32 + (31 - (16 * b + 4 * g + e)));
                            }
                        }
                    if (q0 + qs < nq)
                        minima[(2 * rt + lh) * nq_max + q0 + qs] = 32 * __umul24(pq, wb) + 31 - (uint32_t)best;
                    continue;
                }
                const float nratio = -(float)wa * mt::inv_sw(pq);
#pragma unroll
                for (int b = 0; b < 2; b++) {
                    // 16 rows at once, then four at a time, then one (most miss by far)
                    mt::Quad x[4];
#pragma unroll
                    for (int g = 0; g < 4; g++)
                        x[g] = mt::quad_test(acc[a][b], g,
                                             *reinterpret_cast<const float4 *>(tpw + 32 * b + 8 * g + 4 * lh), nratio);
                    const float mx = fmaxf(fmaxf(x[0].max(), x[1].max()), fmaxf(x[2].max(), x[3].max()));
                    if (ballot(mx >= bound) == 0) continue;
                    const u64 th = sm.thr[qs];
                    // K = |q|*wB + |t|*wA - C*(wA + wB): 24-bit multiplies (C <= 4096
                    // and wA + wB <= 4097; every term below 2^26)
                    const uint32_t P = __umul24(pq, wb);
                    const int nsw = -(int)(wa + wb);
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        if (ballot(x[g].max() >= bound) == 0) continue;
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const bool act = x[g].v[e] >= bound;
                            if (ballot(act) == 0) continue;
                            const int ro = 32 * b + 8 * g + 4 * lh + e;
                            const uint32_t row = (uint32_t)row0 + ro;
                            const uint32_t K = (uint32_t)((int)(P + __umul24((uint32_t)tpw[ro], wa)) +
                                                          __mul24((int)mt::count(acc[a][b][4 * g + e]), nsw));
                            const bool pass = act & ((((u64)K << 32) | row) <= th);
                            const u64 pm = ballot(pass);
                            if (pass) {
                                const uint32_t at = nqe + lanes_below(pm);
                                cq[at][0] = qs;
                                cq[at][1] = K;
                                cq[at][2] = row;
                            }
                            nqe += (uint32_t)__popcll(pm);
                            if (nqe > kMidQueue - 64) flush(q0);  // the next row adds at most 64
                        }
                    }
                }
            }
            if (!more) break;
            u += kMidWaves;
            qt = nqt;
            rt = nrt;
            qrow = nqrow;
        }
        flush(q0);
    }
}

// Selection among a query's m <= cap candidates by the whole block: thread t
// holds the K of candidates t, t + 256, ... (R of them; no candidate: all
// ones).  The k-th smallest of the threads' least K, which every wave finds for
// itself by bisection over 256 values, leaves little more than k candidates to
// rank; where more than 256 are left (ties), the k-th K and then the row are
// bisected over all of them, a barrier per count.
template <int R>
struct Pick {
    uint32_t kv[R];
    uint32_t (*s_part)[4];  // LDS, [2][4]: the waves' counts, alternating (one barrier per count)
    int ph = 0;
    template <class F>
    __device__ __forceinline__ Pick(F &&key, uint32_t m, uint32_t (*part)[4]) : s_part(part) {
#pragma unroll
        for (int j = 0; j < R; j++) {
            const uint32_t i = threadIdx.x + (uint32_t)kBlock * j;
            kv[j] = i < m ? key(i) : 0xFFFFFFFFu;
        }
    }
    template <class F>
    __device__ __forceinline__ uint32_t count(F &&f) {  // candidates j for which f(j), in every thread
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < R; j++) c += (uint32_t)__popcll(ballot(f(j)));
        if ((threadIdx.x & 63) == 0) s_part[ph][threadIdx.x >> 6] = c;
        __syncthreads();
        c = s_part[ph][0] + s_part[ph][1] + s_part[ph][2] + s_part[ph][3];
        ph ^= 1;
        return c;
    }
    __device__ __forceinline__ uint32_t kth(uint32_t k) {  // the k-th smallest K (at least k candidates)
        uint32_t lo = 0, hi = (1u << 25) - 1;              // keys are below 2^25
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2;
            if (count([&](int j) { return kv[j] <= mid; }) >= k)
                hi = mid;
            else
                lo = mid + 1;
        }
        return lo;
    }
    // the need-th smallest row(i) of the candidates i of K = kth (at least need >= 1 of them)
    template <class F>
    __device__ __forceinline__ uint32_t nth_row(uint32_t kth, uint32_t need, F &&row) {
        uint32_t rv[R];
#pragma unroll
        for (int j = 0; j < R; j++) rv[j] = kv[j] == kth ? row(threadIdx.x + (uint32_t)kBlock * j) : 0xFFFFFFFFu;
        uint32_t lo = 0, hi = 0xFFFFFFFFu;
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if (count([&](int j) { return rv[j] <= mid; }) >= need)
                hi = mid;
            else
                lo = mid + 1;
        }
        return lo;
    }
    // a K that k candidates or more, usually few more, do not exceed (at least k candidates, k <= 64)
    __device__ __forceinline__ uint32_t near(uint32_t k) {
        __shared__ uint32_t s_least[kBlock];
        uint32_t mn = kv[0], v[4];
#pragma unroll
        for (int j = 1; j < R; j++) mn = min(mn, kv[j]);
        s_least[threadIdx.x] = mn;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = s_least[64 * i + (threadIdx.x & 63)];
        uint32_t lo = 0, hi = (1u << 25) - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2;
            uint32_t c = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) c += (uint32_t)__popcll(ballot(v[i] <= mid));
            if (c >= k)
                hi = mid;
            else
                lo = mid + 1;
        }
        return lo;
    }
    // the k-th smallest (K << 32 | row(i)) of the candidates (at least k of them, k <= 64)
    template <class F>
    __device__ __forceinline__ u64 kth_key(uint32_t k, F &&row) {
        __shared__ u64 s_key[kBlock], s_kth;
        __shared__ uint32_t s_n;
        if (threadIdx.x == 0) s_n = 0;
        const uint32_t U = near(k);  // (its barrier publishes s_n)
#pragma unroll
        for (int j = 0; j < R; j++)
            if (kv[j] <= U) {
                const uint32_t at = atomicAdd(&s_n, 1u);
                if (at < (uint32_t)kBlock) s_key[at] = ((u64)kv[j] << 32) | row(threadIdx.x + (uint32_t)kBlock * j);
            }
        __syncthreads();
        const uint32_t n = s_n;
        if (n > (uint32_t)kBlock) {
            const uint32_t K = kth(k), need = k - count([&](int j) { return kv[j] < K; });
            return ((u64)K << 32) | nth_row(K, need, row);
        }
        if (threadIdx.x < n) {
            uint32_t rank = 0;
            for (uint32_t j = 0; j < n; j++) rank += s_key[j] < s_key[threadIdx.x];
            if (rank == k - 1) s_kth = s_key[threadIdx.x];
        }
        __syncthreads();
        return s_kth;
    }
};

// After a part of a pass: the k-th smallest key found so far bounds the rest
// (those k rows are real).  One block per query.
__global__ __launch_bounds__(kBlock) void tighten_kernel(const uint32_t *__restrict__ cnt,
                                                         const u64 *__restrict__ cand, uint32_t cap, uint32_t k,
                                                         u64 *__restrict__ thr, const uint32_t *__restrict__ nq_dev) {
    __shared__ uint32_t s_part[2][4];
    const uint32_t qi = blockIdx.x;
    if (nq_dev && qi >= *nq_dev) return;  // whole block
    const uint32_t m = cnt[qi];
    if (m > cap && threadIdx.x == 0) thr[qi] = 0;  // searched again: nothing more is listed now
    if (m < k || m > cap) return;
    const u64 *c = cand + (uint64_t)qi * cap;
    auto key = [&](uint32_t i) { return (uint32_t)(c[i] >> 32); };
    auto row = [&](uint32_t i) { return (uint32_t)c[i]; };
    const u64 t = m <= 4 * kBlock ? Pick<4>(key, m, s_part).kth_key(k, row)
                                  : Pick<kCap / kBlock>(key, m, s_part).kth_key(k, row);
    if (threadIdx.x == 0 && t < thr[qi]) thr[qi] = t;
}

// The k smallest of m candidates (all of them if fewer) into keys[0 .. *n), in
// any order, with others, at most kBlock: the keys up to near(k), or, where these
// are more than kBlock, up to the k-th K, or, where more tie there, the tied rows
// up to the last one needed.
template <int R>
__device__ __forceinline__ void pick_keys(const u64 *cand, uint32_t m, uint32_t k, uint32_t (*s_part)[4], u64 *keys,
                                          uint32_t *n) {
    Pick<R> P([&](uint32_t i) { return (uint32_t)(cand[i] >> 32); }, m, s_part);
    uint32_t kth = P.near(k), last = 0xFFFFFFFFu;  // rows above `last` with K = kth are left out
    if (P.count([&](int j) { return P.kv[j] <= kth; }) > (uint32_t)kBlock) {
        kth = P.kth(k);
        if (P.count([&](int j) { return P.kv[j] <= kth; }) > (uint32_t)kBlock) {
            const uint32_t need = k - P.count([&](int j) { return P.kv[j] < kth; });
            last = P.nth_row(kth, need, [&](uint32_t i) { return (uint32_t)cand[i]; });
        }
    }
#pragma unroll
    for (int j = 0; j < R; j++) {
        const uint32_t i = threadIdx.x + (uint32_t)kBlock * j;
        if (P.kv[j] <= kth && i < m) {
            const u64 e = cand[i];
            if (P.kv[j] < kth || (uint32_t)e <= last) keys[atomicAdd(n, 1u)] = e;
        }
    }
}

// The k best of a query's m <= cap candidates into keys[0 .. result), in
// order, by the whole block (up to kBlock of them, at least k if m is).
// Selecting before sorting leaves a few keys to order: 0.08 ms for
// 4,096 queries with 1,000 candidates each, where sorting them all took 0.32.
__device__ __forceinline__ uint32_t best_candidates(const u64 *c, uint32_t m, uint32_t k, uint32_t (*s_part)[4],
                                                    u64 *keys, uint32_t *s_n) {
    uint32_t nk = m;
    if (m <= (uint32_t)kBlock) {
        if (threadIdx.x < m) keys[threadIdx.x] = c[threadIdx.x];
    } else {  // m > k
        if (threadIdx.x == 0) *s_n = 0;  // read after the selection's barriers
        if (m <= 4 * kBlock)
            pick_keys<4>(c, m, k, s_part, keys, s_n);
        else
            pick_keys<kCap / kBlock>(c, m, k, s_part, keys, s_n);
        __syncthreads();
        nk = *s_n;
    }
    __syncthreads();
    rank_sort(keys, nk);
    return nk;
}

// The k best of all n rows for one query, in order, into keys[0 .. k), by the
// whole block; thr: the key of a k-th row or of a later one.  8 lanes per row,
// 128 rows a step; the keys up to the bound are collected and cut to the k
// smallest whenever 128 are there.  For a query that overflows twice only.
__device__ __forceinline__ void best_of_all(const uint4 *db, uint64_t n, const uint4 *q, uint32_t k, u64 thr, u64 *keys,
                                            uint32_t *s_n) {
    const int g = threadIdx.x >> 3, j = threadIdx.x & 7;
    uint4 qv[4];
    uint32_t pq = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        qv[i] = q[j + 8 * i];
        pq += popc4(qv[i]);
    }
    pq = sum8(pq);
    const uint32_t wa = pq > 1 ? pq : 1, wb = (QD_BITS - pq) > 1 ? QD_BITS - pq : 1;
    if (threadIdx.x == 0) *s_n = 0;
    __syncthreads();
    for (uint64_t base = 0; base < n; base += 4 * (kBlock / 8)) {
        uint32_t c[4], tp[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint64_t r = base + u * (kBlock / 8) + g, row = r < n ? r : n - 1;
            c[u] = tp[u] = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint4 t = db[row * 32 + j + 8 * i];
                c[u] += popc_and4(t, qv[i]);
                tp[u] += popc4(t);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint64_t r = base + u * (kBlock / 8) + g;
            const uint32_t o = sum8(c[u]), a = pq - o, b = sum8(tp[u]) - o;
            const u64 key = ((u64)(a * wb + b * wa) << 32) | (uint32_t)r;
            if (j == 0 && r < n && key <= thr) keys[atomicAdd(s_n, 1u)] = key;
        }
        __syncthreads();
        const uint32_t m = *s_n;
        __syncthreads();  // every thread has read it
        if (m > (uint32_t)kBlock / 2 || base + 4 * (kBlock / 8) >= n) {
            rank_sort(keys, m);
            if (m > k) thr = keys[k - 1];
            if (threadIdx.x == 0) *s_n = m < k ? m : k;
            __syncthreads();
        }
    }
}

// One block per query: the k best of its candidates and their results.  An
// overflowed query (its candidates held are any cap of the rows that passed)
// is listed in `list` for another pass, bounded by the k-th smallest of them.
__global__ __launch_bounds__(kBlock) void select_emit_kernel(uint32_t *__restrict__ cnt, const u64 *__restrict__ cand,
                                                             uint32_t cap, uint32_t k, const uint4 *__restrict__ q,
                                                             const uint4 *__restrict__ db, uint32_t *idx,
                                                             int32_t *missed, int32_t *extra, float *dist,
                                                             u64 *__restrict__ thr, uint32_t *__restrict__ list,
                                                             uint32_t *__restrict__ n_list,
                                                             const uint32_t *__restrict__ nq_dev) {
    __shared__ u64 keys[kBlock];
    __shared__ uint32_t s_part[2][4], s_n;
    const uint32_t qi = blockIdx.x;
    if (nq_dev && qi >= *nq_dev) return;  // whole block
    const uint32_t m = cnt[qi];
    const u64 *c = cand + (uint64_t)qi * cap;
    if (m > cap) {
        const u64 t = Pick<kCap / kBlock>([&](uint32_t i) { return (uint32_t)(c[i] >> 32); }, cap, s_part)
                          .kth_key(k, [&](uint32_t i) { return (uint32_t)c[i]; });
        if (threadIdx.x == 0) {
            list[atomicAdd(n_list, 1u)] = qi;
            thr[qi] = t;
            cnt[qi] = 0;
        }
        return;
    }
    const uint32_t nk = best_candidates(c, m, k, s_part, keys, &s_n);
    emit_rows(keys, nk < k ? nk : k, k, q + (uint64_t)qi * 32, db, (uint64_t)qi * k, idx, missed, extra, dist);
}

// The results of the queries that were passed over the rows again.
__global__ __launch_bounds__(kBlock) void select_again_kernel(const uint32_t *__restrict__ cnt,
                                                              const u64 *__restrict__ cand, uint32_t cap, uint32_t k,
                                                              const uint4 *__restrict__ q,
                                                              const uint4 *__restrict__ db, uint64_t n, uint32_t *idx,
                                                              int32_t *missed, int32_t *extra, float *dist,
                                                              const u64 *__restrict__ thr,
                                                              const uint32_t *__restrict__ list,
                                                              const uint32_t *__restrict__ n_list) {
    __shared__ u64 keys[kBlock];
    __shared__ uint32_t s_part[2][4], s_n;
    const uint32_t n_again = *n_list;
    for (uint32_t i = blockIdx.x; i < n_again; i += gridDim.x) {
        const uint32_t qi = list[i], m = cnt[qi];
        uint32_t nk = k;
        if (m <= cap)
            nk = best_candidates(cand + (uint64_t)qi * cap, m, k, s_part, keys, &s_n);
        else
            best_of_all(db, n, q + (uint64_t)qi * 32, k, thr[qi], keys, &s_n);
        emit_rows(keys, nk < k ? nk : k, k, q + (uint64_t)qi * 32, db, (uint64_t)qi * k, idx, missed, extra, dist);
        __syncthreads();  // the next query writes over the keys
    }
}

// thr[q] = the k-th smallest key (K << 32 | row) of the query's m <= kMaxGroups
// sample minima (m >= k); clears the pass's candidate counts and its overflow
// count.  One block per query.
__global__ __launch_bounds__(kBlock) void sample_threshold_kernel(const uint32_t *__restrict__ minima, uint32_t m,
                                                                  uint64_t sample_step, uint32_t nq, uint32_t k, u64 *__restrict__ thr,
                                                                  uint32_t *__restrict__ cnt,
                                                                  uint32_t *__restrict__ n_again,
                                                                  const uint32_t *__restrict__ nq_dev) {
    __shared__ uint32_t s_part[2][4];
    const uint32_t qi = blockIdx.x;
    if (threadIdx.x == 0) {
        cnt[qi] = 0;
        if (qi == 0) *n_again = 0;
    }
    if (nq_dev && qi >= *nq_dev) return;  // whole block
    auto key = [&](uint32_t i) { return minima[(uint64_t)i * nq + qi] >> 5; };
    auto row = [&](uint32_t i) {  // of group i = (tile i / 2, lane half i % 2), as scan_mfma_kernel's lanes hold them
        const uint32_t e = minima[(uint64_t)i * nq + qi] & 31;
        const uint32_t slot = 32 * (e >> 4) + 8 * ((e >> 2) & 3) + 4 * (i & 1) + (e & 3);
        return (uint32_t)sample_row(sample_entry(slot, sample_turn(slot, m / 2), i >> 1, m / 2), sample_step);
    };
    const u64 t = m <= 4 * kBlock ? Pick<4>(key, m, s_part).kth_key(k, row)
                                  : Pick<kMaxGroups / kBlock>(key, m, s_part).kth_key(k, row);
    if (threadIdx.x == 0) thr[qi] = t;
}

inline size_t al256(size_t b) { return (b + 255) / 256 * 256; }

}  // namespace

// Which batches take the matrix pass rather than the row scan (its 16-query
// matrix tiles; vector tiles for 1 and 2 queries).  The row scan needs two
// launches and no bounds, but expands every row once per 16 queries and keeps
// k-lists per wave, whose insertions grow with k; the matrix pass has six
// launches (about 30 us).  Measured, matrix pass / row scan, us per call among
// others:
//   k = 1, 17 queries: 30,000 rows 59 / 54, 66,000 59 / 62, 300,000 63 / 84;
//     33: 30,000 57 / 61, 66,000 58 / 70; 44: 16,800 61 / 56
//   k = 2, 17 queries: 8,192 rows 49 / 57, 66,000 60 / 74, 1M 139 / 182;
//     12: 30,000 1.17 times the row scan, 66,000 1.03, 1M 1.07
//   k = 10, 8 queries: 8,192 to 66,000 rows 0.8 to 1.0 times, 3M 0.97
//   few queries: 6 with k = 16 8,192 and 30,000 rows 1.17 and 1.11 times, 66,000
//     0.88, 1M 0.84, 3M 0.98, 10M 1.04; 4 with k = 24 66,000 0.99, 300,000 0.70,
//     10M 1.05; 3 with k = 48 66,000 1.05, 300,000 0.62, 10M 1.04
//   8,192 rows, 1,000 queries, k = 1 / 2 / 3: 0.80 / 0.75 / 0.63 times among others,
//     but 1.5 / 1.1 / 1.05 where each call is waited for (its allocation counts)
// So: from 17 queries up, for k < 4 from 2^14 rows (k = 1: 33 queries and 2^20
// pairs, or 2^18 rows), and fewer where nq k is 90, which small
// databases need 8 queries for and large ones, whose scan is one read of the
// rows either way, 144.  Below 8,192 rows (or 256 k) the sample would be most of
// the rows.
bool mfma_eligible(uint64_t n, uint32_t nq, uint32_t k) {
    if (n < 8192 || n < (uint64_t)k * 256) return false;
    if (nq >= 17) return k >= 4 || (n >= (1u << 14) && (k >= 2 || (nq >= 33 && n * nq >= (1u << 20)) || n >= (1u << 18)));
    if (nq >= 8) return nq * k >= 90;
    return nq >= 3 && n >= (1u << 16) && nq * k >= (n < (1u << 21) ? 90u : 144u);
}

// The layout of batches of nq queries each.
static MfmaLayout mfma_batch_layout(uint64_t n, uint32_t nq, uint32_t k) {
    MfmaLayout L;
    L.n = n;
    L.qb = nq;
    const uint64_t tiles = (n + kMidR - 1) / kMidR, n_qt = (nq + kMidQ - 1) / kMidQ;
    // The pass's first part ends where about 512 candidates per query are
    // expected from the sample's bounds (of up to kCap = 8,192 slots), each next one
    // eight times further (about 7 k more).  Sampling k n / r rows puts the
    // first end at 512 n / r: r = 4,096, an eighth of the rows, where that
    // eighth fills the chip several times over and there are candidates enough
    // to save (512 more per query cost about 0.1 us each query, a part of a
    // pass about 30 us), else the whole pass in one part.  At least 4 k groups
    // of 32 rows are sampled, so that k groups seldom share their nearest.
    // Where all near rows lie in the first part, it lists r of them on average;
    // for small k the sample's bound varies (k = 1: an exponential distribution,
    // 13% of the queries past 8,192), so a split pass samples as for k = 4.
    // A pass in one part samples as for k = 16 at least, up to 32,768 rows: that
    // many cost 10 us at most, and fewer candidates save more (64 queries, k = 4,
    // as for k / as for 16: 66,000 rows 118 / 67 us, 1M 189 / 149).
    const bool split = nq >= 512 && tiles / 8 * n_qt >= 8ull * kMidWaves * device_cus();
    const uint32_t ks = split ? std::max(k, 4u) : k;
    const uint64_t rows = std::max<uint64_t>({n / (split ? 4096 : 512) * ks, (uint64_t)k * 128,
                                              split ? 0 : std::min<uint64_t>(n / 512 * 16, 32768)});
    L.sample_tiles = std::min<uint64_t>({(rows + kMidR - 1) / kMidR, tiles, kMaxGroups / 2});
    L.sample_step = (n << 32) / (L.sample_tiles * kMidR);
    for (uint64_t end = L.sample_tiles * 512 / ks; 2 * end <= tiles; end *= 8) L.ends.push_back(end);
    L.ends.push_back(tiles);
    // Slots: of a pass in one part, as many as a query overflows once in some ten
    // million times.  Its candidates are those before its k-th sampled row; k n /
    // sample of them are expected (a quarter more, as some sampled rows share a
    // group), and the number's spread falls with k.  8,192 slots for every batch
    // made a workspace whose allocation alone took up to 0.2 ms (1,000 queries x
    // 8,192 rows, k = 4: 0.39 ms a call, 0.16 with the row scan); from 2 MB on an
    // allocation after a wait takes 0.1 ms.
    L.cap = kCap;
    if (L.ends.size() == 1) {
        const double many = 1.25 * (double)k * (double)n / (double)(L.sample_tiles * kMidR);
        const double most = many * (1 + 5.2 / sqrt((double)k) + 9.0 / k);
        L.cap = std::min<uint32_t>(kCap, ((uint32_t)most / kBlock + 1) * kBlock);
    }
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t at = o;
        o += al256(b);
        return at;
    };
    L.minima = take((size_t)L.sample_tiles * 2 * nq * 4);
    L.thr = take((size_t)nq * 8);
    L.cnt = take((size_t)nq * 4);
    L.cand = take((size_t)nq * L.cap * 8);
    L.again = take((size_t)nq * 4);
    L.n_again = take(4);
    L.bytes = o;
    return L;
}

MfmaLayout mfma_layout(uint64_t n, uint32_t nq, uint32_t k) {
    const MfmaLayout L = mfma_batch_layout(n, nq, k);
    const uint64_t most = std::max<uint64_t>(kMinBatch, kBatchBytes / (L.bytes / nq + 1));
    if (nq <= most) return L;
    // batches of one size, whole groups of queries
    const uint64_t batches = (nq + most - 1) / most, each = (nq + batches - 1) / batches;
    return mfma_batch_layout(n, (uint32_t)((each + kGroupQ - 1) / kGroupQ * kGroupQ), k);
}

int mfma_run(const MfmaLayout &L, char *ws, const uint64_t *d_db, const uint64_t *d_q, uint32_t nq,
             const uint32_t *nq_dev, uint32_t k, uint32_t *d_idx, int32_t *d_missed, int32_t *d_extra, float *d_dist,
             hipStream_t s) {
    const uint64_t n = L.n, n_qt = (nq + kMidQ - 1) / kMidQ;
    u64 *thr = (u64 *)(ws + L.thr), *cand = (u64 *)(ws + L.cand);
    uint32_t *minima = (uint32_t *)(ws + L.minima), *cnt = (uint32_t *)(ws + L.cnt),
             *again = (uint32_t *)(ws + L.again), *n_again = (uint32_t *)(ws + L.n_again);
    const uint4 *db4 = reinterpret_cast<const uint4 *>(d_db), *q4 = reinterpret_cast<const uint4 *>(d_q);
    const size_t lds = mid_lds_bytes(nq);
    // one workgroup per CU (registers), fewer when there are fewer units
    auto grid = [&](uint64_t row_tiles) {
        return dim3((uint32_t)std::min<uint64_t>((row_tiles * n_qt + kMidWaves - 1) / kMidWaves, device_cus()));
    };
    {
        KernelTimer timer("wh_scan_mfma_sample", s);
        // (a small sample one unit per workgroup: its scattered rows are a chain of misses)
        const dim3 g((uint32_t)std::min<uint64_t>(L.sample_tiles * n_qt, device_cus()));
        hipLaunchKernelGGL(scan_mfma_kernel<kSample>, g, dim3(kMidBlock), lds, s, db4, n, 0ull, L.sample_tiles,
                           L.sample_step, q4, nq, nullptr, nullptr, nullptr, L.cap, minima, nullptr, nq_dev);
        hipLaunchKernelGGL(sample_threshold_kernel, dim3(nq), dim3(kBlock), 0, s, minima,
                           (uint32_t)(2 * L.sample_tiles), L.sample_step, nq, k, thr, cnt, n_again, nq_dev);
    }
    {
        KernelTimer timer("wh_scan_mfma", s);
        for (size_t i = 0; i < L.ends.size(); i++) {
            const uint64_t t0 = i ? L.ends[i - 1] : 0, nt = L.ends[i] - t0;
            if (i)
                hipLaunchKernelGGL(tighten_kernel, dim3(nq), dim3(kBlock), 0, s, cnt, cand, L.cap, k, thr,
                                   nq_dev);
            hipLaunchKernelGGL(scan_mfma_kernel<kFirst>, grid(nt), dim3(kMidBlock), lds, s, db4, n, t0, nt, 0ull, q4,
                               nq, thr, cnt, cand, L.cap, nullptr, nullptr, nq_dev);
        }
    }
    {
        KernelTimer timer("topk_select", s);
        hipLaunchKernelGGL(select_emit_kernel, dim3(nq), dim3(kBlock), 0, s, cnt, cand, L.cap, k, q4, db4, d_idx,
                           d_missed, d_extra, d_dist, thr, again, n_again, nq_dev);
    }
    // the overflowed queries, whose list and count stay on the device: without
    // any these launches find no work
    hipLaunchKernelGGL(scan_mfma_kernel<kAgain>, grid(L.ends.back()), dim3(kMidBlock), lds, s, db4, n, 0ull,
                       L.ends.back(), 0ull, q4, nq, thr, cnt, cand, L.cap, nullptr, again, n_again);
    hipLaunchKernelGGL(select_again_kernel, dim3(std::min<uint32_t>(nq, device_cus())), dim3(kBlock), 0, s, cnt, cand,
                       L.cap, k, q4, db4, n, d_idx, d_missed, d_extra, d_dist, thr, again, n_again);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? QD_OK : fail(QD_ERR_DEVICE, "matrix-core scan: %s", hipGetErrorString(e));
}

// Matrix-core path for large batches; returns QD_ERR_UNSUPPORTED when the
// shape is not worth it or its workspace cannot be had (the caller then uses the
// row scan, which needs a few MB).
int knn_bruteforce_mfma(const uint64_t *d_db, uint64_t n, const uint64_t *d_q, uint32_t nq, uint32_t k,
                        uint32_t *d_idx, int32_t *d_missed, int32_t *d_extra, float *d_dist, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    if (!mfma_eligible(n, nq, k)) return QD_ERR_UNSUPPORTED;
    const MfmaLayout L = mfma_layout(n, nq, k);
    char *ws = nullptr;
    if (hipMallocAsync((void **)&ws, L.bytes, s) != hipSuccess) {
        (void)hipGetLastError();
        return QD_ERR_UNSUPPORTED;
    }
    int rc = QD_OK;
    for (uint64_t b = 0; b < nq && rc == QD_OK; b += L.qb) {
        const uint64_t o = b * k;
        rc = mfma_run(L, ws, d_db, d_q + b * QD_WORDS, (uint32_t)std::min<uint64_t>(L.qb, nq - b), nullptr, k, d_idx + o,
                      d_missed + o, d_extra + o, d_dist + o, s);
    }
    (void)hipFreeAsync(ws, s);
    return rc;
}

}  // namespace qd
