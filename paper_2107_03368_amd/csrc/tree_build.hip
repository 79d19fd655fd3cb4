// Dissimilarity Tree construction on the GPU (Section 4.1, Listing 1).
//
// The paper's split of a node takes bit positions in ascending popularity
// (ties: ascending bit index) and moves every descriptor still in the similar
// set that has the bit set, stopping once the dissimilar set holds at least
// half of the node and never applying a move that would empty the similar
// set.  A descriptor therefore leaves with the first processed bit it has
// set: its least popular set bit, fr(t) = the set bit b minimising the key
// (popularity(b), b).  With the keys of all members known, the loop collapses
// to a cut on that key:
//   x* = the ceil(n/2)-th smallest member key (zero rows have no key and
//        sort last);
//   D  = {t : key(t) <= x*}, unless that is the whole node, then
//   D  = {t : key(t) <  x*};
//   if every member's key is absent or fewer than ceil(n/2) rows are nonzero,
//   D = the nonzero rows.
// The tree is built level by level.  Each node is a segment of a permutation
// of the rows; a split writes the similar rows, then the dissimilar rows, each
// in their previous order (a stable partition), so the layout matches a
// breadth-first numbering with the similar child first.  Nodes of at most
// kSmall rows are split by one block each; larger nodes use a multi-block path
// with global counters.  Sum (OR) and product (AND) images
// are then formed for every node, leaves from their rows and inner nodes from
// their children, deepest level first.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <vector>

#include "band_weight.h"
#include "qd_device.h"
#include "qd_internal.h"
#include "qd_tree.h"

namespace qd {
namespace {

constexpr int kBlock = 256;
// Which kernel splits a node.  One block per node up to kSmall rows: its
// threads share one set of counters, and a level of such nodes is one launch;
// several blocks per node take eight launches (some 50 us of a level's time even
// for a few nodes).  Above kMid the block has 512 threads, because a million
// rows are then only 500 to 2,000 blocks (1,950-row nodes: 0.46 ms per million
// rows, 0.71 with 256 threads).  Up to kKept rows they stay in registers
// between the two passes over them, which the register file allows for 16 rows
// per half-wave.
constexpr uint32_t kSmall = 2048;
constexpr uint32_t kMid = 512;
constexpr uint32_t kKept = 128;
constexpr uint32_t kChunk = 1024;  // rows per work item of a large node
// Counts of masked bits per member (see "the least popular set bit"): enough to
// reach half the members at the first try nearly always.  A million generated
// rows need up to 20 at the first levels (with 24, those took the second try),
// fewer in smaller nodes.
constexpr uint32_t kLambdaKept = 6, kLambdaSmall = 12, kLambdaBig = 64;
constexpr uint16_t kNoRank = 0xFFFF;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;

// ---- counting set bits by column ----
//
// Half-waves read whole rows: lane c of a half-wave holds dwords 4c .. 4c+3
// of its row (16 bytes), so a lane meets the same 128 bit positions in every
// row and counts them bit-sliced: plane k of a dword holds bit k of its 32
// counts, and eight rows enter through seven full adders.  That is about 3
// operations per row and dword, whatever the rows' density: 0.095 ms per
// million rows, 5.4 TB/s.  One LDS atomic per set bit (some 280 per row of the
// generator's databases) took 0.40 ms.

__device__ __forceinline__ void full_add(uint32_t a, uint32_t b, uint32_t c, uint32_t &sum, uint32_t &carry) {
    sum = a ^ b ^ c;
    carry = (a & b) | (a & c) | (b & c);
}

__device__ __forceinline__ uint32_t dword_of(const uint4 &v, int d) {
    return d == 0 ? v.x : d == 1 ? v.y : d == 2 ? v.z : v.w;
}

// Add 8 rows to the bit-sliced counts of the lane's four dwords (P planes: up
// to 2^P - 1 rows).
template <int P>
__device__ __forceinline__ void planes_add8(uint32_t (&p)[4][P], const uint4 (&v)[8]) {
#pragma unroll
    for (int d = 0; d < 4; d++) {
        uint32_t s1, s2, s3, c1, c2, c3, c4, t, d1, d2, e;
        full_add(dword_of(v[0], d), dword_of(v[1], d), dword_of(v[2], d), s1, c1);
        full_add(dword_of(v[3], d), dword_of(v[4], d), dword_of(v[5], d), s2, c2);
        full_add(dword_of(v[6], d), dword_of(v[7], d), p[d][0], s3, c3);
        full_add(s1, s2, s3, p[d][0], c4);
        full_add(c1, c2, c3, t, d1);
        full_add(t, c4, p[d][1], p[d][1], d2);
        full_add(d1, d2, p[d][2], p[d][2], e);
#pragma unroll
        for (int k = 3; k < P; k++) {
            const uint32_t o = p[d][k] & e;
            p[d][k] ^= e;
            e = o;
        }
    }
}

// a += b, both bit-sliced with P planes; the sum has P + 1.
template <int P>
__device__ __forceinline__ void planes_sum(const uint32_t (&a)[P], const uint32_t (&b)[P], uint32_t (&o)[P + 1]) {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < P; k++) full_add(a[k], b[k], c, o[k], c);
    o[P] = c;
}

// Load the rows the half-wave `hw` of `kHalves` owns in batch b (members
// (8b + i) * kHalves + hw, i = 0 .. 7).  The batch's last members past m repeat
// member m - 1, so the loads are unconditional and all in flight together.
template <uint32_t kHalves>
__device__ __forceinline__ void load_rows8(const uint4 *__restrict__ db, const uint32_t *rows, uint32_t m, uint32_t b,
                                           uint32_t hw, uint32_t c, uint4 (&v)[8]) {
    uint32_t row[8];
#pragma unroll
    for (uint32_t i = 0; i < 8; i++) row[i] = rows[min((8 * b + i) * kHalves + hw, m - 1)];
#pragma unroll
    for (uint32_t i = 0; i < 8; i++) v[i] = db[(uint64_t)row[i] * 32 + c];
}

// f(rows, b) for every batch of m rows; the next batch's rows are loaded while
// f works on this one.
template <uint32_t kHalves, class F>
__device__ __forceinline__ void each_batch(const uint4 *__restrict__ db, const uint32_t *rows, uint32_t m, uint32_t hw,
                                           uint32_t c, F f) {
    const uint32_t batches = (m + 8 * kHalves - 1) / (8 * kHalves);
    uint4 v[8], u[8];
    load_rows8<kHalves>(db, rows, m, 0, hw, c, v);
    for (uint32_t b = 0; b < batches; b += 2) {
        if (b + 1 < batches) load_rows8<kHalves>(db, rows, m, b + 1, hw, c, u);
        f(v, b);
        if (b + 1 >= batches) break;
        if (b + 2 < batches) load_rows8<kHalves>(db, rows, m, b + 2, hw, c, v);
        f(u, b + 1);
    }
}

// Clear those of the batch's rows that only repeat member m - 1.
template <uint32_t kHalves>
__device__ __forceinline__ void clear_past(uint32_t m, uint32_t b, uint32_t hw, uint4 (&v)[8]) {
    if ((8 * b + 8) * kHalves <= m) return;  // uniform
#pragma unroll
    for (uint32_t i = 0; i < 8; i++) {
        const bool in = (8 * b + i) * kHalves + hw < m;
        v[i] = make_uint4(in ? v[i].x : 0, in ? v[i].y : 0, in ? v[i].z : 0, in ? v[i].w : 0);
    }
}

// Sum the half-waves' planes over the block: thread t of kWaves * 64 gets the
// counts of its 4096 / (kWaves * 64) consecutive bit positions.  The two
// halves of a wave add by swapping (each half then holds two of the four
// dwords' sums), the waves through `buf` (kWaves x (P + 1) x 128 words).
template <int kWaves, int P, int kCols>
__device__ __forceinline__ void column_counts(uint32_t (&p)[4][P], uint32_t *buf, uint32_t (&cnt)[kCols]) {
    static_assert(kCols * kWaves * 64 == QD_BITS && (kCols == 16 || kCols == 8), "columns per thread");
    const uint32_t t = threadIdx.x, w = t >> 6, lane = t & 63;
#pragma unroll
    for (int h = 0; h < 4; h += 2) {
        uint32_t a[P], b[P], o[P + 1];
#pragma unroll
        for (int k = 0; k < P; k++) {
            // lanes 0-31: dword h of both halves; lanes 32-63: dword h + 1
            const auto r = __builtin_amdgcn_permlane32_swap(p[h][k], p[h + 1][k], false, false);
            a[k] = r[0];
            b[k] = r[1];
        }
        planes_sum<P>(a, b, o);
#pragma unroll
        for (int k = 0; k <= P; k++) buf[(w * (P + 1) + k) * 128 + 4 * (lane & 31) + h + (lane >> 5)] = o[k];
    }
    __syncthreads();
    constexpr int kPer = 32 / kCols;  // threads per dword
    constexpr int L = kWaves == 4 ? 2 : 3;
    uint32_t pl[P + 1 + L];
    {
        const uint32_t dw = t / kPer;
        uint32_t s[kWaves][P + 1];
#pragma unroll
        for (int x = 0; x < kWaves; x++)
#pragma unroll
            for (int k = 0; k <= P; k++) s[x][k] = buf[(x * (P + 1) + k) * 128 + dw];
        uint32_t s2[kWaves / 2][P + 2];
#pragma unroll
        for (int x = 0; x < kWaves / 2; x++) planes_sum<P + 1>(s[2 * x], s[2 * x + 1], s2[x]);
        if constexpr (kWaves == 4) {
            planes_sum<P + 2>(s2[0], s2[1], pl);
        } else {
            uint32_t s3[2][P + 3];
#pragma unroll
            for (int x = 0; x < 2; x++) planes_sum<P + 2>(s2[2 * x], s2[2 * x + 1], s3[x]);
            planes_sum<P + 3>(s3[0], s3[1], pl);
        }
    }
    const uint32_t sh = kCols * (t % kPer);
#pragma unroll
    for (int k = 0; k < P + 1 + L; k++) pl[k] >>= sh;
#pragma unroll
    for (int i = 0; i < kCols; i++) {
        uint32_t v = 0;
#pragma unroll
        for (int k = P + L; k >= 0; k--) v = (v << 1) | ((pl[k] >> i) & 1u);
        cnt[i] = v;
    }
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    v = sum8(v);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row_mirror: 16 lanes
    return readlane(v, 0) + readlane(v, 16) + readlane(v, 32) + readlane(v, 48);
}

// Smallest over each 32-lane half of the wave; every lane gets its half's.
__device__ __forceinline__ uint32_t min32_half(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false));
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false));
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false));
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false));
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return min((uint32_t)r[0], (uint32_t)r[1]);
}

// ---- the least popular set bit ----
//
// Only the members up to the cut matter, and those leave with one of the
// least popular bits.  So a row's set bits are first cut to a mask of the least
// popular positions, taken so wide that their counts add to several times the
// members (the generator's databases need 2 to 20 per member to reach half the
// node, of 280 set bits).  The masked positions form bands of the popularity
// order, stored as bit planes, and a row's least band falls out of a few
// AND / select steps without a loop over its bits.  The band that the half-th
// member falls into is the only one whose members need an exact key, a small
// share of the rows.  If the masked bits reach fewer than half the members, the
// split repeats with all bits.  Looking up every set bit's count took 0.59 ms
// per million rows of large nodes; the band pass takes 0.11 (4.6 TB/s) and the
// exact keys 0.03 to 0.05.

// Smallest c in 1 .. m such that the counts of at most c add to `want` or
// more (m if none does).  kCoarse: among 1, 2, 3, 4, 6, 8, 12, .. only, which
// halves the steps.  S: the type that holds the sum of all counts.  sums:
// 2 * kWaves words.
template <int kWaves, bool kCoarse, class S, int kCols>
__device__ __forceinline__ uint32_t count_threshold(const uint32_t (&cnt)[kCols], uint32_t m, S want, S *sums) {
    auto value = [&](uint32_t e) -> uint32_t {
        if (!kCoarse) return e + 1;
        return min(m, e == 0 ? 1u : (e & 1) ? 2u << (e / 2) : 3u << (e / 2 - 1));
    };
    uint32_t lo = 0, hi = kCoarse ? 2 * (32 - (uint32_t)__builtin_clz(m)) : m - 1, it = 0;
    while (lo < hi) {  // uniform in the block
        const uint32_t mid = lo + (hi - lo) / 2, c = value(mid);
        uint32_t x = 0;
#pragma unroll
        for (int i = 0; i < kCols; i++) x += cnt[i] <= c ? cnt[i] : 0u;
        // up to 16 counts of 2^27 rows fit 32 bits, a wave's 64 sums need more
        const S s = sizeof(S) == 4 ? (S)wave_sum(x) : (S)wave_sum(x & 0xFFFFu) + ((S)wave_sum(x >> 16) << 16);
        S *b = sums + (it++ & 1) * kWaves;
        if ((threadIdx.x & 63) == 0) b[threadIdx.x >> 6] = s;
        __syncthreads();
        S total = 0;
#pragma unroll
        for (int y = 0; y < kWaves; y++) total += b[y];
        if (total >= want)
            hi = mid;
        else
            lo = mid + 1;
    }
    __syncthreads();
    return value(lo);
}

// The lane's set bits of x (its 128 positions, first position `base`) one at
// a time, from the lowest.
template <class F>
__device__ __forceinline__ void each_bit(uint4 x, uint32_t base, F f) {
    while (x.x | x.y | x.z | x.w) {
        const uint32_t w = x.x ? x.x : x.y ? x.y : x.z ? x.z : x.w;
        const uint32_t d = x.x ? 0u : x.y ? 32u : x.z ? 64u : 96u;
        f(base + d + (uint32_t)__builtin_ctz(w));
        const uint32_t r = w & (w - 1);
        if (x.x)
            x.x = r;
        else if (x.y)
            x.y = r;
        else if (x.z)
            x.z = r;
        else
            x.w = r;
    }
}

__device__ __forceinline__ uint4 and4(const uint4 &a, const uint4 &b) {
    return make_uint4(a.x & b.x, a.y & b.y, a.z & b.z, a.w & b.w);
}

// Bands are runs of the popularity order.  Plane k of `band` holds bit k of
// every position's band; x: the lane's set bits among the masked ones.  The
// least band of the half-wave's row (kNoBand without a bit), in every lane.
constexpr uint32_t kNoBand = 0xFF;
template <int B>
__device__ __forceinline__ uint32_t least_band(uint4 x, const uint4 (&band)[B]) {
    if (ballot((x.x | x.y | x.z | x.w) != 0) == 0) return kNoBand;  // neither of the wave's rows
    uint32_t v = (x.x | x.y | x.z | x.w) ? 0u : kNoBand;
#pragma unroll
    for (int k = B - 1; k >= 0; k--) {
        const uint4 y = make_uint4(x.x & ~band[k].x, x.y & ~band[k].y, x.z & ~band[k].z, x.w & ~band[k].w);
        const bool any = (y.x | y.y | y.z | y.w) != 0;
        v |= any ? 0u : 1u << k;
        if (k) x = make_uint4(any ? y.x : x.x, any ? y.y : x.y, any ? y.z : x.z, any ? y.w : x.w);
    }
    return min32_half(v);
}

// The positions of band b, among the masked ones.
template <int B>
__device__ __forceinline__ uint4 band_mask(uint4 mask, const uint4 (&band)[B], uint32_t b) {
#pragma unroll
    for (int k = 0; k < B; k++) {
        const uint32_t f = (b >> k) & 1 ? 0u : ~0u;
        mask = make_uint4(mask.x & (band[k].x ^ f), mask.y & (band[k].y ^ f), mask.z & (band[k].z ^ f),
                          mask.w & (band[k].w ^ f));
    }
    return mask;
}

// The band that holds the half-th member, from the bands' member counts
// (n_bands if the banded members are fewer); lower: members of bands below it.
__device__ __forceinline__ uint32_t cut_band(const uint32_t *hist, uint32_t n_bands, uint32_t half, uint32_t *lower) {
    uint32_t run = 0, b = 0;
    for (; b < n_bands && run + hist[b] < half; b++) run += hist[b];
    *lower = run;
    return b;
}

// One block splits one node of at most kRows rows.
//
// kKeep: 16 rows per half-wave, read once and held in registers; otherwise the
// rows are read twice.  Members' keys are (count << 12 | bit), below 2^24.
// Bound by instruction issue and by the chain of short steps between barriers
// (counts, threshold, bands, keys, cut), not by memory: a million rows in nodes
// of about 1,950 / 490 / 61 rows take 0.46 / 0.28 / 0.30 ms (1.2 to 2.6 ms with
// an atomic and a lookup per set bit).
template <int kWaves, uint32_t kRows, bool kKeep>
__global__ __launch_bounds__(64 * kWaves, 4) void split_small_kernel(const uint4 *__restrict__ db,
                                                                     const uint32_t *__restrict__ perm_in,
                                                                     uint32_t *__restrict__ perm_out,
                                                                     const uint64_t *__restrict__ nbegin,
                                                                     const uint32_t *__restrict__ ncount,
                                                                     uint32_t *__restrict__ nd_out) {
    constexpr uint32_t T = 64 * kWaves, kHalves = 2 * kWaves;
    constexpr int P = 32 - __builtin_clz(kRows / kHalves);  // a half-wave counts kRows / kHalves rows
    static_assert(!kKeep || kRows == 16 * kHalves, "rows in registers");
    constexpr int kCols = QD_BITS / T;
    constexpr uint32_t kPerThread = (kRows + T - 1) / T;
    constexpr int B = kKeep ? 3 : 4;  // 8 or 16 bands of counts
    __shared__ uint32_t rows[kRows];
    union Shared {
        uint32_t planes[kWaves * (P + 1) * 128];
        struct {
            uint16_t cnt[QD_BITS];
            uint32_t key[kRows];  // a member's band, then its key
            uint32_t mask[B + 1][QD_BITS / 32];  // looked up; then the planes of their bands
        } f;
    };
    __shared__ __attribute__((aligned(16))) Shared sh;
    __shared__ uint32_t sums[2 * kWaves];
    __shared__ uint32_t tally[kPerThread * kWaves], result[3], hist[1 << B];
    __shared__ uint16_t listed[kRows];
    const uint64_t begin = nbegin[blockIdx.x];
    const uint32_t m = ncount[blockIdx.x];
    const uint32_t t = threadIdx.x, w = t >> 6, lane = t & 63, c = t & 31, hw = t >> 5;
    if (m > kRows) return;  // whole block; the host sends no such node
    for (uint32_t r = t; r < m; r += T) rows[r] = perm_in[begin + r];
    __syncthreads();
    const uint32_t batches = (m + 8 * kHalves - 1) / (8 * kHalves);
    uint4 keep[kKeep ? 2 : 1][8];
    uint32_t cnt[kCols];
    {
        uint32_t p[4][P] = {};
        if constexpr (kKeep) {
            load_rows8<kHalves>(db, rows, m, 0, hw, c, keep[0]);
            if (batches > 1) load_rows8<kHalves>(db, rows, m, 1, hw, c, keep[1]);
            clear_past<kHalves>(m, 0, hw, keep[0]);
            planes_add8<P>(p, keep[0]);
            if (batches > 1) {
                clear_past<kHalves>(m, 1, hw, keep[1]);
                planes_add8<P>(p, keep[1]);
            }
        } else {
            each_batch<kHalves>(db, rows, m, hw, c, [&](uint4(&v)[8], uint32_t b) {
                clear_past<kHalves>(m, b, hw, v);
                planes_add8<P>(p, v);
            });
        }
        column_counts<kWaves, P, kCols>(p, sh.planes, cnt);
    }
    __syncthreads();  // the planes' words are written over
#pragma unroll
    for (int i = 0; i < kCols; i += 2)
        *reinterpret_cast<uint32_t *>(&sh.f.cnt[kCols * t + i]) = cnt[i] | (cnt[i + 1] << 16);
    const uint32_t half = (m + 1) / 2;
    uint32_t cut = 0, nd = 0;
    for (int attempt = 0; attempt < 2; attempt++) {
        const uint32_t cmax =
            attempt ? m
                    : count_threshold<kWaves, kKeep>(cnt, m, m * (kKeep ? kLambdaKept : kLambdaSmall), sums);
        {
            // bands of equal width over counts 1 .. cmax
            const uint32_t wide = 32 - (uint32_t)__builtin_clz(cmax), shift = wide > B ? wide - B : 0;
            uint32_t bits[B + 1] = {};
#pragma unroll
            for (int i = 0; i < kCols; i++) {
                bits[0] |= (cnt[i] <= cmax ? 1u : 0u) << i;
#pragma unroll
                for (int k = 0; k < B; k++) bits[k + 1] |= ((cnt[i] >> (shift + k)) & 1u) << i;
            }
#pragma unroll
            for (int k = 0; k <= B; k++)
                if constexpr (kCols == 16)
                    reinterpret_cast<uint16_t *>(sh.f.mask[k])[t] = (uint16_t)bits[k];
                else
                    reinterpret_cast<uint8_t *>(sh.f.mask[k])[t] = (uint8_t)bits[k];
        }
        __syncthreads();
        const uint4 mask = reinterpret_cast<const uint4 *>(sh.f.mask[0])[c];
        uint4 band[B];
#pragma unroll
        for (int k = 0; k < B; k++) band[k] = reinterpret_cast<const uint4 *>(sh.f.mask[k + 1])[c];
        if (t < (1u << B)) hist[t] = 0;
        // every member's band
        auto find_bands = [&](const uint4(&v)[8], uint32_t b) {
#pragma unroll
            for (uint32_t i = 0; i < 8; i++) {
                const uint32_t r = (8 * b + i) * kHalves + hw;
                const uint32_t best = least_band<B>(and4(v[i], mask), band);
                if (c == 0 && r < m) sh.f.key[r] = best;
            }
        };
        if constexpr (kKeep) {
            find_bands(keep[0], 0);
            if (batches > 1) find_bands(keep[1], 1);
        } else {
            each_batch<kHalves>(db, rows, m, hw, c, find_bands);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kPerThread; i++) {
            const uint32_t r = i * T + t;
            if (r < m && sh.f.key[r] != kNoBand) atomicAdd(&hist[sh.f.key[r]], 1u);
        }
        __syncthreads();
        // the band of the half-th member; only its members' keys are looked up
        uint32_t lower;
        const uint32_t cb = cut_band(hist, 1u << B, half, &lower);
        const uint4 cmask = band_mask<B>(mask, band, cb);
        // list them, then look up two per wave (their rows come from a cache)
        if (t == 0) result[0] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kPerThread; i++) {
            const uint32_t r = i * T + t;
            const uint32_t rb = r < m ? sh.f.key[r] : kNoBand;
            if (r < m) sh.f.key[r] = rb < cb ? 0u : kNoKey;
            const u64 in = ballot(r < m && rb == cb);
            uint32_t at = 0;
            if (lane == 0 && in) at = atomicAdd(&result[0], (uint32_t)__popcll(in));
            at = readfirst(at) + lanes_below(in);
            if ((in >> lane) & 1) listed[at] = (uint16_t)r;
        }
        __syncthreads();
        const uint32_t n_listed = result[0];
        for (uint32_t i = hw; (i & ~1u) < n_listed; i += kHalves) {  // a wave's halves together
            const uint32_t r = listed[min(i, n_listed - 1)];
            uint32_t best = kNoKey;
            each_bit(and4(db[(uint64_t)rows[r] * 32 + c], cmask), 128 * c, [&](uint32_t bit) {
                best = min(best, ((uint32_t)sh.f.cnt[bit] << 12) | bit);
            });
            best = min32_half(best);
            if (c == 0) sh.f.key[r] = best;
        }
        __syncthreads();
        // x* = the half-th smallest key: the smallest x with half the keys at
        // or below it, from its top bit down
        constexpr int kSelect = kKeep ? 1 : kWaves;  // waves that hold the keys
        if (w < kSelect) {
            constexpr uint32_t kPer = kRows / (64 * kSelect);
            uint32_t key[kPer], it = 0;
#pragma unroll
            for (uint32_t i = 0; i < kPer; i++) {
                const uint32_t r = i * (64 * kSelect) + t;
                key[i] = r < m ? sh.f.key[r] : kNoKey;
            }
            auto at_most = [&](uint32_t x) {  // keys <= x in the block
                uint32_t s = 0;
#pragma unroll
                for (uint32_t i = 0; i < kPer; i++)
                    if (i * 64 * kSelect < m) s += (uint32_t)__popcll(ballot(key[i] <= x));
                if constexpr (kSelect == 1) return s;
                uint32_t *b = sums + (it++ & 1) * kWaves;
                if (lane == 0) b[w] = s;
                __syncthreads();
                uint32_t total = 0;
#pragma unroll
                for (int y = 0; y < kWaves; y++) total += b[y];
                return total;
            };
            // with every bit looked up and fewer than half reached: D = the nonzero rows
            uint32_t x = kNoKey - 1, below = at_most(x);
            const bool redo = below < half && cmax < m;
            if (below >= half) {
                x = 0;
                for (int bit = 31 - __builtin_clz((cmax << 12) | 0xFFFu); bit >= 0; bit--)
                    if (at_most(x | ((1u << bit) - 1)) < half) x |= 1u << bit;
                below = at_most(x);
                if (below == m) below = at_most(--x);  // the whole node: D = the keys below x*
            }
            if (t == 0) {
                result[0] = redo;
                result[1] = x;
                result[2] = below;
            }
        }
        __syncthreads();
        cut = result[1];
        nd = result[2];
        if (!result[0]) break;
        __syncthreads();  // the second try writes over the masks and the result
    }
    // stable partition: similar members first, each side in its order
    u64 dm[kPerThread];
#pragma unroll
    for (uint32_t i = 0; i < kPerThread; i++) {
        const uint32_t r = i * T + t;
        dm[i] = ballot(r < m && nd != 0 && sh.f.key[r] <= cut);
        if (lane == 0 && i * T < m) tally[i * kWaves + w] = (uint32_t)__popcll(dm[i]);
    }
    __syncthreads();
    const uint32_t ns = m - nd;
    uint32_t before = 0, g = 0;  // dissimilar members in the groups of 64 before this one
#pragma unroll
    for (uint32_t i = 0; i < kPerThread; i++) {
        if (i * T >= m) break;
        for (; g < i * kWaves + w; g++) before += tally[g];
        const uint32_t r = i * T + t;
        if (r < m) {
            const uint32_t d = before + lanes_below(dm[i]);
            perm_out[begin + ((dm[i] >> lane) & 1 ? ns + d : r - d)] = rows[r];
        }
    }
    if (t == 0) nd_out[blockIdx.x] = nd;
}

// ---- large nodes: work items are (node slot, row range) chunks ----

struct Item {
    uint32_t slot;  // index among the level's large nodes
    uint32_t first; // first member (relative to node begin)
    uint32_t count; // members in this chunk
    uint32_t pad;
};

// A large node's split, as its kernels leave it for the next ones.  A
// member's code (fr_pos): its band; then 0 if it is below the cut band, 1 + its
// least bit's rank in the cut band, or kNoRank.
struct BigCut {
    uint32_t limit;  // D = the members of a code below it
    uint32_t band;   // the cut band
    uint32_t nb;     // bits of the cut band
    uint32_t lower;  // members of lower bands
    uint32_t redo;   // the banded bits reach fewer than half the members
    uint32_t all;    // 1: every bit is banded; 2: in the second try
};

// Where a large node's counts come from.  Of a large parent's children only the
// one of fewer rows is counted; the other's counts are the parent's less those
// (1M rows: 0.51 ms for the counts of all levels, 0.92 when every large node was
// counted).
struct CountSource {
    uint32_t job;     // counted node, among the level's counted ones
    uint32_t parent;  // kNoKey: the job counted this node; else its parent's slot, one level up
};

// A node's counts are stored by (bit % 16, bit / 16): thread t of a block
// owns bits 16t .. 16t + 15 and its accesses stay consecutive over t.
__device__ __forceinline__ uint32_t count_at(uint32_t t, uint32_t i) { return i * kBlock + t; }

__global__ __launch_bounds__(kBlock) void big_count_kernel(const uint4 *__restrict__ db,
                                                           const uint32_t *__restrict__ perm_in,
                                                           const uint64_t *__restrict__ nbegin,
                                                           const Item *__restrict__ items,
                                                           uint32_t *__restrict__ gcnt) {
    constexpr int P = 8;  // a half-wave counts kChunk / 8 = 128 rows
    static_assert(kChunk / 8 < (1u << P), "planes");
    __shared__ uint32_t rows[kChunk];
    __shared__ uint32_t planes[4 * (P + 1) * 128];
    const Item it = items[blockIdx.x];
    const uint64_t begin = nbegin[it.slot] + it.first;
    const uint32_t m = it.count, t = threadIdx.x;
    for (uint32_t r = t; r < m; r += kBlock) rows[r] = perm_in[begin + r];
    __syncthreads();
    uint32_t p[4][P] = {};
    for (uint32_t b = 0; b < (m + 63) / 64; b++) {
        uint4 v[8];
        load_rows8<8>(db, rows, m, b, t >> 5, t & 31, v);
        clear_past<8>(m, b, t >> 5, v);
        planes_add8<P>(p, v);
    }
    uint32_t cnt[16];
    column_counts<4, P, 16>(p, planes, cnt);
    uint32_t *g = gcnt + (uint64_t)it.slot * QD_BITS;
#pragma unroll
    for (int i = 0; i < 16; i++)
        if (cnt[i]) atomicAdd(&g[count_at(t, i)], cnt[i]);
}

constexpr int kBandPlanes = 5;  // 32 bands
constexpr uint32_t kBands = 1u << kBandPlanes;
constexpr uint32_t kMaskWords = (kBandPlanes + 1) * (QD_BITS / 32);  // a node's banded bits, then their bands' planes

// Band the least popular bits of a node by count: `lambda` times the members'
// worth of them, or all (lambda 0, the second try: only where the first fell
// short).  Also completes the node's counts.  The first half of the bands holds a quarter of the counts.  One block per large node,
// 1,024 threads because it is a chain of short steps.
__global__ __launch_bounds__(1024) void big_band_kernel(const CountSource *__restrict__ src,
                                                        const uint32_t *__restrict__ counted,
                                                        const uint32_t *__restrict__ above, uint32_t *__restrict__ gcnt,
                                                        const uint32_t *__restrict__ ncount, uint32_t lambda,
                                                        uint32_t *__restrict__ mask, uint32_t *__restrict__ bhist,
                                                        BigCut *__restrict__ cuts, uint32_t *__restrict__ any_redo) {
    constexpr uint32_t kBins = 256;
    __shared__ uint32_t bits[kBandPlanes + 1][QD_BITS / 32];
    __shared__ uint32_t bins[kBins];
    __shared__ u64 sums[32];
    const uint32_t slot = blockIdx.x, t = threadIdx.x, m = ncount[slot];
    if (!lambda && !cuts[slot].redo) return;  // whole block
    const CountSource from = src[slot];
    uint32_t cnt[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint32_t at = count_at(t & 255, 4 * (t >> 8) + i);
        cnt[i] = counted[(uint64_t)from.job * QD_BITS + at];
        if (from.parent != kNoKey) cnt[i] = above[(uint64_t)from.parent * QD_BITS + at] - cnt[i];
        gcnt[(uint64_t)slot * QD_BITS + at] = cnt[i];
    }
    if (lambda && slot == 0 && t == 0) *any_redo = 0;
    for (uint32_t i = t; i < kMaskWords; i += 1024) (&bits[0][0])[i] = 0;
    if (t < kBins) bins[t] = 0;
    const uint32_t cmax = lambda ? count_threshold<16, false>(cnt, m, (u64)m * lambda, sums) : m;
    __syncthreads();
    // counts in 256 bins of equal width; weights so that all together fit 32 bits
    const uint32_t wshift = band_weight_shift(m), shift = max(0, 24 - __builtin_clz(cmax));
#pragma unroll
    for (int i = 0; i < 4; i++)
        if (cnt[i] && cnt[i] <= cmax) atomicAdd(&bins[cnt[i] >> shift], (cnt[i] >> wshift) + 1);
    __syncthreads();
    if (t < 64) {  // a bin's band: half the bands for the first quarter of the weight
        uint32_t x[4], s = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            x[i] = bins[4 * t + i];
            s += x[i];
        }
        uint32_t run = s;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)run, o);
            if ((int)t >= o) run += y;
        }
        const uint32_t total = max(1u, readlane(run, 63));
        run -= s;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t f = (uint32_t)((u64)run * (4 * kBands / 2) / total);  // in 1/64 of the weight
            bins[4 * t + i] = f < kBands / 2 ? f : min(kBands - 1, kBands / 2 + (f - kBands / 2) / 3);
            run += x[i];
        }
    }
    __syncthreads();
    uint32_t mine[kBandPlanes + 1] = {};
#pragma unroll
    for (int i = 0; i < 4; i++)
        if (cnt[i] && cnt[i] <= cmax) {
            const uint32_t b = bins[cnt[i] >> shift];
            mine[0] |= 1u << i;
#pragma unroll
            for (int k = 0; k < kBandPlanes; k++) mine[k + 1] |= ((b >> k) & 1) << i;
        }
#pragma unroll
    for (int k = 0; k <= kBandPlanes; k++)  // bits 16 (t % 256) + 4 (t / 256) + i
        atomicOr(&bits[k][(t & 255) >> 1], mine[k] << (16 * (t & 1) + 4 * (t >> 8)));
    __syncthreads();
    for (uint32_t i = t; i < kMaskWords; i += 1024) mask[(uint64_t)slot * kMaskWords + i] = (&bits[0][0])[i];
    if (t < kBands) bhist[(uint64_t)slot * kBands + t] = 0;
    if (t == 0) cuts[slot] = {0, 0, 0, 0, 0, !lambda ? 2u : cmax >= m ? 1u : 0u};
}

// Each member's least band, and the node's histogram of them.
__global__ __launch_bounds__(kBlock) void big_first_kernel(const uint4 *__restrict__ db,
                                                           const uint32_t *__restrict__ perm_in,
                                                           const uint64_t *__restrict__ nbegin,
                                                           const Item *__restrict__ items,
                                                           const uint32_t *__restrict__ gmask,
                                                           const BigCut *__restrict__ cuts, uint32_t again,
                                                           uint16_t *__restrict__ fr_pos,
                                                           uint32_t *__restrict__ bhist) {
    __shared__ uint32_t rows[kChunk];
    __shared__ uint16_t first[kChunk];
    __shared__ uint32_t hist[kBands];
    const Item it = items[blockIdx.x];
    if (again && cuts[it.slot].all != 2) return;  // whole block: the first try stands
    const uint64_t begin = nbegin[it.slot] + it.first;
    const uint32_t m = it.count, t = threadIdx.x, c = t & 31, hw = t >> 5;
    for (uint32_t r = t; r < m; r += kBlock) rows[r] = perm_in[begin + r];
    if (t < kBands) hist[t] = 0;
    const uint4 *gm = reinterpret_cast<const uint4 *>(gmask + (uint64_t)it.slot * kMaskWords);
    const uint4 mask = gm[c];
    uint4 band[kBandPlanes];
#pragma unroll
    for (int k = 0; k < kBandPlanes; k++) band[k] = gm[32 * (k + 1) + c];
    __syncthreads();
    each_batch<8>(db, rows, m, hw, c, [&](const uint4(&x)[8], uint32_t b) {
#pragma unroll
        for (uint32_t i = 0; i < 8; i++) {
            const uint32_t r = (8 * b + i) * 8 + hw;
            const uint32_t best = least_band<kBandPlanes>(and4(x[i], mask), band);
            if (c == 0 && r < m) {
                first[r] = (uint16_t)best;
                if (best != kNoBand) atomicAdd(&hist[best], 1u);
            }
        }
    });
    __syncthreads();
    for (uint32_t r = t; r < m; r += kBlock) fr_pos[begin + r] = first[r];
    if (t < kBands && hist[t]) atomicAdd(&bhist[(uint64_t)it.slot * kBands + t], hist[t]);
}

// The cut band of a node, and its bits' ranks by (count, bit).  One block per
// large node; also clears the histogram of those ranks.
__global__ __launch_bounds__(1024) void big_rank_kernel(const uint32_t *__restrict__ gcnt,
                                                        const uint32_t *__restrict__ ncount,
                                                        const uint32_t *__restrict__ mask,
                                                        const uint32_t *__restrict__ bhist, uint32_t again,
                                                        uint16_t *__restrict__ rank, uint32_t *__restrict__ ghist,
                                                        BigCut *__restrict__ cuts, uint32_t *__restrict__ nd_out,
                                                        uint32_t *__restrict__ any_redo) {
    __shared__ u64 keys[QD_BITS];
    __shared__ uint32_t hist[kBands];
    __shared__ uint32_t counter;
    const uint32_t slot = blockIdx.x, t = threadIdx.x, m = ncount[slot], half = (m + 1) / 2;
    const uint32_t all = cuts[slot].all;
    if (again && all != 2) return;  // whole block
    if (t < kBands) hist[t] = bhist[(uint64_t)slot * kBands + t];
    if (t == 0) counter = 0;
    __syncthreads();
    uint32_t lower;
    const uint32_t cb = cut_band(hist, kBands, half, &lower);
    if (cb == kBands) {  // every bit banded: D = the nonzero rows; else another try
        if (t == 0) {
            cuts[slot] = {1, cb, 0, lower, all ? 0u : 1u, all};
            nd_out[slot] = lower;
            if (!all) *any_redo = 1;
        }
        return;
    }
    const uint32_t *gm = mask + (uint64_t)slot * kMaskWords;
    for (uint32_t j = 0; j < 4; j++) {
        const uint32_t bit = 1024 * j + t, wd = bit >> 5, sh = bit & 31;
        bool in = (gm[wd] >> sh) & 1;
        for (int k = 0; k < kBandPlanes; k++) in = in && ((gm[128 * (k + 1) + wd] >> sh) & 1) == ((cb >> k) & 1);
        const u64 b = ballot(in);
        uint32_t at = 0;
        if ((t & 63) == 0 && b) at = atomicAdd(&counter, (uint32_t)__popcll(b));
        at = readfirst(at) + lanes_below(b);
        if (in) keys[at] = ((u64)gcnt[(uint64_t)slot * QD_BITS + count_at(bit >> 4, bit & 15)] << 12) | bit;
    }
    __syncthreads();
    const uint32_t nb = counter;
    if (nb <= 1024) {
        rank_sort(keys, nb);
    } else {
        const uint32_t np = next_pow2(nb);
        for (uint32_t i = nb + t; i < np; i += 1024) keys[i] = ~0ull;
        __syncthreads();
        block_bitonic_sort(keys, np);
    }
    for (uint32_t i = t; i < nb; i += 1024) {
        rank[(uint64_t)slot * QD_BITS + (keys[i] & 4095)] = (uint16_t)i;
        ghist[(uint64_t)slot * QD_BITS + i] = 0;
    }
    if (t == 0) cuts[slot] = {0, cb, nb, lower, 0, all};
}

// The codes of the cut band's members, and the histogram of their ranks.
__global__ __launch_bounds__(kBlock) void big_refine_kernel(const uint4 *__restrict__ db,
                                                            const uint32_t *__restrict__ perm_in,
                                                            const uint64_t *__restrict__ nbegin,
                                                            const Item *__restrict__ items,
                                                            const uint16_t *__restrict__ grank,
                                                            const uint32_t *__restrict__ gmask,
                                                            const BigCut *__restrict__ cuts, uint32_t again,
                                                            uint16_t *__restrict__ fr_pos,
                                                            uint32_t *__restrict__ ghist) {
    __shared__ uint32_t rows[kChunk];
    __shared__ uint16_t listed[kChunk];
    __shared__ uint32_t hist[QD_BITS];
    __shared__ __attribute__((aligned(16))) uint16_t rank[QD_BITS];
    __shared__ uint32_t counter;
    const Item it = items[blockIdx.x];
    const BigCut cu = cuts[it.slot];
    if (again && cu.all != 2) return;  // whole block
    const uint64_t begin = nbegin[it.slot] + it.first;
    const uint32_t m = it.count, t = threadIdx.x, lane = t & 63, c = t & 31, hw = t >> 5;
    if (t == 0) counter = 0;
    __syncthreads();
    for (uint32_t r0 = 0; r0 < m; r0 += kBlock) {
        const uint32_t r = r0 + t;
        const uint32_t b = r < m ? fr_pos[begin + r] : kNoBand;
        const u64 in = ballot(r < m && b == cu.band);
        uint32_t at = 0;
        if (lane == 0 && in) at = atomicAdd(&counter, (uint32_t)__popcll(in));
        at = readfirst(at) + lanes_below(in);
        if ((in >> lane) & 1) {
            listed[at] = (uint16_t)r;
            rows[at] = perm_in[begin + r];
        } else if (r < m) {
            fr_pos[begin + r] = b < cu.band ? (uint16_t)0 : kNoRank;
        }
    }
    __syncthreads();
    const uint32_t n = counter;
    if (n == 0) return;  // whole block
    const uint4 *gm = reinterpret_cast<const uint4 *>(gmask + (uint64_t)it.slot * kMaskWords);
    uint4 mask = gm[c], band[kBandPlanes];
#pragma unroll
    for (int k = 0; k < kBandPlanes; k++) band[k] = gm[32 * (k + 1) + c];
    mask = band_mask<kBandPlanes>(mask, band, cu.band);
    // histogram in LDS: the cut band of a large node is a few bits, whose
    // counters in memory would take every member's update in turn
    for (uint32_t i = t; i < cu.nb; i += kBlock) hist[i] = 0;
    for (uint32_t i = t; i < QD_BITS / 8; i += kBlock)
        reinterpret_cast<uint4 *>(rank)[i] = reinterpret_cast<const uint4 *>(grank + (uint64_t)it.slot * QD_BITS)[i];
    __syncthreads();
    for (uint32_t b = 0; b < (n + 63) / 64; b++) {
        uint4 v[8];
        load_rows8<8>(db, rows, n, b, hw, c, v);
#pragma unroll
        for (uint32_t i = 0; i < 8; i++) {
            const uint32_t r = (8 * b + i) * 8 + hw;
            if ((r & ~1u) >= n) break;  // both of the wave's rows
            uint32_t best = kNoRank;
            each_bit(and4(v[i], mask), 128 * c, [&](uint32_t bit) { best = min(best, (uint32_t)rank[bit]); });
            best = min32_half(best);
            if (c == 0 && r < n) {
                fr_pos[begin + listed[r]] = (uint16_t)(best + 1);
                atomicAdd(&hist[best], 1u);
            }
        }
    }
    __syncthreads();
    for (uint32_t i = t; i < cu.nb; i += kBlock)
        if (hist[i]) atomicAdd(&ghist[(uint64_t)it.slot * QD_BITS + i], hist[i]);
}

// The cut of a node from the histogram of the cut band's ranks.
__global__ __launch_bounds__(kBlock) void big_cut_kernel(const uint32_t *__restrict__ ghist,
                                                         const uint32_t *__restrict__ ncount, uint32_t again,
                                                         BigCut *__restrict__ cuts, uint32_t *__restrict__ nd_out) {
    __shared__ uint32_t part[4];
    const uint32_t slot = blockIdx.x, t = threadIdx.x, m = ncount[slot], half = (m + 1) / 2;
    const BigCut cu = cuts[slot];
    if (cu.band == kBands || (again && cu.all != 2)) return;  // whole block: the cut stands
    uint32_t h[16], s = 0;
#pragma unroll
    for (uint32_t i = 0; i < 16; i++) {
        const uint32_t r = 16 * t + i;
        h[i] = r < cu.nb ? ghist[(uint64_t)slot * QD_BITS + r] : 0;
        s += h[i];
    }
    uint32_t run = s;  // inclusive over the wave
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)run, o);
        if ((int)(t & 63) >= o) run += y;
    }
    if ((t & 63) == 63) part[t >> 6] = run;
    __syncthreads();
    for (uint32_t x = 0; x < (t >> 6); x++) run += part[x];
    run += cu.lower - s;  // members before this thread's bits
#pragma unroll
    for (uint32_t i = 0; i < 16; i++) {
        if (run < half && run + h[i] >= half) {
            const bool whole = run + h[i] == m;  // D = the codes below this one
            cuts[slot].limit = 1 + 16 * t + i + (whole ? 0u : 1u);
            nd_out[slot] = whole ? run : run + h[i];
        }
        run += h[i];
    }
}

__global__ __launch_bounds__(kBlock) void big_dcount_kernel(const uint64_t *__restrict__ nbegin,
                                                            const Item *__restrict__ items,
                                                            const BigCut *__restrict__ cuts,
                                                            const uint16_t *__restrict__ fr_pos,
                                                            uint32_t *__restrict__ dcount) {
    __shared__ uint32_t total;
    const Item it = items[blockIdx.x];
    const uint64_t begin = nbegin[it.slot] + it.first;
    const uint32_t limit = cuts[it.slot].limit;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    uint32_t c = 0;
    for (uint32_t r = threadIdx.x; r < it.count; r += kBlock) c += fr_pos[begin + r] < limit;
    atomicAdd(&total, c);
    __syncthreads();
    if (threadIdx.x == 0) dcount[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBlock) void big_scatter_kernel(const uint32_t *__restrict__ perm_in,
                                                             uint32_t *__restrict__ perm_out,
                                                             const uint64_t *__restrict__ nbegin,
                                                             const uint32_t *__restrict__ ncount,
                                                             const Item *__restrict__ items,
                                                             const BigCut *__restrict__ cuts,
                                                             const uint32_t *__restrict__ nds,
                                                             const uint16_t *__restrict__ fr_pos,
                                                             const uint32_t *__restrict__ dcount) {
    __shared__ uint32_t tally[kChunk / 64], part[kBlock / 64];
    const Item it = items[blockIdx.x];
    const uint64_t nb0 = nbegin[it.slot], begin = nb0 + it.first;
    const uint32_t limit = cuts[it.slot].limit, t = threadIdx.x, w = t >> 6, lane = t & 63;
    constexpr uint32_t kPerThread = kChunk / kBlock;
    u64 dm[kPerThread];
#pragma unroll
    for (uint32_t i = 0; i < kPerThread; i++) {
        const uint32_t r = i * kBlock + t;
        dm[i] = ballot(r < it.count && fr_pos[begin + r] < limit);
        if (lane == 0) tally[i * 4 + w] = (uint32_t)__popcll(dm[i]);
    }
    // dissimilar members of the node's earlier items, which come just before
    // this one's (at most a few thousand)
    uint32_t s = 0;
    for (uint32_t i = t; i < it.first / kChunk; i += kBlock) s += dcount[blockIdx.x - it.first / kChunk + i];
    s = wave_sum(s);
    if (lane == 0) part[w] = s;
    __syncthreads();
    const uint32_t ns = ncount[it.slot] - nds[it.slot];
    uint32_t before = part[0] + part[1] + part[2] + part[3], g = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPerThread; i++) {
        for (; g < i * 4 + w; g++) before += tally[g];
        const uint32_t r = i * kBlock + t;
        if (r < it.count) {
            const uint32_t d = before + lanes_below(dm[i]);
            perm_out[nb0 + ((dm[i] >> lane) & 1 ? ns + d : it.first + r - d)] = perm_in[begin + r];
        }
    }
}

// ---- images and the leaf-ordered copy ----

// sorted[i] = db[perm[i]]
__global__ __launch_bounds__(kBlock) void gather_rows_kernel(const uint4 *__restrict__ db,
                                                             const uint32_t *__restrict__ perm, uint64_t n,
                                                             uint4 *__restrict__ sorted) {
    const uint64_t tid = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t e = tid; e < n * 32; e += stride) sorted[e] = db[(uint64_t)perm[e >> 5] * 32 + (e & 31)];
}

// Smallest and largest of a wave's 64 values (every lane gets them).
__device__ __forceinline__ void wave_min_max(uint32_t &mn, uint32_t &mx) {
#pragma unroll
    for (int sh = 1; sh < 64; sh <<= 1) {
        const uint32_t a = (uint32_t)__shfl_xor((int)mn, sh), b = (uint32_t)__shfl_xor((int)mx, sh);
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
    }
}

// One wave per node, for the leaves: OR / AND over a leaf's rows of the
// leaf-ordered copy, and the popcount range of the rows (when pmin is given).
__global__ __launch_bounds__(kBlock) void leaf_images_kernel(const uint4 *__restrict__ sorted,
                                                             const int32_t *__restrict__ child, uint32_t n_nodes,
                                                             const uint32_t *__restrict__ begin,
                                                             const uint32_t *__restrict__ count,
                                                             uint4 *__restrict__ or_img, uint4 *__restrict__ and_img,
                                                             const uint16_t *__restrict__ pop,
                                                             uint16_t *__restrict__ pmin, uint16_t *__restrict__ pmax) {
    const uint32_t node = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (node >= n_nodes || child[2 * (uint64_t)node] >= 0) return;  // whole wave
    const int lane = threadIdx.x & 63;
    const uint32_t c = lane & 31, half = lane >> 5;
    const uint64_t b = begin[node];
    const uint32_t m = count[node];
    uint4 o = make_uint4(0, 0, 0, 0), a = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (uint32_t r = half; r < m; r += 2) {
        const uint4 v = sorted[(b + r) * 32 + c];
        o.x |= v.x; o.y |= v.y; o.z |= v.z; o.w |= v.w;
        a.x &= v.x; a.y &= v.y; a.z &= v.z; a.w &= v.w;
    }
    // combine the two half-waves (lane l with lane l^32)
    uint4 o2, a2;
    o2.x = __shfl_xor(o.x, 32); o2.y = __shfl_xor(o.y, 32); o2.z = __shfl_xor(o.z, 32); o2.w = __shfl_xor(o.w, 32);
    a2.x = __shfl_xor(a.x, 32); a2.y = __shfl_xor(a.y, 32); a2.z = __shfl_xor(a.z, 32); a2.w = __shfl_xor(a.w, 32);
    if (half == 0) {
        or_img[(uint64_t)node * 32 + c] = make_uint4(o.x | o2.x, o.y | o2.y, o.z | o2.z, o.w | o2.w);
        if (and_img) and_img[(uint64_t)node * 32 + c] = make_uint4(a.x & a2.x, a.y & a2.y, a.z & a2.z, a.w & a2.w);
    }
    if (pmin) {
        uint32_t mn = 0xFFFFu, mx = 0;
        for (uint32_t r = lane; r < m; r += 64) {
            const uint32_t v = pop[b + r];
            mn = v < mn ? v : mn;
            mx = v > mx ? v : mx;
        }
        wave_min_max(mn, mx);
        if (lane == 0) {
            pmin[node] = (uint16_t)mn;
            pmax[node] = (uint16_t)mx;
        }
    }
}

// One level's nodes first .. first + n - 1: their depth, their children's
// parent, and the inner ones' images and popcount range, which combine the
// two children's.
__global__ __launch_bounds__(kBlock) void inner_images_kernel(uint32_t first, uint32_t n, uint8_t level,
                                                              const int32_t *__restrict__ child,
                                                              uint4 *__restrict__ or_img, uint4 *__restrict__ and_img,
                                                              uint16_t *__restrict__ pmin, uint16_t *__restrict__ pmax,
                                                              int32_t *__restrict__ parent,
                                                              uint8_t *__restrict__ depth) {
    const uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= (uint64_t)n * 32) return;
    const uint32_t c = e & 31;
    const uint64_t node = first + (e >> 5);
    const int32_t s = child[2 * node], d = child[2 * node + 1];
    if (c == 0) depth[node] = level;
    if (node == 0 && c == 1) parent[0] = -1;
    if (s < 0) return;
    const uint4 x = or_img[(uint64_t)s * 32 + c], y = or_img[(uint64_t)d * 32 + c];
    or_img[node * 32 + c] = make_uint4(x.x | y.x, x.y | y.y, x.z | y.z, x.w | y.w);
    if (and_img) {
        const uint4 p = and_img[(uint64_t)s * 32 + c], r = and_img[(uint64_t)d * 32 + c];
        and_img[node * 32 + c] = make_uint4(p.x & r.x, p.y & r.y, p.z & r.z, p.w & r.w);
    }
    if (c == 0) parent[s] = parent[d] = (int32_t)node;
    if (pmin && c == 0) {
        pmin[node] = pmin[s] < pmin[d] ? pmin[s] : pmin[d];
        pmax[node] = pmax[s] > pmax[d] ? pmax[s] : pmax[d];
    }
}

__global__ __launch_bounds__(kBlock) void identity_kernel(uint32_t *__restrict__ perm, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock)
        perm[i] = (uint32_t)i;
}

__global__ __launch_bounds__(kBlock) void invert_perm_kernel(const uint32_t *__restrict__ perm, uint64_t n,
                                                             uint32_t *__restrict__ iperm) {
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock)
        iperm[perm[i]] = (uint32_t)i;
}

}  // namespace

void tree_release(qd_tree_s *t) {
    if (!t) return;
    void *ptrs[] = {t->d_sorted, t->d_perm,  t->d_or,     t->d_and,   t->d_child, t->d_begin, t->d_count,
                    t->d_pop,    t->d_parent, t->d_depth, t->d_iperm, t->d_blk,   t->d_pmin,  t->d_pmax,
                    t->d_bpop,   t->d_split_roots};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    delete t;
}

int tree_build_impl(const uint64_t *d_db, uint64_t n, const qd_build_params *params, void *stream, qd_tree_t *out) {
    if (!out) return fail(QD_ERR_INVALID, "null output handle");
    *out = nullptr;
    if (!d_db) return fail(QD_ERR_INVALID, "null database");
    if (n < 1 || n > QD_MAX_ROWS) return fail(QD_ERR_INVALID, "n=%llu outside 1..%llu", (u64)n, (u64)QD_MAX_ROWS);
    if (!aligned16(d_db)) return fail(QD_ERR_INVALID, "database must be 16-byte aligned");
    const uint32_t max_leaf = params && params->max_leaf ? params->max_leaf : 32;
    const bool want_and = params && params->store_and_image;
    const bool want_pop = !(params && params->plain_bound);
    if (max_leaf > kSmall) return fail(QD_ERR_INVALID, "max_leaf %u above %u", max_leaf, kSmall);
    if (abort_requested()) return fail(QD_ERR_ABORTED, "tree build aborted");
    hipStream_t s = (hipStream_t)stream;
    const uint4 *db4 = reinterpret_cast<const uint4 *>(d_db);

    // Scratch for all levels, in the memory of the leaf-ordered rows, which are
    // written last: a level's split nodes are disjoint and hold more than
    // max_leaf rows each (large ones more than kSmall), which bounds the lists
    // and the large nodes' tables to some 50 bytes per row.  Buffers of each
    // level's own (ten allocations and frees, each a wait), id lists for the
    // images and an uploaded identity order left the GPU idle for 4.5 ms of a
    // build of 1M rows that now takes 8; one allocation and free still took 0.6.
    const uint64_t max_split = n / (max_leaf + 1) + 1, max_big = n / (kSmall + 1) + 1, max_items = n / kChunk + max_big;
    size_t bytes = 0;
    auto take = [&](size_t b) {
        const size_t at = bytes;
        bytes += (b + 255) & ~(size_t)255;
        return at;
    };
    // a level's lists, uploaded in one piece: begins and counts of the split
    // nodes; of the large ones the items and count sources, and the counted
    // nodes' begins and items
    const uint64_t max_up = max_split * 12 + max_items * 2 * sizeof(Item) + max_big * (8 + sizeof(CountSource)) + 128;
    const size_t o_pa = take(n * 4), o_pb = take(n * 4), o_fr = take(n * 2), o_up = take(max_up),
                 o_nd = take((max_split + 1) * 4), o_dc = take(max_items * 4), o_ga = take(max_big * QD_BITS * 4),
                 o_gb = take(max_big * QD_BITS * 4), o_jc = take(max_big * QD_BITS * 4),
                 o_gh = take(max_big * QD_BITS * 4), o_rank = take(max_big * QD_BITS * 2),
                 o_mask = take(max_big * kMaskWords * 4), o_bh = take(max_big * kBands * 4),
                 o_cuts = take(max_big * sizeof(BigCut));
    std::unique_ptr<qd_tree_s, void (*)(qd_tree_s *)> tree(new qd_tree_s(), tree_release);
    QD_HIP_CHECK(hipMalloc((void **)&tree->d_sorted, std::max<size_t>(n * 512, bytes)));
    QD_HIP_CHECK(hipMalloc((void **)&tree->d_perm, n * 4));
    char *const scratch = (char *)tree->d_sorted;
    char *const d_up = scratch + o_up;
    uint32_t *const d_nd = (uint32_t *)(scratch + o_nd), *const dc = (uint32_t *)(scratch + o_dc),
             *const counted = (uint32_t *)(scratch + o_jc), *const gh = (uint32_t *)(scratch + o_gh),
             *const mask = (uint32_t *)(scratch + o_mask), *const bh = (uint32_t *)(scratch + o_bh);
    uint32_t *gc = (uint32_t *)(scratch + o_ga), *above = (uint32_t *)(scratch + o_gb);  // this level's counts, the last's
    uint16_t *const fr_pos = (uint16_t *)(scratch + o_fr), *const rank = (uint16_t *)(scratch + o_rank);
    BigCut *const cuts = (BigCut *)(scratch + o_cuts);
    uint32_t *pin = (uint32_t *)(scratch + o_pa), *pout = (uint32_t *)(scratch + o_pb);
    hipLaunchKernelGGL(identity_kernel, dim3((uint32_t)std::min<uint64_t>((n + kBlock - 1) / kBlock, 4096)),
                       dim3(kBlock), 0, s, pin, n);

    std::vector<uint64_t> begin{0};
    std::vector<uint32_t> count{(uint32_t)n};
    std::vector<int32_t> child{-1, -1};
    std::vector<uint32_t> level_first{0};
    std::vector<uint32_t> last_big;  // per pair of the level's nodes, the parent's slot (kNoKey: not large)
    uint64_t lv0 = 0, lv1 = 1;
    while (lv0 < lv1) {
        if (abort_requested()) {  // between levels: nothing of this level is queued yet
            (void)hipStreamSynchronize(s);
            return fail(QD_ERR_ABORTED, "tree build aborted");
        }
        std::vector<uint32_t> small, big;  // small: by the kernel that splits them
        size_t nkept = 0, nmid = 0;
        for (uint32_t lo : {0u, kKept, kMid, kSmall}) {
            const uint32_t hi = lo == 0 ? kKept : lo == kKept ? kMid : lo == kMid ? kSmall : ~0u;
            for (uint64_t i = lv0; i < lv1; i++)
                if (count[i] > max_leaf && count[i] > lo && count[i] <= hi)
                    (lo == kSmall ? big : small).push_back((uint32_t)i);
            if (lo == 0) nkept = small.size();
            if (lo == kKept) nmid = small.size();
        }
        if (small.empty() && big.empty()) break;
        QD_HIP_CHECK(hipMemcpyAsync(pout, pin, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
        const size_t nsplit = small.size() + big.size();
        std::vector<Item> items, count_items;
        std::vector<CountSource> sources;
        std::vector<uint64_t> jobs;  // the counted nodes' begins
        auto add_items = [](std::vector<Item> &to, size_t slot, uint32_t m) {
            for (uint32_t f = 0; f < m; f += kChunk) to.push_back({(uint32_t)slot, f, std::min(kChunk, m - f), 0});
        };
        for (size_t i = 0; i < big.size(); i++) {
            const uint32_t node = big[i];
            add_items(items, i, count[node]);
            if (node == 0) {  // the root is counted itself
                sources.push_back({0, kNoKey});
                jobs.push_back(0);
                add_items(count_items, 0, count[0]);
                continue;
            }
            // a level's nodes are pairs of siblings; the pair's first large node starts its job
            const uint64_t first = lv0 + ((node - lv0) & ~1ull), few = first + (count[first + 1] < count[first] ? 1 : 0);
            if (node == first || count[first] <= kSmall) {
                add_items(count_items, jobs.size(), count[few]);
                jobs.push_back(begin[few]);
            }
            sources.push_back({(uint32_t)jobs.size() - 1, node == few ? kNoKey : last_big[(first - lv0) / 2]});
        }
        std::vector<char> up;
        auto put = [&](const void *from, size_t b) {
            const size_t at = up.size();
            up.resize((at + b + 15) & ~(size_t)15);
            if (b) memcpy(up.data() + at, from, b);
            return at;
        };
        std::vector<uint64_t> hb(nsplit);
        std::vector<uint32_t> hc(nsplit);
        for (size_t i = 0; i < nsplit; i++) {
            const uint32_t node = i < small.size() ? small[i] : big[i - small.size()];
            hb[i] = begin[node];
            hc[i] = count[node];
        }
        const size_t u_begin = put(hb.data(), nsplit * 8), u_count = put(hc.data(), nsplit * 4),
                     u_items = put(items.data(), items.size() * sizeof(Item)),
                     u_cit = put(count_items.data(), count_items.size() * sizeof(Item)),
                     u_jobs = put(jobs.data(), jobs.size() * 8),
                     u_src = put(sources.data(), sources.size() * sizeof(CountSource));
        if (up.size() > max_up) return fail(QD_ERR_DEVICE, "tree build: level lists past their bound");
        QD_HIP_CHECK(hipMemcpyAsync(d_up, up.data(), up.size(), hipMemcpyHostToDevice, s));
        const uint64_t *const d_begin = (const uint64_t *)(d_up + u_begin);
        const uint32_t *const d_count = (const uint32_t *)(d_up + u_count);
        auto split = [&](auto kernel, uint32_t threads, size_t first, size_t last) {
            if (first < last)
                hipLaunchKernelGGL(kernel, dim3((uint32_t)(last - first)), dim3(threads), 0, s, db4, pin, pout,
                                   d_begin + first, d_count + first, d_nd + first);
        };
        split(split_small_kernel<4, kKept, true>, 256, 0, nkept);
        split(split_small_kernel<4, kMid, false>, 256, nkept, nmid);
        split(split_small_kernel<8, kSmall, false>, 512, nmid, small.size());
        QD_HIP_CHECK(hipGetLastError());
        const size_t nbig = big.size(), ni = items.size();
        const Item *const d_items = (const Item *)(d_up + u_items);
        const uint64_t *const bbeg = d_begin + small.size();
        const uint32_t *const bcnt = d_count + small.size();
        uint32_t *const bnd_out = d_nd + small.size(), *const any_redo = d_nd + nsplit;
        // with the least popular bits, or, where they reach too few members, with all
        auto split_big = [&](uint32_t again) {
            hipLaunchKernelGGL(big_band_kernel, dim3((uint32_t)nbig), dim3(1024), 0, s,
                               (const CountSource *)(d_up + u_src), counted, above, gc, bcnt, again ? 0u : kLambdaBig,
                               mask, bh, cuts, any_redo);
            hipLaunchKernelGGL(big_first_kernel, dim3((uint32_t)ni), dim3(kBlock), 0, s, db4, pin, bbeg, d_items, mask,
                               cuts, again, fr_pos, bh);
            hipLaunchKernelGGL(big_rank_kernel, dim3((uint32_t)nbig), dim3(1024), 0, s, gc, bcnt, mask, bh, again,
                               rank, gh, cuts, bnd_out, any_redo);
            hipLaunchKernelGGL(big_refine_kernel, dim3((uint32_t)ni), dim3(kBlock), 0, s, db4, pin, bbeg, d_items,
                               rank, mask, cuts, again, fr_pos, gh);
            hipLaunchKernelGGL(big_cut_kernel, dim3((uint32_t)nbig), dim3(kBlock), 0, s, gh, bcnt, again, cuts,
                               bnd_out);
            hipLaunchKernelGGL(big_dcount_kernel, dim3((uint32_t)ni), dim3(kBlock), 0, s, bbeg, d_items, cuts, fr_pos,
                               dc);
            hipLaunchKernelGGL(big_scatter_kernel, dim3((uint32_t)ni), dim3(kBlock), 0, s, pin, pout, bbeg, bcnt,
                               d_items, cuts, bnd_out, fr_pos, dc);
        };
        if (nbig) {
            QD_HIP_CHECK(hipMemsetAsync(counted, 0, jobs.size() * QD_BITS * 4, s));
            hipLaunchKernelGGL(big_count_kernel, dim3((uint32_t)count_items.size()), dim3(kBlock), 0, s, db4, pin,
                               (const uint64_t *)(d_up + u_jobs), (const Item *)(d_up + u_cit), counted);
            split_big(0);
            QD_HIP_CHECK(hipGetLastError());
        }
        std::vector<uint32_t> hnd(nsplit + 1, 0);
        const size_t n_back = (nsplit + (nbig ? 1 : 0)) * 4;  // and the flag of a large node's second try
        QD_HIP_CHECK(hipMemcpyAsync(hnd.data(), d_nd, n_back, hipMemcpyDeviceToHost, s));
        QD_HIP_CHECK(hipStreamSynchronize(s));
        if (hnd[nsplit]) {
            split_big(1);
            QD_HIP_CHECK(hipGetLastError());
            QD_HIP_CHECK(hipMemcpyAsync(hnd.data(), d_nd, n_back, hipMemcpyDeviceToHost, s));
            QD_HIP_CHECK(hipStreamSynchronize(s));
        }
        // children in breadth-first order: parents in id order, similar first
        std::vector<uint32_t> nd_of(lv1 - lv0, 0), slot_of(lv1 - lv0, kNoKey);
        for (size_t i = 0; i < nsplit; i++) nd_of[(i < small.size() ? small[i] : big[i - small.size()]) - lv0] = hnd[i];
        for (size_t i = 0; i < nbig; i++) slot_of[big[i] - lv0] = (uint32_t)i;
        last_big.clear();
        const uint64_t next0 = begin.size();
        for (uint64_t node = lv0; node < lv1; node++) {
            const uint32_t nd = nd_of[node - lv0], m = count[node];
            if (nd == 0 || nd >= m) continue;  // no split possible: the node stays a leaf
            last_big.push_back(slot_of[node - lv0]);
            const int32_t sid = (int32_t)begin.size();
            begin.push_back(begin[node]);
            count.push_back(m - nd);
            begin.push_back(begin[node] + (m - nd));
            count.push_back(nd);
            child[2 * node] = sid;
            child[2 * node + 1] = sid + 1;
            child.push_back(-1);
            child.push_back(-1);
            child.push_back(-1);
            child.push_back(-1);
        }
        std::swap(pin, pout);
        std::swap(gc, above);
        lv0 = next0;
        lv1 = begin.size();
        if (lv1 > lv0) level_first.push_back((uint32_t)lv0);
    }
    level_first.push_back((uint32_t)begin.size());

    // The final permutation is in `pin`.
    const uint64_t nn = begin.size();
    qd_tree_s *t = tree.release();
    t->n = n;
    t->n_nodes = nn;
    t->max_leaf = max_leaf;
    t->has_and = want_and;
    if (hipMemcpyAsync(t->d_perm, pin, n * 4, hipMemcpyDeviceToDevice, s) != hipSuccess) {
        tree_release(t);
        return fail(QD_ERR_DEVICE, "tree upload failed");
    }
    {
        uint64_t blocks = std::min<uint64_t>((n * 32 + kBlock - 1) / kBlock, (uint64_t)device_cus() * 64);
        hipLaunchKernelGGL(gather_rows_kernel, dim3((uint32_t)blocks), dim3(kBlock), 0, s, db4, t->d_perm, n,
                           reinterpret_cast<uint4 *>(t->d_sorted));
    }
    std::vector<uint32_t> hb32(nn);
    for (uint64_t i = 0; i < nn; i++) hb32[i] = (uint32_t)begin[i];
    const int rc = tree_finish(t, child, hb32, count, want_pop, s);
    if (rc != QD_OK) return rc;  // tree_finish released t
    *out = t;
    return QD_OK;
}

int tree_finish(qd_tree_s *t, const std::vector<int32_t> &child, const std::vector<uint32_t> &begin,
                const std::vector<uint32_t> &count, bool want_pop, hipStream_t s) {
    const uint64_t n = t->n, nn = t->n_nodes;
    const bool want_and = t->has_and;
    auto cleanup = [&](int code) {
        tree_release(t);
        return code;
    };
    if (hipMalloc((void **)&t->d_or, nn * 512) != hipSuccess || hipMalloc((void **)&t->d_child, nn * 8) != hipSuccess ||
        hipMalloc((void **)&t->d_begin, nn * 4) != hipSuccess || hipMalloc((void **)&t->d_count, nn * 4) != hipSuccess ||
        hipMalloc((void **)&t->d_pop, n * 2) != hipSuccess || hipMalloc((void **)&t->d_parent, nn * 4) != hipSuccess ||
        hipMalloc((void **)&t->d_depth, nn) != hipSuccess || hipMalloc((void **)&t->d_iperm, n * 4) != hipSuccess ||
        (want_and && hipMalloc((void **)&t->d_and, nn * 512) != hipSuccess) ||
        (want_pop && (hipMalloc((void **)&t->d_pmin, nn * 2) != hipSuccess ||
                      hipMalloc((void **)&t->d_pmax, nn * 2) != hipSuccess)))
        return cleanup(fail(QD_ERR_OOM, "tree allocation failed"));
    if (hipMemcpyAsync(t->d_child, child.data(), nn * 8, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(t->d_begin, begin.data(), nn * 4, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(t->d_count, count.data(), nn * 4, hipMemcpyHostToDevice, s) != hipSuccess)
        return cleanup(fail(QD_ERR_DEVICE, "tree upload failed"));
    {
        const int rc = qd_popcount_rows(t->d_sorted, n, t->d_pop, s);  // leaf-order rows
        if (rc != QD_OK) return cleanup(rc);
    }
    hipLaunchKernelGGL(leaf_images_kernel, dim3((uint32_t)((nn + 3) / 4)), dim3(kBlock), 0, s,
                       reinterpret_cast<const uint4 *>(t->d_sorted), t->d_child, (uint32_t)nn, t->d_begin, t->d_count,
                       reinterpret_cast<uint4 *>(t->d_or), reinterpret_cast<uint4 *>(t->d_and), t->d_pop, t->d_pmin,
                       t->d_pmax);
    uint64_t n_leaves = 0;
    for (uint64_t i = 0; i < nn; i++) n_leaves += child[2 * i] < 0;
    t->n_leaves = n_leaves;
    // breadth-first numbering: a level's nodes are consecutive, children after parents
    std::vector<uint32_t> level(nn, 0);
    for (uint64_t i = 0; i < nn; i++)
        if (child[2 * i] >= 0) level[child[2 * i]] = level[child[2 * i + 1]] = level[i] + 1;
    std::vector<uint32_t> level_first{0};
    for (uint64_t i = 1; i < nn; i++)
        if (level[i] != level[i - 1]) level_first.push_back((uint32_t)i);
    level_first.push_back((uint32_t)nn);
    t->depth = (uint32_t)level_first.size() - 1;
    t->level_max.assign(t->depth, 0);
    for (uint64_t i = 0; i < nn; i++) t->level_max[level[i]] = std::max(t->level_max[level[i]], count[i]);
    // The per-query search split into n subtree searches: position p (its
    // log2(n) bits from the most significant, 0 = the similar child) is the
    // node reached from the root along p's bits; a leaf met on the way is the
    // subtree of the first position below it, the other positions below it
    // are empty.  With the nodes under each node (children come after their
    // parents), the most nodes of any subtree bounds one search's queue.
    std::vector<int32_t> split_roots(2 * kMaxCut - 1, -1);
    {
        std::vector<uint32_t> under(nn, 1);
        for (uint64_t i = nn; i-- > 0;)
            if (child[2 * i] >= 0) under[i] = 1 + under[child[2 * i]] + under[child[2 * i + 1]];
        for (uint32_t e = 0; e <= kCutLevels; e++) {
            const uint32_t ns = 1u << e;
            uint64_t most = 0;
            for (uint32_t p = 0; p < ns; p++) {
                int32_t c = 0;
                for (uint32_t l = 0; l < e; l++) {
                    const int32_t a = child[2 * (uint64_t)c], b = child[2 * (uint64_t)c + 1];
                    if (a < 0) {
                        if ((p & ((1u << (e - l)) - 1u)) != 0) c = -1;
                        break;
                    }
                    c = (p >> (e - 1 - l)) & 1u ? b : a;
                }
                split_roots[ns - 1 + p] = c;
                if (c >= 0) most = std::max<uint64_t>(most, under[c]);
            }
            t->split_nodes[e] = most;
        }
    }
    if (hipMalloc((void **)&t->d_split_roots, split_roots.size() * 4) != hipSuccess)
        return cleanup(fail(QD_ERR_OOM, "tree allocation failed"));
    if (hipMemcpyAsync(t->d_split_roots, split_roots.data(), split_roots.size() * 4, hipMemcpyHostToDevice, s) != hipSuccess)
        return cleanup(fail(QD_ERR_DEVICE, "tree upload failed"));
    // inner nodes, deepest level first
    for (int L = (int)level_first.size() - 2; L >= 0; L--) {
        const uint32_t first = level_first[L], m = level_first[L + 1] - first;
        hipLaunchKernelGGL(inner_images_kernel, dim3((uint32_t)(((uint64_t)m * 32 + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, s, first, m, (uint8_t)std::min(255, L), t->d_child,
                           reinterpret_cast<uint4 *>(t->d_or), reinterpret_cast<uint4 *>(t->d_and), t->d_pmin,
                           t->d_pmax, t->d_parent, t->d_depth);
    }
    hipLaunchKernelGGL(invert_perm_kernel, dim3((uint32_t)std::min<uint64_t>((n + kBlock - 1) / kBlock, 65535)),
                       dim3(kBlock), 0, s, t->d_perm, n, t->d_iperm);
    int rc = tree_block_images(t, s);
    if (rc != QD_OK) return cleanup(rc);
    if (hipStreamSynchronize(s) != hipSuccess || hipGetLastError() != hipSuccess)
        return cleanup(fail(QD_ERR_DEVICE, "tree build kernels failed"));
    (void)hipGetDevice(&t->device);
    return QD_OK;
}

}  // namespace qd

extern "C" int qd_tree_build(const uint64_t *d_db, uint64_t n, const qd_build_params *p, void *stream,
                             qd_tree_t *out) {
    return qd::tree_build_impl(d_db, n, p, stream, out);
}

extern "C" int qd_tree_free(qd_tree_t t) {
    qd::tree_release(t);
    return QD_OK;
}

extern "C" int qd_tree_info(qd_tree_t t, qd_tree_info_t *info) {
    if (!t || !info) return qd::fail(QD_ERR_INVALID, "null argument");
    info->n = t->n;
    info->n_nodes = t->n_nodes;
    info->n_leaves = t->n_leaves;
    info->depth = t->depth;
    info->max_leaf = t->max_leaf;
    info->has_and_image = t->has_and ? 1 : 0;
    info->has_pop_range = t->d_pmin ? 1 : 0;
    return QD_OK;
}

extern "C" int qd_tree_export(qd_tree_t t, int32_t *h_child, uint32_t *h_begin, uint32_t *h_count, uint64_t *h_or,
                              uint64_t *h_and, uint32_t *h_perm) {
    if (!t) return qd::fail(QD_ERR_INVALID, "null tree");
    if (h_and && !t->has_and) return qd::fail(QD_ERR_INVALID, "tree stores no product images");
    (void)hipSetDevice(t->device);
    struct {
        void *dst;
        const void *src;
        size_t bytes;
    } cp[] = {{h_child, t->d_child, t->n_nodes * 8}, {h_begin, t->d_begin, t->n_nodes * 4},
              {h_count, t->d_count, t->n_nodes * 4}, {h_or, t->d_or, t->n_nodes * 512},
              {h_and, t->d_and, t->n_nodes * 512},   {h_perm, t->d_perm, t->n * 4}};
    for (auto &c : cp)
        if (c.dst) QD_HIP_CHECK(hipMemcpy(c.dst, c.src, c.bytes, hipMemcpyDeviceToHost));
    return QD_OK;
}
