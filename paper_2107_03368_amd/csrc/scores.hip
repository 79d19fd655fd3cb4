// Object-level distance scores (Section 6.4, the object matching behind
// Table 1 and the confusion matrices): the score of query object g against
// database object o is the sum, over g's descriptors in their given order, of
// each descriptor's distance (Eq. 1) to its nearest descriptor of o.
//
// Stage 1 groups the database rows by object (a counting sort of row ids: one
// histogram, one scan that also numbers each object's 64-row tiles, one
// scatter, one record per tile).  Stage 2 is a sequential search on the matrix
// cores (encoding of mfma_tile.h) in which every row tile belongs to one
// object: a wave keeps its 64 descriptors' smallest keys over an object's tiles
// and folds them into minK[descriptor][object] with one atomic minimum per
// descriptor; the minimum does not depend on the order of the tiles.  Stage 3
// gives every (query object, object) pair one thread, which adds the terms
// minK / (wA wB) in float64, descriptor after descriptor.  Query descriptors
// are taken in batches that bound minK; each batch continues the running sums.
// qd_score_rows ranks the objects of each query object and rescales its row
// to [0, 1], the confusion-matrix row.
#include <algorithm>

#include "mfma_tile.h"
#include "qd_device.h"
#include "qd_internal.h"

namespace qd {

int popcount_rows_launch(const uint64_t *d_db, uint64_t n, uint16_t *d_pop, hipStream_t s);

namespace {

constexpr int kBlock = 256;
constexpr int MQ = 256;  // descriptors of a batch come in multiples of it
constexpr int MR = 64;   // rows per tile
constexpr uint32_t kNoKey = 0xFFFFFFFFu;       // above every key (keys are < 2^24)
constexpr uint64_t kMinKBytes = 1ull << 30;    // minK of one batch
constexpr uint64_t kMaxBatch = 1ull << 18;     // query descriptors per batch
constexpr uint32_t kMaxObjects = 65536;        // object ids are uint16

__global__ void fill_u32_kernel(uint32_t *p, uint64_t n, uint32_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void fill_f64_kernel(double *p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// Counting and scattering by object.  One global atomic per row would queue
// the rows of an object, which usually come together, on one address.
// Up to kLdsObjects objects: a block takes kBlockRows rows, counts them in LDS
// and adds each object once; the scatter then hands out the block's reserved
// places from LDS.
// More objects: a wave takes kRun consecutive rows; where they are all of one
// object it adds once, else, 64 rows at a time, the first two objects it
// meets are added once each and what is left (rows of objects in turn) one
// atomic per row, which then spreads over the objects.
// 1.5M rows of 300 objects, count and scatter together: 0.03 ms in any order;
// with an atomic per row 7.5 ms in order, 0.2 ms in turn, 1.2 ms at random.
constexpr uint32_t kLdsObjects = 8192;
constexpr uint32_t kLdsBlock = 1024, kBlockRows = 8 * kLdsBlock;
constexpr uint32_t kRun = 1024;

// Rows [r0, r0 + kRun) of a wave: object of row r0 + 64 i + lane (kNone
// past the end and for ids that belong to no object) and whether all are one object.
constexpr uint32_t kNone = 0xFFFFFFFFu;
__device__ __forceinline__ bool load_run(const uint16_t *__restrict__ obj_of, uint64_t n, uint32_t n_obj, uint64_t r0,
                                         uint32_t (&o)[kRun / 64]) {
    const int lane = lane_id();
#pragma unroll
    for (uint32_t i = 0; i < kRun / 64; i++) {
        const uint64_t t = r0 + 64 * i + lane;
        const uint32_t v = obj_of[t < n ? t : n - 1];
        o[i] = t < n && v < n_obj ? v : kNone;  // ids >= n_obj belong to no object
    }
    const uint32_t first = readfirst(o[0]);
    bool same = first != kNone;
#pragma unroll
    for (uint32_t i = 0; i < kRun / 64; i++) same = same && o[i] == first;
    return ballot(!same) == 0;
}

// add(object, mask) for the rows of one object among the lanes (called by the
// whole wave), single(object) for a lane's row alone.
template <class Add, class Single>
__device__ __forceinline__ void by_object(uint32_t o, Add &&add, Single &&single) {
    u64 left = ballot(o != kNone);
#pragma unroll
    for (int pass = 0; pass < 2; pass++) {
        if (left == 0) return;
        const uint32_t first = readlane(o, __builtin_ctzll(left));
        const u64 m = ballot(o == first);
        add(first, m);
        left &= ~m;
        o = o == first ? kNone : o;
    }
    if (o != kNone) single(o);
}

__global__ __launch_bounds__(kBlock) void obj_count_kernel(const uint16_t *__restrict__ obj_of, uint64_t n,
                                                           uint32_t n_obj, uint32_t *__restrict__ cnt) {
    const int lane = lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * (kBlock / 64);
    for (uint64_t run = (uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); run * kRun < n; run += waves) {
        uint32_t o[kRun / 64];
        if (load_run(obj_of, n, n_obj, run * kRun, o)) {
            if (lane == 0) atomicAdd(&cnt[o[0]], kRun);
            continue;
        }
#pragma unroll
        for (uint32_t i = 0; i < kRun / 64; i++)
            by_object(
                o[i],
                [&](uint32_t ob, u64 m) {
                    if (lane == 0) atomicAdd(&cnt[ob], (uint32_t)__popcll(m));
                },
                [&](uint32_t ob) { atomicAdd(&cnt[ob], 1u); });
    }
}

__global__ __launch_bounds__(kLdsBlock) void obj_count_lds_kernel(const uint16_t *__restrict__ obj_of, uint64_t n,
                                                                  uint32_t n_obj, uint32_t *__restrict__ cnt) {
    __shared__ uint32_t hist[kLdsObjects];
    for (uint32_t i = threadIdx.x; i < n_obj; i += kLdsBlock) hist[i] = 0;
    __syncthreads();
    for (uint64_t r0 = (uint64_t)blockIdx.x * kBlockRows; r0 < n; r0 += (uint64_t)gridDim.x * kBlockRows)
#pragma unroll
        for (uint32_t i = 0; i < kBlockRows / kLdsBlock; i++) {
            const uint64_t t = r0 + i * kLdsBlock + threadIdx.x;
            const uint32_t o = t < n ? obj_of[t] : kLdsObjects;
            if (o < n_obj) atomicAdd(&hist[o], 1u);  // ids >= n_obj belong to no object
        }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_obj; i += kLdsBlock)
        if (hist[i]) atomicAdd(&cnt[i], hist[i]);
}

// One block: roff = exclusive prefix of the row counts, toff = exclusive
// prefix of the tile counts ceil(cnt / 64); both with the total at n_obj.
// Also clears the scatter cursors.
__global__ __launch_bounds__(1024) void obj_offsets_kernel(const uint32_t *__restrict__ cnt, uint32_t n_obj,
                                                           uint64_t *__restrict__ roff, uint32_t *__restrict__ toff,
                                                           uint32_t *__restrict__ cursor) {
    __shared__ uint64_t prow[1024];
    __shared__ uint32_t ptile[1024];
    const uint32_t tid = threadIdx.x;
    const uint32_t chunk = (n_obj + 1023) / 1024;
    const uint32_t c0 = tid * chunk < n_obj ? tid * chunk : n_obj;
    const uint32_t c1 = c0 + chunk < n_obj ? c0 + chunk : n_obj;
    uint64_t sr = 0;
    uint32_t st = 0;
    for (uint32_t o = c0; o < c1; o++) {
        sr += cnt[o];
        st += (cnt[o] + MR - 1) / MR;
    }
    prow[tid] = sr;
    ptile[tid] = st;
    __syncthreads();
    for (uint32_t d = 1; d < 1024; d <<= 1) {
        const uint64_t vr = tid >= d ? prow[tid - d] : 0;
        const uint32_t vt = tid >= d ? ptile[tid - d] : 0;
        __syncthreads();
        prow[tid] += vr;
        ptile[tid] += vt;
        __syncthreads();
    }
    uint64_t rr = prow[tid] - sr;
    uint32_t rt = ptile[tid] - st;
    for (uint32_t o = c0; o < c1; o++) {
        roff[o] = rr;
        toff[o] = rt;
        cursor[o] = 0;
        rr += cnt[o];
        rt += (cnt[o] + MR - 1) / MR;
    }
    if (tid == 1023) {
        roff[n_obj] = prow[1023];
        toff[n_obj] = ptile[1023];
    }
}

// Row ids grouped by object; within an object in any order (a minimum over
// the object's rows does not depend on it).
__global__ __launch_bounds__(kBlock) void obj_scatter_kernel(const uint16_t *__restrict__ obj_of, uint64_t n,
                                                             uint32_t n_obj, const uint64_t *__restrict__ roff,
                                                             uint32_t *__restrict__ cursor,
                                                             uint32_t *__restrict__ order) {
    const int lane = lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * (kBlock / 64);
    for (uint64_t run = (uint64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); run * kRun < n; run += waves) {
        const uint64_t r0 = run * kRun;
        uint32_t o[kRun / 64];
        if (load_run(obj_of, n, n_obj, r0, o)) {
            const uint64_t at = roff[o[0]] + readfirst(lane == 0 ? atomicAdd(&cursor[o[0]], kRun) : 0u);
#pragma unroll
            for (uint32_t i = 0; i < kRun / 64; i++) order[at + 64 * i + lane] = (uint32_t)(r0 + 64 * i + lane);
            continue;
        }
#pragma unroll
        for (uint32_t i = 0; i < kRun / 64; i++) {
            const uint32_t t = (uint32_t)(r0 + 64 * i + lane), mine = o[i];
            by_object(
                mine,
                [&](uint32_t ob, u64 m) {
                    const uint32_t c = readfirst(lane == 0 ? atomicAdd(&cursor[ob], (uint32_t)__popcll(m)) : 0u);
                    if (mine == ob) order[roff[ob] + c + lanes_below(m)] = t;
                },
                [&](uint32_t ob) { order[roff[ob] + atomicAdd(&cursor[ob], 1u)] = t; });
        }
    }
}

__global__ __launch_bounds__(kLdsBlock) void obj_scatter_lds_kernel(const uint16_t *__restrict__ obj_of, uint64_t n,
                                                                    uint32_t n_obj, const uint64_t *__restrict__ roff,
                                                                    uint32_t *__restrict__ cursor,
                                                                    uint32_t *__restrict__ order) {
    __shared__ uint32_t at[kLdsObjects];  // the block's rows of each object, then its next place for one
    for (uint64_t r0 = (uint64_t)blockIdx.x * kBlockRows; r0 < n; r0 += (uint64_t)gridDim.x * kBlockRows) {
        for (uint32_t i = threadIdx.x; i < n_obj; i += kLdsBlock) at[i] = 0;
        __syncthreads();
        uint32_t o[kBlockRows / kLdsBlock];
#pragma unroll
        for (uint32_t i = 0; i < kBlockRows / kLdsBlock; i++) {
            const uint64_t t = r0 + i * kLdsBlock + threadIdx.x;
            o[i] = t < n ? obj_of[t] : kLdsObjects;
            if (o[i] < n_obj) atomicAdd(&at[o[i]], 1u);
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n_obj; i += kLdsBlock)
            if (at[i]) at[i] = (uint32_t)roff[i] + atomicAdd(&cursor[i], at[i]);  // n < 2^32 places
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kBlockRows / kLdsBlock; i++)
            if (o[i] < n_obj) order[atomicAdd(&at[o[i]], 1u)] = (uint32_t)(r0 + i * kLdsBlock + threadIdx.x);
        __syncthreads();  // the next round clears `at`
    }
}

// The row tiles' records, one thread per tile: row tile rt lies in the object o
// with toff[o] <= rt < toff[o + 1] (objects without rows have no tiles);
// rec[rt] = (first row in object order, rows, o).  The grid strides over the
// tiles the offsets counted.
__global__ __launch_bounds__(kBlock) void obj_tiles_kernel(const uint64_t *__restrict__ roff,
                                                           const uint32_t *__restrict__ toff, uint32_t n_obj,
                                                           uint4 *__restrict__ rec) {
    const uint32_t total = toff[n_obj];
    for (uint32_t rt = blockIdx.x * kBlock + threadIdx.x; rt < total; rt += gridDim.x * kBlock) {
        uint32_t lo = 0, hi = n_obj;  // toff[lo] <= rt < toff[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (toff[mid] <= rt)
                lo = mid;
            else
                hi = mid;
        }
        const uint64_t r0 = roff[lo] + (uint64_t)(rt - toff[lo]) * MR, r1 = roff[lo + 1];
        rec[rt] = make_uint4((uint32_t)r0, r1 - r0 < (uint64_t)MR ? (uint32_t)(r1 - r0) : (uint32_t)MR, lo, 0);
    }
}

// The smallest key of every (descriptor, object) pair, on the matrix cores: the
// sequential search's matrix pass with the rows gathered in object order.  A
// workgroup keeps a group of up to 256 descriptors packed in LDS; a wave streams
// 64 rows of one object at a time from memory into the operand registers,
// against 64 of the descriptors (2 x 2 fragments; line layout, bit order and
// expansion as in scan_mfma_kernel, |t| counted from the words).  The work is
// cut into units, (group, 64-row tile, 64-descriptor tile of the group); every
// workgroup takes an equal run of row tiles and its 8 waves take the run's units
// in turn, so with 1, 2 or 4 descriptor tiles a wave keeps its descriptors and
// meets an object's tiles one after another: the minima stay in registers until
// the object (or the descriptors) change, and only then go to memory.
// Bound by the matrix units: 13,700 descriptors x 1.5M rows 23.1 ms, 7.3 PFLOP/s;
// 25.1 ms (and 0.12 for the rows' popcounts) with a streamed 256 x 256 tile per
// workgroup, 38.0 with tiles that waited for their loads and 16 x 16 x 128
// instructions.
constexpr int kScanBlock = 512, kScanWaves = kScanBlock / 64;
constexpr uint32_t kGroupD = 256;       // descriptors of a group
constexpr int kDescStride = 512 + 16;   // bytes per descriptor in LDS: 16-byte reads of 32 on distinct banks
struct ScanSmem {
    uint32_t pop[kGroupD];         // |q|
    float tp[kScanWaves][MR];      // per wave: its rows' |t|
};
inline size_t scan_lds_bytes(uint32_t nq) {
    return sizeof(ScanSmem) + (size_t)(nq < kGroupD ? (nq + 63) / 64 * 64 : kGroupD) * kDescStride;
}
__global__ __launch_bounds__(kScanBlock, 2) void objscan_kernel(const uint4 *__restrict__ db,
                                                                const uint32_t *__restrict__ order,
                                                                const uint4 *__restrict__ rec,
                                                                const uint32_t *__restrict__ n_rtiles, uint32_t n_obj,
                                                                const uint4 *__restrict__ q, uint32_t nq,
                                                                uint32_t *__restrict__ minK) {
    extern __shared__ __align__(16) uint8_t s_raw[];
    ScanSmem &sm = *reinterpret_cast<ScanSmem *>(s_raw);
    uint8_t *s_q = s_raw + sizeof(ScanSmem);
    static_assert(sizeof(ScanSmem) % 16 == 0, "the descriptors are read 16 bytes at a time");
    const uint64_t tiles = *n_rtiles;
    const int lane = threadIdx.x & 63, wv = (int)readfirst(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;
    float *tpw = sm.tp[wv];
    // a lane-varying zero: keeps the record loads vector loads (a scalar load
    // shares its completion counter with the LDS reads)
    const uint32_t vz = __builtin_amdgcn_mbcnt_lo(0u, 0u);
    // this workgroup's units [ua, ub) of all groups' (each group: its
    // descriptor tiles x tiles), rounded down to whole row tiles at both ends
    const uint32_t n_qt = (nq + 63) / 64;
    const uint64_t units = tiles * n_qt;
    const uint64_t ua = units / gridDim.x * blockIdx.x + min((uint64_t)blockIdx.x, units % gridDim.x);
    const uint64_t ub = ua + units / gridDim.x + (blockIdx.x < units % gridDim.x ? 1 : 0);
    const uint64_t per_group = 4 * tiles;  // units of a full group
    if (tiles == 0) return;                // whole workgroup
    for (uint64_t g0 = ua / per_group * per_group; g0 < ub; g0 += per_group) {
        const uint32_t q0 = (uint32_t)(g0 / per_group) * kGroupD;  // the group's first descriptor
        const uint32_t gqt = min(4u, n_qt - q0 / 64);              // its descriptor tiles
        const uint64_t ra = (ua > g0 ? ua - g0 : 0) / gqt;         // its row tiles here
        const uint64_t rb = min((ub - g0) / gqt, tiles);
        __syncthreads();  // every wave is done with the group before
        for (uint32_t e = threadIdx.x; e < gqt * 64 * 32; e += kScanBlock) {
            const uint32_t qi = q0 + (e >> 5);
            const uint4 x = qi < nq ? q[(uint64_t)qi * 32 + (e & 31)] : make_uint4(0, 0, 0, 0);
            *reinterpret_cast<uint4 *>(s_q + (size_t)(e >> 5) * kDescStride + (e & 31) * 16) = x;
            const uint32_t pq = sum32_half(popc4(x));  // a half wave holds one descriptor
            if ((e & 31) == 0) sm.pop[e >> 5] = pq;
        }
        __syncthreads();
        // the wave's units wv, wv + 8, ... of (rb - ra) row tiles x gqt descriptor tiles
        const uint64_t un = rb > ra ? (rb - ra) * gqt : 0;
        uint64_t u = (uint64_t)wv;
        if (u >= un) continue;
        uint32_t qt = (uint32_t)wv % gqt;
        uint64_t rt = ra + (uint32_t)wv / gqt;
        // a tile's record, then its rows: fragment b's is lane li's (past the
        // end: the tile's last row, masked in the test)
        auto row_of = [&](const uint4 &r, int b) {
            const uint32_t i = 32 * b + (uint32_t)li;
            return order[r.x + (i < r.y ? i : r.y - 1)];
        };
        uint4 v[2][2][4];  // [line parity][fragment][piece pair]
        auto load = [&](const uint32_t (&row)[2], int L, uint4 (&x)[2][4]) {
#pragma unroll
            for (int b = 0; b < 2; b++) {
                const uint4 *src = db + (uint64_t)row[b] * 32 + 8 * L + lh;
#pragma unroll
                for (int i = 0; i < 4; i++) x[b][i] = src[2 * i];
            }
        };
        auto q_row = [&](uint32_t t) { return s_q + (size_t)(t * 64 + li) * kDescStride + lh * 16; };
        auto word = [](const uint4 &x, int c) { return c == 0 ? x.x : c == 1 ? x.y : c == 2 ? x.z : x.w; };
        const uint8_t *qrow = q_row(qt);
        uint4 qw[2][2];              // descriptors' pieces: [piece pair parity][fragment]
        mt::v8i qv[2][2], rv[2][2];  // operands: [step parity][fragment]
        uint32_t tp[2] = {0, 0};
        auto read_q = [&](const uint8_t *row, int pair) {
#pragma unroll
            for (int a = 0; a < 2; a++)
                qw[pair & 1][a] = *reinterpret_cast<const uint4 *>(row + 32 * a * kDescStride + pair * 32);
        };
        auto expand = [&](int S, int f) {  // fragment f of step S (mod 64): rows 0, 1, then descriptors
            const int L = (S >> 4) & 3, i = (S >> 2) & 3, c = S & 3;
            if (f < 2) {
                const uint32_t x = word(v[L & 1][f][i], c);
                rv[S & 1][f] = mt::expand_r(x);
                tp[f] += __popc(x);
            } else {
                qv[S & 1][f - 2] = mt::expand_q(word(qw[(4 * L + i) & 1][f - 2], c));
            }
        };
        // the minima so far: K = |q|*wB - (C*(wA + wB) - |t|*wA), so the smallest
        // K is |q|*wB minus the largest C*(wA + wB) - |t|*wA.  In fp32 every
        // value is exact: integers below 2^24, but for C = |q| = 4096, where
        // C*(wA + wB) = 4096 * 4097 < 2^25 is even.
        float vmax[2] = {-1e38f, -1e38f};
        auto store_minima = [&](uint32_t o) {
#pragma unroll
            for (int a = 0; a < 2; a++) {
                const uint32_t qs = qt * 64 + 32 * a + li, pq = sm.pop[qs];
                const float m = fmaxf(vmax[a], __shfl_xor(vmax[a], 32));  // the other 16 rows of each fragment
                const int32_t K = (int32_t)(pq * ((QD_BITS - pq) > 1 ? QD_BITS - pq : 1)) - (int32_t)m;
                if (lh == 0 && q0 + qs < nq) atomicMin(&minK[(uint64_t)(q0 + qs) * n_obj + o], (uint32_t)K);
                vmax[a] = -1e38f;
            }
        };
        uint4 cur = rec[rt + vz];
        uint32_t row[2];
#pragma unroll
        for (int b = 0; b < 2; b++) row[b] = row_of(cur, b);
        load(row, 0, v[0]);
        read_q(qrow, 0);
#pragma unroll
        for (int f = 0; f < 4; f++) expand(0, f);
        for (;;) {
            // the wave's next unit (after the last: this one again, unused)
            const bool more = u + kScanWaves < un;
            uint32_t nqt = qt + kScanWaves % gqt;
            const uint32_t wrap = nqt >= gqt ? 1 : 0;
            nqt -= wrap ? gqt : 0;
            const uint64_t nrt = more ? rt + kScanWaves / gqt + wrap : rt;  // row tile, then descriptor tile
            const uint8_t *nqrow = q_row(more ? nqt : qt);
            uint4 nrec;
            uint32_t nrow[2], tcur[2];
            mt::v16f acc[2][2];
#pragma unroll
            for (int L = 0; L < 4; L++) {
                if (L == 0) nrec = rec[nrt + vz];
                if (L == 2) {
#pragma unroll
                    for (int b = 0; b < 2; b++) nrow[b] = row_of(nrec, b);
                }
                load(L < 3 ? row : nrow, (L + 1) & 3, v[(L + 1) & 1]);
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
#pragma unroll
            for (int b = 0; b < 2; b++) {
                tcur[b] += (uint32_t)__shfl_xor((int)tcur[b], 32);
                if (lh == b) tpw[32 * b + li] = 32 * b + (uint32_t)li < cur.y ? (float)tcur[b] : mt::kNoRow;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int a = 0; a < 2; a++) {
                const uint32_t pq = sm.pop[qt * 64 + 32 * a + li];  // this lane's descriptor
                const uint32_t wa = pq > 1 ? pq : 1;
                const float nwa = -(float)wa, sw = (float)(wa + ((QD_BITS - pq) > 1 ? QD_BITS - pq : 1));
#pragma unroll
                for (int b = 0; b < 2; b++)
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const float4 t4 = *reinterpret_cast<const float4 *>(tpw + 32 * b + 8 * g + 4 * lh);
                        const float t[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            vmax[a] = fmaxf(vmax[a], __builtin_fmaf(t[e], nwa, acc[a][b][4 * g + e] * sw));
                    }
            }
            const uint32_t o = readfirst(cur.z);
            if (!more || nqt != qt || readfirst(nrec.z) != o) store_minima(o);
            if (!more) break;
            u += kScanWaves;
            qt = nqt;
            rt = nrt;
            qrow = nqrow;
            cur = nrec;
            row[0] = nrow[0];
            row[1] = nrow[1];
        }
    }
}

// Thread (g, o) for the query objects that overlap this batch, descriptors
// [d0, d0 + nb): adds the batch's terms of g's descriptors, in order, to the
// running score.  g_lo .. g_hi is found per thread by binary search on qoff.
__global__ __launch_bounds__(kBlock) void score_sum_kernel(const uint32_t *__restrict__ minK,
                                                           const uint16_t *__restrict__ qpop, uint64_t d0,
                                                           uint32_t nb, const uint64_t *__restrict__ qoff,
                                                           uint32_t nqo, const uint64_t *__restrict__ roff,
                                                           uint32_t n_obj, double *__restrict__ scores) {
    const uint64_t d1 = d0 + nb;
    // first g whose descriptors end after d0; first g whose descriptors start at or after d1
    uint32_t lo = 0, hi = nqo;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (qoff[mid + 1] <= d0)
            lo = mid + 1;
        else
            hi = mid;
    }
    const uint32_t g_lo = lo;
    hi = nqo;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (qoff[mid] < d1)
            lo = mid + 1;
        else
            hi = mid;
    }
    const uint32_t g_hi = lo;
    const uint64_t total = (uint64_t)(g_hi - g_lo) * n_obj;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t g = g_lo + (uint32_t)(i / n_obj), o = (uint32_t)(i % n_obj);
        const uint64_t a = qoff[g] > d0 ? qoff[g] : d0, b = qoff[g + 1] < d1 ? qoff[g + 1] : d1;
        if (a >= b) continue;
        const bool empty = roff[o + 1] == roff[o];  // the minimum over no rows is +infinity
        double s = scores[(uint64_t)g * n_obj + o];
#pragma unroll 8
        for (uint64_t d = a; d < b; d++) {
            const uint32_t P = qpop[d - d0];
            const uint32_t wa = P > 1 ? P : 1, wb = (QD_BITS - P) > 1 ? QD_BITS - P : 1;
            const double term =
                empty ? __builtin_inf() : (double)minK[(d - d0) * n_obj + o] / ((double)wa * (double)wb);
            s += term;
        }
        scores[(uint64_t)g * n_obj + o] = s;
    }
}

// One block per row of scores: the lowest finite score (ties to the lower
// object id) and the highest, by a block reduction; then, with normalize, the
// row rescaled in place.
__global__ __launch_bounds__(kBlock) void score_rows_kernel(double *__restrict__ scores, uint32_t nqo, uint32_t n_obj,
                                                            int normalize, int32_t *__restrict__ best) {
    __shared__ double s_mn[kBlock], s_mx[kBlock];
    __shared__ int32_t s_arg[kBlock];
    const uint32_t tid = threadIdx.x;
    for (uint32_t g = blockIdx.x; g < nqo; g += gridDim.x) {
        double *row = scores + (uint64_t)g * n_obj;
        double mn = __builtin_inf(), mx = -__builtin_inf();
        int32_t arg = -1;
        for (uint32_t o = tid; o < n_obj; o += kBlock) {  // increasing o: a tie keeps the first
            const double v = row[o];
            if (!__builtin_isfinite(v)) continue;
            if (v < mn) {
                mn = v;
                arg = (int32_t)o;
            }
            mx = v > mx ? v : mx;
        }
        s_mn[tid] = mn;
        s_mx[tid] = mx;
        s_arg[tid] = arg;
        __syncthreads();
        for (uint32_t h = kBlock / 2; h > 0; h >>= 1) {
            if (tid < h) {
                const double m2 = s_mn[tid + h];
                const int32_t a2 = s_arg[tid + h];
                if (a2 >= 0 && (s_arg[tid] < 0 || m2 < s_mn[tid] || (m2 == s_mn[tid] && a2 < s_arg[tid]))) {
                    s_mn[tid] = m2;
                    s_arg[tid] = a2;
                }
                s_mx[tid] = s_mx[tid + h] > s_mx[tid] ? s_mx[tid + h] : s_mx[tid];
            }
            __syncthreads();
        }
        const double lo = s_mn[0], hi = s_mx[0];
        if (tid == 0) best[g] = s_arg[0];
        if (normalize) {
            for (uint32_t o = tid; o < n_obj; o += kBlock) {
                const double v = row[o];
                row[o] = !__builtin_isfinite(v) ? 1.0 : hi > lo ? (v - lo) / (hi - lo) : 0.0;
            }
        }
        __syncthreads();  // the next row reuses the reduction arrays
    }
}

uint32_t blocks_for(uint64_t n, uint64_t cap) {
    const uint64_t b = (n + kBlock - 1) / kBlock;
    return (uint32_t)(b < 1 ? 1 : b > cap ? cap : b);
}

}  // namespace
}  // namespace qd

extern "C" int qd_object_scores(const uint64_t *d_db, uint64_t n, const uint16_t *d_obj_of, uint32_t n_obj,
                                const uint64_t *d_qdesc, uint64_t n_qdesc, const uint64_t *d_qoff, uint32_t nqo,
                                double *d_scores, void *stream) {
    using namespace qd;
    clear_error();
    if (n_obj < 1 || n_obj > kMaxObjects) return fail(QD_ERR_INVALID, "n_obj=%u outside 1..65536", n_obj);
    if (nqo == 0) return QD_OK;
    if (!d_qoff || !d_scores || (n && (!d_db || !d_obj_of)) || (n_qdesc && !d_qdesc))
        return fail(QD_ERR_INVALID, "null pointer");
    if ((n && !aligned16(d_db)) || (n_qdesc && !aligned16(d_qdesc)))
        return fail(QD_ERR_INVALID, "descriptor arrays must be 16-byte aligned");
    if (n > 0xFFFFFFFFull) return fail(QD_ERR_INVALID, "more than 2^32 - 1 database rows");
    hipStream_t s = (hipStream_t)stream;
    const uint64_t n_scores = (uint64_t)nqo * n_obj;
    const uint32_t cap = (uint32_t)device_cus() * 16;
    hipLaunchKernelGGL(fill_f64_kernel, dim3(blocks_for(n_scores, cap)), dim3(kBlock), 0, s, d_scores, n_scores);
    QD_HIP_CHECK(hipGetLastError());
    if (n_qdesc == 0) return QD_OK;

    uint64_t nb_max = kMinKBytes / 4 / n_obj / MQ * MQ;
    if (nb_max < (uint64_t)MQ) nb_max = MQ;
    if (nb_max > kMaxBatch) nb_max = kMaxBatch;
    if (nb_max > n_qdesc) nb_max = n_qdesc;
    // scratch: row order, counts / cursors, offsets, batch popcounts, minK
    const size_t o_order = 0, o_cnt = o_order + ((n * 4 + 255) & ~255ull);
    const size_t o_cur = o_cnt + (((size_t)n_obj * 4 + 255) & ~255ull);
    const size_t o_roff = o_cur + (((size_t)n_obj * 4 + 255) & ~255ull);
    const size_t o_toff = o_roff + ((((size_t)n_obj + 1) * 8 + 255) & ~255ull);
    // row tiles: at most one ragged tile per object that has rows
    const uint64_t row_tiles_max = (n + MR - 1) / MR + (n < n_obj ? n : n_obj);
    const size_t o_rec = o_toff + ((((size_t)n_obj + 1) * 4 + 255) & ~255ull);
    const size_t o_qpop = o_rec + (((size_t)row_tiles_max * 16 + 255) & ~255ull);
    const size_t o_mink = o_qpop + ((nb_max * 2 + 255) & ~255ull);
    const size_t bytes = o_mink + nb_max * n_obj * 4;
    char *ws = nullptr;
    QD_HIP_CHECK(hipMallocAsync((void **)&ws, bytes, s));
    uint32_t *order = reinterpret_cast<uint32_t *>(ws + o_order);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(ws + o_cnt);
    uint32_t *cursor = reinterpret_cast<uint32_t *>(ws + o_cur);
    uint64_t *roff = reinterpret_cast<uint64_t *>(ws + o_roff);
    uint32_t *toff = reinterpret_cast<uint32_t *>(ws + o_toff);
    uint4 *rec = reinterpret_cast<uint4 *>(ws + o_rec);
    uint16_t *qpop = reinterpret_cast<uint16_t *>(ws + o_qpop);
    uint32_t *minK = reinterpret_cast<uint32_t *>(ws + o_mink);
    auto done = [&](int rc) {
        (void)hipFreeAsync(ws, s);
        return rc;
    };

    {
        KernelTimer timer("object_group", s);
        hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks_for(n_obj, cap)), dim3(kBlock), 0, s, cnt, (uint64_t)n_obj,
                           0u);
        const uint32_t run_blocks = blocks_for((n + kRun - 1) / kRun * 64, cap);
        const uint32_t lds_blocks = (uint32_t)std::min<uint64_t>((n + kBlockRows - 1) / kBlockRows, cap);
        if (n) {
            if (n_obj <= kLdsObjects)
                hipLaunchKernelGGL(obj_count_lds_kernel, dim3(lds_blocks), dim3(kLdsBlock), 0, s, d_obj_of, n, n_obj,
                                   cnt);
            else
                hipLaunchKernelGGL(obj_count_kernel, dim3(run_blocks), dim3(kBlock), 0, s, d_obj_of, n, n_obj, cnt);
        }
        hipLaunchKernelGGL(obj_offsets_kernel, dim3(1), dim3(1024), 0, s, cnt, n_obj, roff, toff, cursor);
        if (n) {
            if (n_obj <= kLdsObjects)
                hipLaunchKernelGGL(obj_scatter_lds_kernel, dim3(lds_blocks), dim3(kLdsBlock), 0, s, d_obj_of, n, n_obj,
                                   roff, cursor, order);
            else
                hipLaunchKernelGGL(obj_scatter_kernel, dim3(run_blocks), dim3(kBlock), 0, s, d_obj_of, n, n_obj, roff,
                                   cursor, order);
            hipLaunchKernelGGL(obj_tiles_kernel, dim3(blocks_for(row_tiles_max, cap)), dim3(kBlock), 0, s, roff, toff,
                               n_obj, rec);
        }
        if (hipGetLastError() != hipSuccess) return done(fail(QD_ERR_DEVICE, "object grouping launch failed"));
    }
    for (uint64_t d0 = 0; d0 < n_qdesc; d0 += nb_max) {
        const uint32_t nb = (uint32_t)(n_qdesc - d0 < nb_max ? n_qdesc - d0 : nb_max);
        const uint64_t *qb = d_qdesc + d0 * QD_WORDS;
        int rc = popcount_rows_launch(qb, nb, qpop, s);
        if (rc != QD_OK) return done(rc);
        if (n) {
            const uint64_t m = (uint64_t)nb * n_obj;
            hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks_for(m, cap)), dim3(kBlock), 0, s, minK, m, kNoKey);
            KernelTimer timer("object_scan", s);
            // persistent: one workgroup per CU (LDS and registers leave room for one)
            const uint64_t n_units = (uint64_t)((nb + 63) / 64) * row_tiles_max;
            const uint64_t grid = std::min<uint64_t>((n_units + kScanWaves - 1) / kScanWaves, (uint64_t)device_cus());
            hipLaunchKernelGGL(objscan_kernel, dim3((uint32_t)grid), dim3(kScanBlock), scan_lds_bytes(nb), s,
                               reinterpret_cast<const uint4 *>(d_db), order, rec, toff + n_obj, n_obj,
                               reinterpret_cast<const uint4 *>(qb), nb, minK);
            if (hipGetLastError() != hipSuccess) return done(fail(QD_ERR_DEVICE, "object scan launch failed"));
        }
        {
            KernelTimer timer("object_sum", s);
            const uint64_t pairs = (uint64_t)(nqo < nb ? nqo : nb + 1) * n_obj;  // query objects overlapping the batch
            hipLaunchKernelGGL(score_sum_kernel, dim3(blocks_for(pairs, cap * 4)), dim3(kBlock), 0, s, minK, qpop, d0,
                               nb, d_qoff, nqo, roff, n_obj, d_scores);
            if (hipGetLastError() != hipSuccess) return done(fail(QD_ERR_DEVICE, "score sum launch failed"));
        }
    }
    return done(QD_OK);
}

extern "C" int qd_score_rows(double *d_scores, uint32_t nqo, uint32_t n_obj, int normalize, int32_t *d_best,
                             void *stream) {
    using namespace qd;
    clear_error();
    if (nqo == 0) return QD_OK;
    if (n_obj < 1) return fail(QD_ERR_INVALID, "n_obj=0");
    if (!d_scores || !d_best) return fail(QD_ERR_INVALID, "null pointer");
    hipStream_t s = (hipStream_t)stream;
    const uint32_t cap = (uint32_t)device_cus() * 16;
    KernelTimer timer("score_rows", s);
    hipLaunchKernelGGL(score_rows_kernel, dim3(nqo < cap ? nqo : cap), dim3(kBlock), 0, s, d_scores, nqo, n_obj,
                       normalize ? 1 : 0, d_best);
    QD_HIP_CHECK(hipGetLastError());
    return QD_OK;
}

