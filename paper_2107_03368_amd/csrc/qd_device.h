// Wavefront-level helpers for gfx950 (64-lane waves).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qd.h"

namespace qd {

typedef unsigned long long u64;

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ u64 ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Set bits of mask in the lanes below this one (a lane's rank among the set lanes).
__device__ __forceinline__ uint32_t lanes_below(u64 mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint32_t readlane(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ u64 readlane64(u64 v, int l) {
    return (u64)readlane((uint32_t)v, l) | ((u64)readlane((uint32_t)(v >> 32), l) << 32);
}
__device__ __forceinline__ uint32_t readfirst(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// v_writelane_b32: `old` with lane l's value replaced by the uniform `v`.
__device__ int write_lane(int v, int l, int old) __asm("llvm.amdgcn.writelane.i32");

// v from lane (lane - 1); lane 0 keeps its own value.
__device__ __forceinline__ u64 shift_up64(u64 v) {
    int l = lane_id();
    int src = (l > 0 ? l - 1 : 0) << 2;
    uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)v);
    uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)(v >> 32));
    return (u64)lo | ((u64)hi << 32);
}

// Sum over each aligned group of 8 lanes; every lane of the group gets the sum.
// DPP: quad_perm [1,0,3,2], quad_perm [2,3,0,1], then row_half_mirror
// (lane i <-> 7-i inside 8 lanes, which pairs the two quads).
__device__ __forceinline__ uint32_t sum8(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);
    return v;
}

// Sum over each 32-lane half of the wave; every lane gets its half's sum.
__device__ __forceinline__ uint32_t sum32_half(uint32_t v) {
    v = sum8(v);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row_mirror (16 lanes)
    v += (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);             // xor 16 within 32
    return v;
}

// Float sum over the wave in a fixed butterfly order (every lane gets it).
__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

__device__ __forceinline__ uint32_t popc4(uint4 a) {
    return __popc(a.x) + __popc(a.y) + __popc(a.z) + __popc(a.w);
}
__device__ __forceinline__ uint32_t popc_and4(uint4 a, uint4 b) {
    return __popc(a.x & b.x) + __popc(a.y & b.y) + __popc(a.z & b.z) + __popc(a.w & b.w);
}

// Insert candidate c into a sorted k-list held one entry per lane (lane r has
// the r-th smallest; unused slots and lanes >= k hold KEY_NONE).  Requires c
// to be smaller than the k-th entry.
__device__ __forceinline__ u64 list_insert(u64 e, u64 c, uint32_t k) {
    const u64 none = ~0ull;
    int l = lane_id();
    int pos = __popcll(ballot(e < c));
    u64 up = shift_up64(e);
    u64 r = l < pos ? e : (l == pos ? c : up);
    return l < (int)k ? r : none;
}

// Ascending bitonic sort of n (a power of two) keys in LDS by the whole block.
// Must be entered by every thread after the keys are written and synced.
__device__ inline void block_bitonic_sort(u64 *a, uint32_t n) {
    for (uint32_t size = 2; size <= n; size <<= 1)
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            for (uint32_t t = threadIdx.x; t < n / 2; t += blockDim.x) {
                uint32_t lo = 2 * t - (t & (stride - 1));
                uint32_t hi = lo + stride;
                bool up = (lo & size) == 0;
                u64 x = a[lo], y = a[hi];
                if ((x > y) == up) {
                    a[lo] = y;
                    a[hi] = x;
                }
            }
            __syncthreads();
        }
}

__device__ __forceinline__ uint32_t next_pow2(uint32_t v) {
    uint32_t p = 1;
    while (p < v) p <<= 1;
    return p;
}

// Ascending order of a[0 .. n) in place, n <= the block's threads: every thread
// finds its entry's rank by counting (ties by position), so it takes two
// barriers where a sorting network takes one per step.
__device__ __forceinline__ void rank_sort(u64 *a, uint32_t n) {
    const uint32_t i = threadIdx.x;
    const u64 mine = i < n ? a[i] : 0;
    uint32_t rank = 0;
    if (i < n)
        for (uint32_t j = 0; j < n; j++) rank += a[j] < mine || (a[j] == mine && j < i);
    __syncthreads();
    if (i < n) a[rank] = mine;
    __syncthreads();
}

// A query's results from its sorted keys (K << 32 | row; keys[0 .. nc) in LDS,
// the ranks past them padded) by the whole block: 8 lanes per result row.
// q4, db4: the query's and the database's rows; out[o0 + rank].
__device__ __forceinline__ void emit_rows(const u64 *keys, uint32_t nc, uint32_t k, const uint4 *q4, const uint4 *db4,
                                          uint64_t o0, uint32_t *idx, int32_t *missed, int32_t *extra, float *dist) {
    const int j = lane_id() & 7;
    uint4 qv[4];
    uint32_t pq = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        qv[i] = q4[j + 8 * i];
        pq += popc4(qv[i]);
    }
    pq = sum8(pq);
    const uint32_t wa = pq > 1 ? pq : 1, wb = (QD_BITS - pq) > 1 ? QD_BITS - pq : 1;
    for (uint32_t r = threadIdx.x >> 3; r < k; r += blockDim.x >> 3) {  // the same r in 8 lanes
        const bool none = r >= nc;
        const uint32_t row = none ? 0 : (uint32_t)keys[r];
        uint32_t c = 0, tp = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint4 t = db4[(uint64_t)row * 32 + j + 8 * i];
            c += popc_and4(t, qv[i]);
            tp += popc4(t);
        }
        c = sum8(c);
        tp = sum8(tp);
        if (j != 0) continue;
        const uint32_t a = pq - c, b = tp - c, K = a * wb + b * wa;
        idx[o0 + r] = none ? QD_PAD_IDX : row;
        missed[o0 + r] = none ? -1 : (int32_t)a;
        extra[o0 + r] = none ? -1 : (int32_t)b;
        dist[o0 + r] = none ? __builtin_inff() : (float)((double)K / ((double)wa * (double)wb));
    }
}

}  // namespace qd
