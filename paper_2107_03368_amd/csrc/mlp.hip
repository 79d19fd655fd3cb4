// Learned frontier order: a small MLP that scores (query, tree node) pairs,
// with hand-written BF16 kernels (FP32 accumulation) for inference and
// training.  The score only decides which child the depth-first search visits
// first; pruning uses the exact bounds, so results never depend on it.
//
// Network: x = [query bits (4096, 0/1); node features f (32)]
//   h1 = ReLU(x W1 + b1)      W1 = [W1q (4096 x 256); W1f (32 x 256)]
//   h2 = ReLU(h1 W2 + b2)     W2: 256 x 256
//   s  = h2 . w3 + b3
// All weight matrices are stored [input][output].  Because the query part of
// x is binary and shared by every node scored for that query, u_q = b1 +
// sum over the query's set bits of the W1q rows is formed once per query (a
// gather-add); a pair then costs u_q + f W1f (32 x 256, fp32), the 256 x 256
// layer in BF16 and the 256-wide head, all in one kernel per batch of pairs
// (mlp_forward_kernel): nothing of a pair's activations goes through memory.
// The layer-1 activations enter the BF16 product as two BF16 terms (hi + lo,
// with lo the rounding residual), so only the weights are rounded to BF16.
// Training (binary cross-entropy on the logit, mean over pairs): the forward
// kernel keeps the layer-1 terms and, per pair, the logit's gradient ds and
// one bit per hidden unit of either layer (was it positive), from which the
// two backward kernels form d2 = ds w3 [h2 > 0] where they need it.  Every
// reduction has a fixed order, so gradients are reproducible bit for bit.
// Parameters are FP32 masters with Adam moments; each update refreshes their
// BF16 copies.
#include <math.h>

#include <algorithm>
#include <vector>

#include "qd_device.h"
#include "qd_internal.h"
#include "qd_tree.h"

struct qd_model_s {
    int device = 0;
    float *p = nullptr;      // QD_MLP_NPARAMS fp32 master parameters
    float *m = nullptr;      // Adam first moments
    float *v = nullptr;      // Adam second moments
    uint16_t *w = nullptr;   // bf16 copy of p (same layout)
    uint16_t *w2t = nullptr;  // bf16 W2 transposed ([output][input]): the layer-2 operand, 16 bytes per lane
    uint64_t step = 0;
};

namespace qd {
namespace {

constexpr int kBlock = 256;
constexpr int H = QD_MLP_HIDDEN;
constexpr int NF = QD_MLP_FEATURES;
constexpr size_t OFF_W1Q = 0;
constexpr size_t OFF_W1F = OFF_W1Q + (size_t)QD_BITS * H;
constexpr size_t OFF_B1 = OFF_W1F + (size_t)NF * H;
constexpr size_t OFF_W2 = OFF_B1 + H;
constexpr size_t OFF_B2 = OFF_W2 + (size_t)H * H;
constexpr size_t OFF_W3 = OFF_B2 + H;
constexpr size_t OFF_B3 = OFF_W3 + H;
static_assert(OFF_B3 + 1 == QD_MLP_NPARAMS, "parameter layout");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
// float -> bf16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// Two floats to two bf16 (round to nearest even) in one word.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    uint32_t r;
    __builtin_memcpy(&r, &v, 4);
    return r;
}

// Sum over each row of 16 lanes (every lane of the row gets it).
__device__ __forceinline__ float sum16(float v) {
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, false));  // row_half_mirror
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, false));  // row_mirror
    return v;
}

// ---------------------------------------------------------------------------
// Node features for (query, node) pairs.  Pair p is (pair_q[p], pair_node[p]),
// or, with null pair arrays, (q0 + p / n_nodes_per_q, p % n_nodes_per_q).
// Features (|q| read as max(|q|,1); a_lb = popcount(q AND NOT OR),
// ov = popcount(q AND OR); bands = image rows 0-5, 6-11, ..., 54-59, 60-63):
//   0 a_lb/|q|  1 ov/|q|  2 popcount(OR)/4096  3 sibling's a_lb/|q| (0 at the
//   root)  4 depth/32  5 log2(rows under the node)/24  6 is leaf
//   7 is the similar child  8 |q|/512  9 popcount(OR AND NOT q)/4096
//   10..20 band a_lb/|q|  21..31 band ov/|q|
// Two pairs per wave, one per 32-lane half; lane c of a half holds the
// 16-byte chunk c (image rows 2c, 2c+1).
// ---------------------------------------------------------------------------
struct PairIdx {
    const uint32_t *pq, *pn;
    uint32_t q0, per_q;
    __device__ __forceinline__ uint32_t q(uint64_t p) const { return pq ? pq[p] : q0 + (uint32_t)(p / per_q); }
    __device__ __forceinline__ uint32_t node(uint64_t p) const { return pn ? pn[p] : (uint32_t)(p % per_q); }
};

__global__ __launch_bounds__(kBlock) void features_kernel(const uint4 *__restrict__ q, const uint4 *__restrict__ orimg,
                                                          const int32_t *__restrict__ child,
                                                          const int32_t *__restrict__ parent,
                                                          const uint8_t *__restrict__ depth,
                                                          const uint32_t *__restrict__ count, PairIdx P,
                                                          uint64_t n_pairs, float *__restrict__ feat) {
    __shared__ uint32_t band_a[kBlock / 32][32], band_o[kBlock / 32][32];
    const int half = threadIdx.x >> 5, c = threadIdx.x & 31;
    const uint64_t p = (uint64_t)blockIdx.x * (kBlock / 32) + half;
    const bool live = p < n_pairs;
    const uint64_t pp = live ? p : 0;
    const uint32_t qi = P.q(pp), node = P.node(pp);
    const int32_t par = parent[node];
    const int32_t sib = par < 0 ? -1 : (child[2 * par] == (int32_t)node ? child[2 * par + 1] : child[2 * par]);
    const uint4 qv = q[(uint64_t)qi * 32 + c];
    const uint4 ov = orimg[(uint64_t)node * 32 + c];
    const uint4 sv = sib >= 0 ? orimg[(uint64_t)sib * 32 + c] : make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
    // rows 2c (x, y) and 2c+1 (z, w)
    const uint32_t a0 = __popc(qv.x & ~ov.x) + __popc(qv.y & ~ov.y), a1 = __popc(qv.z & ~ov.z) + __popc(qv.w & ~ov.w);
    const uint32_t o0 = __popc(qv.x & ov.x) + __popc(qv.y & ov.y), o1 = __popc(qv.z & ov.z) + __popc(qv.w & ov.w);
    band_a[half][c] = a0 + a1;
    band_o[half][c] = o0 + o1;
    const uint32_t pq = sum32_half(popc4(qv));
    const uint32_t a_lb = sum32_half(a0 + a1);
    const uint32_t ovl = sum32_half(o0 + o1);
    const uint32_t orp = sum32_half(popc4(ov));
    const uint32_t extra = sum32_half(__popc(ov.x & ~qv.x) + __popc(ov.y & ~qv.y) + __popc(ov.z & ~qv.z) +
                                      __popc(ov.w & ~qv.w));
    const uint32_t sib_a = sum32_half(__popc(qv.x & ~sv.x) + __popc(qv.y & ~sv.y) + __popc(qv.z & ~sv.z) +
                                      __popc(qv.w & ~sv.w));
    __syncthreads();
    if (!live) return;
    const float inv = 1.0f / (float)(pq > 1 ? pq : 1);
    float *f = feat + p * NF;
    if (c == 0) {
        f[0] = (float)a_lb * inv;
        f[1] = (float)ovl * inv;
        f[2] = (float)orp * (1.0f / 4096.0f);
        f[3] = sib >= 0 ? (float)sib_a * inv : 0.0f;
        f[4] = (float)depth[node] * (1.0f / 32.0f);
        f[5] = log2f((float)count[node]) * (1.0f / 24.0f);
        f[6] = child[2 * node] < 0 ? 1.0f : 0.0f;
        f[7] = (par >= 0 && child[2 * par] == (int32_t)node) ? 1.0f : 0.0f;
        f[8] = (float)pq * (1.0f / 512.0f);
        f[9] = (float)extra * (1.0f / 4096.0f);
    }
    if (c < 11) {
        // band c covers chunks 3c .. 3c+2 (the last band chunks 30, 31)
        const int c0 = 3 * c, c1 = c == 10 ? 32 : 3 * c + 3;
        uint32_t sa = 0, so = 0;
        for (int i = c0; i < c1; i++) {
            sa += band_a[half][i];
            so += band_o[half][i];
        }
        f[10 + c] = (float)sa * inv;
        f[21 + c] = (float)so * inv;
    }
}

// u[qi][j] = b1[j] + sum over set bits b of query q0+qi of W1q[b][j] (bf16
// weights; bits summed in ascending order).  One block per query; the loop's
// loads do not depend on its sums, so several are in flight.
__global__ __launch_bounds__(kBlock) void uq_kernel(const uint64_t *__restrict__ q, uint32_t q0,
                                                    const uint16_t *__restrict__ w, float *__restrict__ u) {
    __shared__ uint16_t bits[QD_BITS];
    __shared__ uint32_t s_nb;
    const uint64_t *qq = q + (uint64_t)(q0 + blockIdx.x) * QD_WORDS;
    const int t = threadIdx.x;
    if (t < 64) {
        uint64_t x = qq[t];
        const uint32_t c = (uint32_t)__popcll(x);
        uint32_t incl = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)incl, d);
            incl += t >= d ? v : 0u;
        }
        uint32_t o = incl - c;
        while (x) {
            bits[o++] = (uint16_t)(64 * t + __builtin_ctzll(x));
            x &= x - 1;
        }
        if (t == 63) s_nb = incl;
    }
    __syncthreads();
    float acc = bf2f(w[OFF_B1 + t]);
    const uint32_t nb = s_nb;
    uint32_t i = 0;
    for (; i + 8 <= nb; i += 8) {
        uint16_t x[8];
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] = w[OFF_W1Q + (size_t)bits[i + e] * H + t];
#pragma unroll
        for (int e = 0; e < 8; e++) acc += bf2f(x[e]);
    }
    for (; i < nb; i++) acc += bf2f(w[OFF_W1Q + (size_t)bits[i] * H + t]);
    u[(size_t)blockIdx.x * H + t] = acc;
}

// ---------------------------------------------------------------------------
// The fused MLP kernels.  Work comes in tiles of TP = 64 pairs, four matrix
// tiles of 16 rows each; a workgroup of 8 waves serves a tile and wave w owns
// the hidden units 32w .. 32w+31, two column blocks of 16 (block nb = 2w + n).
// Matrix tiles (lane l, li = l % 16, lg = l / 16): the operands hold row (or
// column) li at k = 8 lg .. +7 (bf16, depth 32) or k = lg (fp32, depth 4);
// the result holds rows 4 lg + r, r = 0..3, of column li.  So a lane's result
// entry (m, n, r) belongs to pair 16 m + 4 lg + r and unit 16 nb + li, and
//  - a bit per (pair, unit) is kept as one ballot per (m, r, nb): a word whose
//    bit l is the lane's own, which a later kernel in the same layout uses as
//    a lane mask without any bit work (kMaskWords words per tile);
//  - the k index of a product over pairs is theirs to permute, the same for
//    both operands: k = 8 lg + 4 (m % 2) + r is a lane's own 8 entries of two
//    matrix tiles, so the layer-1 terms are stored as the operand of dW2 =
//    h1^T d2 with no transposition, 16 bytes per lane (h1t: per half tile of
//    32 pairs, hi and lo, 16 column blocks, 64 lanes), and k = lg of step
//    (m, r) makes dz's own registers the operand of the fp32 product
//    dW1f = f^T dz.
// ---------------------------------------------------------------------------
constexpr int kMlpBlock = 512;
constexpr int TP = 64;
constexpr int kMT = TP / 16;                      // matrix tiles of rows per tile
constexpr uint32_t kMaskWords = kMT * 4 * (H / 16);  // ballots of a tile: word (m * 4 + r) * 16 + nb
constexpr int kHaStride = 2 * H + 8;              // bf16 per row of layer-1 terms in LDS (hi, lo, pad)
constexpr uint32_t kHeadPartLen = 2 * H + 2;      // per workgroup: sum ds h2 [H], sum ds [h2 > 0] [H], sum ds, sum loss

__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 load_frag(const uint16_t *p) {
    bf16x8 v;
    const uint4 x = *reinterpret_cast<const uint4 *>(p);
    __builtin_memcpy(&v, &x, 16);
    return v;
}
// lane l's entry of a word held in the scalar registers
__device__ __forceinline__ void put_lane(uint32_t &lo, uint32_t &hi, u64 word, int l) {
    lo = (uint32_t)write_lane((int)(uint32_t)word, l, (int)lo);
    hi = (uint32_t)write_lane((int)(uint32_t)(word >> 32), l, (int)hi);
}

// Scores (s_out) or, with kTrain, everything the backward kernels need: the
// layer-1 terms h1t, the masks m1 = [h1 > 0] and m2 = [h2 > 0], ds[p] =
// (sigmoid(s) - y) / n_pairs and this workgroup's head sums (part).  Pairs
// past n_pairs count as zero rows.
// Bound by the matrix cores (per pair 256 x 32 in fp32 and 2 x 256 x 256 in
// bf16) with the vector work between them; W2 stays in registers (64 per
// lane), the next tile's features and layer-1 sums are loaded during this
// tile's second layer.  1,048,064 pairs of 512 queries: 0.83 ms, against
// 3.2 ms for a layer-1, a GEMM and a head kernel with the activations in
// memory between them; in training 307,000 pairs 0.32 ms against 1.07 ms.
template <bool kTrain>
__global__ __launch_bounds__(kMlpBlock, 2) void mlp_forward_kernel(
    const float *__restrict__ u, PairIdx P, uint32_t q0, const float *__restrict__ feat, uint64_t n_pairs,
    const uint16_t *__restrict__ w, const uint16_t *__restrict__ w2t, const float *__restrict__ y,
    float *__restrict__ s_out, uint4 *__restrict__ h1t, u64 *__restrict__ m1, u64 *__restrict__ m2,
    float *__restrict__ ds_out, float *__restrict__ part) {
    __shared__ __align__(16) uint16_t ha[TP * kHaStride];
    __shared__ float s_sum[kMlpBlock / 64][TP];  // per wave: its units' part of every pair's logit
    const int lane = threadIdx.x & 63, wv = (int)readfirst(threadIdx.x >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int col = 32 * wv + li;  // this lane's unit of column block n: col + 16 n
    bf16x8 b2f[8][2];
    float w1[8][2], b2[2], w3[2];
#pragma unroll
    for (int n = 0; n < 2; n++) {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            b2f[k][n] = load_frag(w2t + (size_t)(col + 16 * n) * H + 32 * k + 8 * lg);
            w1[k][n] = bf2f(w[OFF_W1F + (size_t)(4 * k + lg) * H + col + 16 * n]);
        }
        b2[n] = bf2f(w[OFF_B2 + col + 16 * n]);
        w3[n] = bf2f(w[OFF_W3 + col + 16 * n]);
    }
    const float b3 = bf2f(w[OFF_B3]);
    const uint64_t tiles = (n_pairs + TP - 1) / TP;

    // loads of one tile: features as the left operand, the queries of this
    // lane's result rows, then their layer-1 sums as the accumulators' start
    float f[8][kMT];
    uint32_t qr[kMT][4];
    f32x4 acc[kMT][2];
    auto load_f = [&](uint64_t t) {
#pragma unroll
        for (int m = 0; m < kMT; m++) {
            uint64_t p = t * TP + 16 * m + li;
            p = p < n_pairs ? p : n_pairs - 1;
#pragma unroll
            for (int k = 0; k < 8; k++) f[k][m] = feat[p * NF + 4 * k + lg];
        }
    };
    auto load_q = [&](uint64_t t) {
        if (P.pq) {
#pragma unroll
            for (int m = 0; m < kMT; m++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    uint64_t p = t * TP + 16 * m + 4 * lg + r;
                    p = p < n_pairs ? p : n_pairs - 1;
                    qr[m][r] = P.pq[p] - q0;
                }
        } else {  // pair p belongs to query q0 + p / per_q
            const uint64_t p0 = t * TP;
            const uint32_t qb = P.q0 - q0 + (uint32_t)(p0 / P.per_q), rem = (uint32_t)(p0 % P.per_q);
            const uint32_t last = (uint32_t)(n_pairs - 1 - p0 < TP - 1 ? n_pairs - 1 - p0 : TP - 1);
#pragma unroll
            for (int m = 0; m < kMT; m++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    uint32_t e = 16 * m + 4 * lg + r;
                    e = rem + (e < last ? e : last);
                    // (a tile of 64 pairs meets a few queries at most unless per_q is small)
                    qr[m][r] = qb + (e < P.per_q ? 0u : P.per_q >= TP ? 1u : e / P.per_q);
                }
        }
    };
    auto load_u = [&]() {
#pragma unroll
        for (int m = 0; m < kMT; m++)
#pragma unroll
            for (int n = 0; n < 2; n++)
#pragma unroll
                for (int r = 0; r < 4; r++) acc[m][n][r] = u[(size_t)qr[m][r] * H + col + 16 * n];
    };
    float ga[2] = {0.f, 0.f}, gb[2] = {0.f, 0.f}, sd = 0.f, sl = 0.f;
    uint64_t t = blockIdx.x;
    if (t < tiles) {
        load_q(t);
        load_f(t);
        load_u();
    }
    for (; t < tiles; t += gridDim.x) {
        const uint64_t p0 = t * TP;
        const uint32_t live = (uint32_t)(n_pairs - p0 < TP ? n_pairs - p0 : TP);
        // layer 1: z = u + f W1f
#pragma unroll
        for (int k = 0; k < 8; k++)
#pragma unroll
            for (int m = 0; m < kMT; m++)
#pragma unroll
                for (int n = 0; n < 2; n++) acc[m][n] = mfma_f32(f[k][m], w1[k][n], acc[m][n]);
        uint64_t tn = t + gridDim.x;
        tn = tn < tiles ? tn : t;  // after the last tile: this one again, unused
        load_q(tn);
        // h = ReLU(z) as two bf16 terms: to LDS (rows of pairs) and, in
        // training, out as the operand of dW2
        uint32_t klo = 0, khi = 0;
#pragma unroll
        for (int n = 0; n < 2; n++)
#pragma unroll
            for (int m = 0; m < kMT; m++) {
                uint32_t hp[2], lp[2];
#pragma unroll
                for (int r = 0; r < 4; r += 2) {
                    float h[2];
#pragma unroll
                    for (int e = 0; e < 2; e++) {
                        const float z = acc[m][n][r + e];
                        h[e] = z > 0.f && (uint32_t)(16 * m + 4 * lg + r + e) < live ? z : 0.f;
                    }
                    hp[r / 2] = pack_bf16(h[0], h[1]);
                    lp[r / 2] = pack_bf16(h[0] - __uint_as_float(hp[r / 2] << 16),
                                          h[1] - __uint_as_float(hp[r / 2] & 0xFFFF0000u));
                    uint16_t *a0 = ha + (16 * m + 4 * lg + r) * kHaStride + col + 16 * n, *a1 = a0 + kHaStride;
                    a0[0] = (uint16_t)hp[r / 2];
                    a1[0] = (uint16_t)(hp[r / 2] >> 16);
                    a0[H] = (uint16_t)lp[r / 2];
                    a1[H] = (uint16_t)(lp[r / 2] >> 16);
                    if (kTrain) {
                        const float g0 = __uint_as_float(hp[r / 2] << 16), g1 = __uint_as_float(hp[r / 2] & 0xFFFF0000u);
                        put_lane(klo, khi, ballot(g0 > 0.f), (m * 4 + r) * 2 + n);
                        put_lane(klo, khi, ballot(g1 > 0.f), (m * 4 + r + 1) * 2 + n);
                    }
                }
                if (kTrain) {  // 8 bytes of the lane's 16: the other matrix tile of the half fills the rest
                    uint2 *o = reinterpret_cast<uint2 *>(
                        h1t + (((2 * t + m / 2) * 2) * (H / 16) + 2 * wv + n) * 64 + lane) + (m & 1);
                    o[0] = make_uint2(hp[0], hp[1]);
                    o[2 * (H / 16) * 64] = make_uint2(lp[0], lp[1]);
                }
            }
        if (kTrain && lane < 8 * kMT)
            m1[t * kMaskWords + (lane >> 1) * (H / 16) + 2 * wv + (lane & 1)] = (u64)klo | ((u64)khi << 32);
        __syncthreads();
        // layer 2: the hi terms' product, then the lo terms'
        load_u();  // the next tile's start, into the accumulators layer 1 just left
        load_f(tn);
        f32x4 z2[kMT][2];
#pragma unroll
        for (int m = 0; m < kMT; m++)
#pragma unroll
            for (int n = 0; n < 2; n++) z2[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 16; k++) {
            bf16x8 a[kMT];
#pragma unroll
            for (int m = 0; m < kMT; m++) a[m] = load_frag(ha + (16 * m + li) * kHaStride + 32 * k + 8 * lg);
#pragma unroll
            for (int m = 0; m < kMT; m++)
#pragma unroll
                for (int n = 0; n < 2; n++) z2[m][n] = mfma_bf16(a[m], b2f[k & 7][n], z2[m][n]);
        }
        // h2 and this wave's part of the logits
#pragma unroll
        for (int m = 0; m < kMT; m++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                float v = 0.f;
#pragma unroll
                for (int n = 0; n < 2; n++) {
                    const float zz = z2[m][n][r] + b2[n];
                    z2[m][n][r] = zz > 0.f ? zz : 0.f;
                    v += z2[m][n][r] * w3[n];
                }
                v = sum16(v);
                if (li == 0) s_sum[wv][16 * m + 4 * lg + r] = v;
            }
        __syncthreads();
        // lane l: pair l of the tile (the same in every wave)
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < kMlpBlock / 64; v++) s += s_sum[v][lane];
        s += b3;
        const bool ok = (uint32_t)lane < live;
        if (!kTrain) {
            if (wv == 0 && ok) s_out[p0 + lane] = s;
            continue;
        }
        const float yy = y[p0 + (ok ? lane : 0)];
        const float ds = ok ? (1.f / (1.f + expf(-s)) - yy) / (float)n_pairs : 0.f;
        if (wv == 0) {
            ds_out[p0 + lane] = ds;
            sd += ds;
            sl += ok ? (s > 0.f ? s + log1pf(expf(-s)) : log1pf(expf(s))) - yy * s : 0.f;
        }
        klo = khi = 0;
#pragma unroll
        for (int m = 0; m < kMT; m++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const uint32_t e = 16 * m + 4 * lg + r;
                const float d = __shfl(ds, (int)e);
#pragma unroll
                for (int n = 0; n < 2; n++) {
                    const bool on = z2[m][n][r] > 0.f && e < live;
                    ga[n] += on ? d * z2[m][n][r] : 0.f;
                    gb[n] += on ? d : 0.f;
                    put_lane(klo, khi, ballot(on), (m * 4 + r) * 2 + n);
                }
            }
        if (lane < 8 * kMT)
            m2[t * kMaskWords + (lane >> 1) * (H / 16) + 2 * wv + (lane & 1)] = (u64)klo | ((u64)khi << 32);
    }
    if (!kTrain) return;
    float *o = part + (size_t)blockIdx.x * kHeadPartLen;
#pragma unroll
    for (int n = 0; n < 2; n++) {
        ga[n] += __shfl_xor(ga[n], 16);
        ga[n] += __shfl_xor(ga[n], 32);
        gb[n] += __shfl_xor(gb[n], 16);
        gb[n] += __shfl_xor(gb[n], 32);
        if (lg == 0) {
            o[col + 16 * n] = ga[n];
            o[H + col + 16 * n] = gb[n];
        }
    }
    if (wv == 0) {
        sd = wave_sum_f(sd);
        sl = wave_sum_f(sl);
        if (lane == 0) {
            o[2 * H] = sd;
            o[2 * H + 1] = sl;
        }
    }
}

// This lane's bf16 entries d2 = ds w3 [h2 > 0] of one unit for the 8 pairs
// (m0, r), (m0 + 1, r) of a half tile: word (m, r) of `m2` is its lane mask.
__device__ __forceinline__ uint4 d2_frag(const float (&d)[2][4], float w3, const u64 (&mask)[2][4]) {
    uint32_t o[4];
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
            const float a = __builtin_amdgcn_inverse_ballot_w64(mask[m][r]) ? d[m][r] * w3 : 0.f;
            const float b = __builtin_amdgcn_inverse_ballot_w64(mask[m][r + 1]) ? d[m][r + 1] * w3 : 0.f;
            o[m * 2 + r / 2] = pack_bf16(a, b);
        }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// dW2 = (h1_hi + h1_lo)^T d2, summed over the tiles blockIdx.x, + gridDim.x,
// ...: part[blockIdx.x][256][256].  Wave w owns rows 32w .. +31 of dW2 (128
// accumulators per lane) and forms d2's column blocks 2w, 2w + 1 for all the
// waves in LDS (two copies: the next half tile's are written while this one's
// are read).  Bound by reading h1t once (1 KB per pair); splitting the sum
// over the pairs one workgroup per CU keeps the whole chip on it, where one
// workgroup per 64 x 64 tile of dW2 filled 16 CUs: 307,000 pairs 0.10 ms
// (4.8 TB/s) against 11.5 ms, and 0.01 ms for the sum of the parts.
__global__ __launch_bounds__(kMlpBlock, 2) void dw2_kernel(const uint4 *__restrict__ h1t, const u64 *__restrict__ m2,
                                                           const float *__restrict__ ds,
                                                           const uint16_t *__restrict__ w, uint64_t tiles,
                                                           float *__restrict__ part) {
    __shared__ __align__(16) uint4 s_d2[2][(H / 16) * 64];
    const int lane = threadIdx.x & 63, wv = (int)readfirst(threadIdx.x >> 6);
    const int li = lane & 15, lg = lane >> 4;
    float w3[2];
#pragma unroll
    for (int n = 0; n < 2; n++) w3[n] = bf2f(w[OFF_W3 + 32 * wv + 16 * n + li]);
    f32x4 acc[2][H / 16];
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < H / 16; b++) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // half tile x: pairs 32x .. 32x+31
    const uint64_t halves = 2 * tiles;
    auto half_of = [&](uint64_t i) { return 2 * (blockIdx.x + (i >> 1) * gridDim.x) + (i & 1); };
    uint4 a_next[2][2];  // [hi, lo][row block]
    float d[2][4];
    u64 mask[2][2][4];   // [n][m][r]
    auto fetch = [&](uint64_t x) {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int a = 0; a < 2; a++)
                a_next[h][a] = h1t[((x * 2 + h) * (H / 16) + 2 * wv + a) * 64 + lane];
#pragma unroll
        for (int m = 0; m < 2; m++) {
            const float4 v = *reinterpret_cast<const float4 *>(ds + x * 32 + 16 * m + 4 * lg);
            d[m][0] = v.x;
            d[m][1] = v.y;
            d[m][2] = v.z;
            d[m][3] = v.w;
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll
                for (int n = 0; n < 2; n++)
                    mask[n][m][r] = m2[(x >> 1) * kMaskWords + ((2 * (x & 1) + m) * 4 + r) * (H / 16) + 2 * wv + n];
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int n = 0; n < 2; n++) s_d2[buf][(2 * wv + n) * 64 + lane] = d2_frag(d, w3[n], mask[n]);
    };
    uint64_t i = 0;
    uint64_t x = half_of(0);
    if (x < halves) {
        fetch(x);
        put(0);
    }
    __syncthreads();
    for (; x < halves; i++) {
        bf16x8 a[2][2];
        __builtin_memcpy(a, a_next, sizeof a);
        const uint64_t xn = half_of(i + 1);
        fetch(xn < halves ? xn : x);
        const int buf = (int)(i & 1);
#pragma unroll
        for (int b = 0; b < H / 16; b++) {
            const bf16x8 bv = load_frag(reinterpret_cast<const uint16_t *>(&s_d2[buf][b * 64 + lane]));
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int q = 0; q < 2; q++) acc[q][b] = mfma_bf16(a[h][q], bv, acc[q][b]);
        }
        put(buf ^ 1);  // read by every wave before the previous barrier
        __syncthreads();
        x = xn;
    }
    float *o = part + (size_t)blockIdx.x * H * H;
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < H / 16; b++)
#pragma unroll
            for (int r = 0; r < 4; r++) o[(size_t)(32 * wv + 16 * a + 4 * lg + r) * H + 16 * b + li] = acc[a][b][r];
}

// g[W2] = the sum of the n parts, row blockIdx.x: each of 4 waves sums a
// quarter of the parts (4 floats per lane), then the quarters in order.
__global__ __launch_bounds__(kBlock) void dw2_sum_kernel(const float *__restrict__ part, uint32_t n,
                                                         float *__restrict__ g) {
    __shared__ float4 s_q[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t per = (n + 3) / 4, k0 = wv * per, k1 = k0 + per < n ? k0 + per : n;
    const float4 *p = reinterpret_cast<const float4 *>(part) + (size_t)blockIdx.x * (H / 4) + lane;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (uint32_t k = k0; k < k1; k++) {
        const float4 v = p[(size_t)k * (H * H / 4)];
        a.x += v.x;
        a.y += v.y;
        a.z += v.z;
        a.w += v.w;
    }
    s_q[wv][lane] = a;
    __syncthreads();
    if (wv != 0) return;
    for (int v = 1; v < 4; v++) {
        a.x += s_q[v][lane].x;
        a.y += s_q[v][lane].y;
        a.z += s_q[v][lane].z;
        a.w += s_q[v][lane].w;
    }
    float *o = g + OFF_W2 + (size_t)blockIdx.x * H + 4 * lane;
    o[0] = a.x;
    o[1] = a.y;
    o[2] = a.z;
    o[3] = a.w;
}

// dz = (d2 W2^T) [h1 > 0]; then g[W1F] = f^T dz, g[B1] = sum dz and du[q] = the
// sum of dz over query q's pairs (pairs are grouped by query).  Block (q, c)
// sums chunk c of query q's pairs: part[block] = (32 feature rows, sum dz) x
// 256.  It walks the half tiles (32 pairs, as the masks are kept) its chunk
// meets; pairs outside the chunk are masked out.  Wave w owns units 32w ..
// +31 as everywhere here; d2 is formed once per half tile, as the left
// operand in LDS.  Bound by the chain of a half tile (d2, barrier, multiply), the
// next half tile's loads being in flight meanwhile (0.25 ms without); 307,000 pairs
// 0.21 ms against 0.63 ms for a GEMM and a reduction over its stored result.
constexpr uint32_t kL1PartLen = (NF + 1) * H;  // gf[NF][H], su[H]
// Chunks per query: enough blocks to fill the chip, more only for few queries,
// and none of less than 64 pairs on average (every chunk holds 34 KB of partial
// sums: 1 query of 10 pairs took 64 chunks and 2.6 MB, whose allocation made
// the call 0.105 ms instead of 0.079).
inline uint32_t l1_chunks(uint32_t nq, uint64_t n_pairs) {
    const uint64_t c = std::min<uint64_t>({64, (1024 + nq - 1) / nq, n_pairs / 64 / nq});
    return c < 1 ? 1 : (uint32_t)c;
}

__global__ __launch_bounds__(kMlpBlock, 2) void layer1_partial_kernel(
    const u64 *__restrict__ m1, const u64 *__restrict__ m2, const float *__restrict__ ds,
    const float *__restrict__ feat, const uint16_t *__restrict__ w, const uint64_t *__restrict__ qoff,
    uint64_t qoff_base, uint64_t n_pairs, uint32_t chunks, float *__restrict__ part) {
    constexpr int kStride = H + 8;
    __shared__ __align__(16) uint16_t s_d2[2][32 * kStride];
    const int lane = threadIdx.x & 63, wv = (int)readfirst(threadIdx.x >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int col = 32 * wv + li;
    const uint32_t qi = blockIdx.x / chunks, c = blockIdx.x % chunks;
    const uint64_t b0 = qoff[qi] - qoff_base, b1 = qoff[qi + 1] - qoff_base;
    const uint64_t chunk = (b1 - b0 + chunks - 1) / chunks;
    const uint64_t p0 = b0 + c * chunk < b1 ? b0 + c * chunk : b1;
    const uint64_t p1 = p0 + chunk < b1 ? p0 + chunk : b1;
    float su[2] = {0.f, 0.f}, w3[2];
    f32x4 gf[2][2];  // [feature block][column block]
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int n = 0; n < 2; n++) gf[a][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (p0 < p1) {
        bf16x8 wf[8][2];  // W2^T: column = unit of layer 1, k = unit of layer 2
#pragma unroll
        for (int n = 0; n < 2; n++) {
            w3[n] = bf2f(w[OFF_W3 + col + 16 * n]);
#pragma unroll
            for (int k = 0; k < 8; k++) wf[k][n] = load_frag(w + OFF_W2 + (size_t)(col + 16 * n) * H + 32 * k + 8 * lg);
        }
        // a half tile's ds and features (row = feature, k of step (m, r) = the
        // lane group's pair), fetched one half tile ahead
        float4 nd[2];
        float nf[2][2][4];
        auto fetch = [&](uint64_t x) {
#pragma unroll
            for (int m = 0; m < 2; m++) {
                nd[m] = *reinterpret_cast<const float4 *>(ds + x * 32 + 16 * m + 4 * lg);
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    uint64_t p = x * 32 + 16 * m + 4 * lg + r;
                    p = p < n_pairs ? p : n_pairs - 1;
#pragma unroll
                    for (int a = 0; a < 2; a++) nf[a][m][r] = feat[p * NF + 16 * a + li];
                }
            }
        };
        int buf = 0;
        fetch(p0 / 32);
        for (uint64_t x = p0 / 32; x * 32 < p1; x++, buf ^= 1) {
            // this lane's pairs (m, r) of the half tile that lie in the chunk
            u64 in[2][4];
            float d[2][4], f[2][2][4];
#pragma unroll
            for (int m = 0; m < 2; m++) {
                d[m][0] = nd[m].x;
                d[m][1] = nd[m].y;
                d[m][2] = nd[m].z;
                d[m][3] = nd[m].w;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const uint64_t p = x * 32 + 16 * m + 4 * lg + r;
                    in[m][r] = ballot(p >= p0 && p < p1);
#pragma unroll
                    for (int a = 0; a < 2; a++)
                        f[a][m][r] = __builtin_amdgcn_inverse_ballot_w64(in[m][r]) ? nf[a][m][r] : 0.f;
                }
            }
            fetch((x + 1) * 32 < p1 ? x + 1 : x);
            const u64 *w1m = m1 + (x >> 1) * kMaskWords + (x & 1) * 8 * (H / 16) + 2 * wv;
            const u64 *w2m = m2 + (x >> 1) * kMaskWords + (x & 1) * 8 * (H / 16) + 2 * wv;
            uint16_t *dst = s_d2[buf];
#pragma unroll
            for (int n = 0; n < 2; n++) {
                u64 mask[2][4];
#pragma unroll
                for (int m = 0; m < 2; m++)
#pragma unroll
                    for (int r = 0; r < 4; r++) mask[m][r] = w2m[(m * 4 + r) * (H / 16) + n] & in[m][r];
                const uint4 v = d2_frag(d, w3[n], mask);
                const uint32_t o[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; e++)  // entry e: pair 16 (e / 4) + 4 lg + e % 4
                    dst[(16 * (e >> 2) + 4 * lg + (e & 3)) * kStride + col + 16 * n] =
                        (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
            }
            u64 mk[2][2][4];  // h1 > 0, fetched while the multiplications run
#pragma unroll
            for (int m = 0; m < 2; m++)
#pragma unroll
                for (int r = 0; r < 4; r++)
#pragma unroll
                    for (int n = 0; n < 2; n++) mk[n][m][r] = w1m[(m * 4 + r) * (H / 16) + n];
            __syncthreads();  // (the other copy was read by every wave before this)
            f32x4 dz[2][2];
#pragma unroll
            for (int m = 0; m < 2; m++)
#pragma unroll
                for (int n = 0; n < 2; n++) dz[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 8; k++) {
                bf16x8 a[2];
#pragma unroll
                for (int m = 0; m < 2; m++) a[m] = load_frag(dst + (16 * m + li) * kStride + 32 * k + 8 * lg);
#pragma unroll
                for (int m = 0; m < 2; m++)
#pragma unroll
                    for (int n = 0; n < 2; n++) dz[m][n] = mfma_bf16(a[m], wf[k][n], dz[m][n]);
            }
#pragma unroll
            for (int m = 0; m < 2; m++)
#pragma unroll
                for (int r = 0; r < 4; r++)
#pragma unroll
                    for (int n = 0; n < 2; n++) {
                        const float v = __builtin_amdgcn_inverse_ballot_w64(mk[n][m][r] & in[m][r]) ? dz[m][n][r] : 0.f;
                        su[n] += v;
#pragma unroll
                        for (int a = 0; a < 2; a++) gf[a][n] = mfma_f32(f[a][m][r], v, gf[a][n]);
                    }
        }
    }
    float *o = part + (size_t)blockIdx.x * kL1PartLen;
#pragma unroll
    for (int n = 0; n < 2; n++) {
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int r = 0; r < 4; r++) o[(size_t)(16 * a + 4 * lg + r) * H + col + 16 * n] = gf[a][n][r];
        su[n] += __shfl_xor(su[n], 16);
        su[n] += __shfl_xor(su[n], 32);
        if (lg == 0) o[(size_t)NF * H + col + 16 * n] = su[n];
    }
}

// The partial sums' last stage, in a fixed order.  Blocks of 16 waves; a block
// of the first two kinds takes 64 columns, wave v sums parts v, v + 16, ...,
// and the waves' sums are added in order:
//  kL1Cols blocks: g[W1F] (32 rows) and g[B1] (row 32) from lpart;
//  kHeadCols blocks: g[W3], g[B2], g[B3] and the loss from hpart;
//  the rest: du[q] from query q's chunks, four queries per block.
constexpr uint32_t kL1Cols = (NF + 1) * H / 64, kHeadCols = (kHeadPartLen + 63) / 64;

__global__ __launch_bounds__(1024) void sum_parts_kernel(const float *__restrict__ lpart, uint32_t nq, uint32_t chunks,
                                                         const float *__restrict__ hpart, uint32_t n_head,
                                                         uint64_t n_pairs, const uint16_t *__restrict__ w,
                                                         float *__restrict__ g, float *__restrict__ loss,
                                                         float *__restrict__ du) {
    __shared__ float s_w[16][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t b = blockIdx.x;
    if (b >= kL1Cols + kHeadCols) {
        const uint32_t qi = (b - kL1Cols - kHeadCols) * 4 + (threadIdx.x >> 8), j = threadIdx.x & 255;
        if (qi >= nq) return;
        float a = 0.f;
#pragma unroll 4
        for (uint32_t c = 0; c < chunks; c++) a += lpart[((size_t)qi * chunks + c) * kL1PartLen + (size_t)NF * H + j];
        du[(size_t)qi * H + j] = a;
        return;
    }
    const bool head = b >= kL1Cols;
    if (head) b -= kL1Cols;
    const float *src = head ? hpart : lpart;
    const uint32_t len = head ? kHeadPartLen : kL1PartLen, n = head ? n_head : nq * chunks;
    const uint32_t c = b * 64 + lane;
    float a = 0.f;
    if (c < len) {
#pragma unroll 8
        for (uint32_t k = wv; k < n; k += 16) a += src[(size_t)k * len + c];
    }
    s_w[wv][lane] = a;
    __syncthreads();
    if (wv != 0 || c >= len) return;
    for (int v = 1; v < 16; v++) a += s_w[v][lane];
    if (!head)
        g[c < (uint32_t)NF * H ? OFF_W1F + c : OFF_B1 + (c - NF * H)] = a;
    else if (c < (uint32_t)H)
        g[OFF_W3 + c] = a;
    else if (c < 2u * H)
        g[OFF_B2 + (c - H)] = a * bf2f(w[OFF_W3 + (c - H)]);
    else if (c == 2u * H)
        g[OFF_B3] = a;
    else if (loss)
        *loss = a / (float)n_pairs;
}

// g[W1Q + b*H + j] = sum_q bit(q, b) du[q][j], the queries in order.  One block
// per bit; 64 queries' bits are looked at at once and only the set ones
// (2-8%) are added.
__global__ __launch_bounds__(kBlock) void w1q_grad_kernel(const uint64_t *__restrict__ q, uint32_t nq,
                                                          const float *__restrict__ du, float *__restrict__ g) {
    const uint32_t b = blockIdx.x;
    const int j = threadIdx.x, lane = threadIdx.x & 63;
    float a = 0.f;
    for (uint32_t q0 = 0; q0 < nq; q0 += 64) {
        const uint32_t qi = q0 + lane < nq ? q0 + lane : nq - 1;
        u64 m = ballot(q0 + lane < nq && ((q[(uint64_t)qi * QD_WORDS + (b >> 6)] >> (b & 63)) & 1ull));
        while (m) {
            a += du[(size_t)(q0 + __builtin_ctzll(m)) * H + j];
            m &= m - 1;
        }
    }
    g[OFF_W1Q + (size_t)b * H + j] = a;
}

__global__ __launch_bounds__(kBlock) void to_bf16_kernel(const float *__restrict__ p, uint16_t *__restrict__ w,
                                                         size_t n) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        w[i] = f2bf(p[i]);
}

__global__ __launch_bounds__(kBlock) void adam_kernel(float *__restrict__ p, float *__restrict__ m,
                                                      float *__restrict__ v, uint16_t *__restrict__ w,
                                                      const float *__restrict__ g, size_t n, float lr, float b1,
                                                      float b2, float eps, float c1, float c2) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        w[i] = f2bf(pi);
    }
}

// w2t = W2 transposed, in bf16: thread j of block i writes w2t[i][j] = W2[j][i].
__global__ __launch_bounds__(H) void transpose_w2_kernel(const uint16_t *__restrict__ w, uint16_t *__restrict__ w2t) {
    w2t[(size_t)blockIdx.x * H + threadIdx.x] = w[OFF_W2 + (size_t)threadIdx.x * H + blockIdx.x];
}

}  // namespace

// ---- entry points -------------------------------------------------------

static int check_model(qd_model_t m) { return m && m->p ? QD_OK : fail(QD_ERR_INVALID, "null model"); }

}  // namespace qd

extern "C" int qd_model_create(const float *d_params, void *stream, qd_model_t *out) {
    using namespace qd;
    if (!out || !d_params) return fail(QD_ERR_INVALID, "null pointer");
    *out = nullptr;
    hipStream_t s = (hipStream_t)stream;
    qd_model_s *m = new qd_model_s();
    const size_t n = QD_MLP_NPARAMS;
    if (hipMalloc((void **)&m->p, n * 4) != hipSuccess || hipMalloc((void **)&m->m, n * 4) != hipSuccess ||
        hipMalloc((void **)&m->v, n * 4) != hipSuccess || hipMalloc((void **)&m->w, n * 2) != hipSuccess ||
        hipMalloc((void **)&m->w2t, (size_t)H * H * 2) != hipSuccess) {
        qd_model_free(m);
        return fail(QD_ERR_OOM, "model allocation failed");
    }
    (void)hipGetDevice(&m->device);
    QD_HIP_CHECK(hipMemcpyAsync(m->p, d_params, n * 4, hipMemcpyDeviceToDevice, s));
    QD_HIP_CHECK(hipMemsetAsync(m->m, 0, n * 4, s));
    QD_HIP_CHECK(hipMemsetAsync(m->v, 0, n * 4, s));
    hipLaunchKernelGGL(to_bf16_kernel, dim3(1024), dim3(kBlock), 0, s, m->p, m->w, n);
    hipLaunchKernelGGL(transpose_w2_kernel, dim3(H), dim3(H), 0, s, m->w, m->w2t);
    QD_HIP_CHECK(hipGetLastError());
    QD_HIP_CHECK(hipStreamSynchronize(s));
    *out = m;
    return QD_OK;
}

extern "C" int qd_model_free(qd_model_t m) {
    if (!m) return QD_OK;
    void *ptrs[] = {m->p, m->m, m->v, m->w, m->w2t};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    delete m;
    return QD_OK;
}

extern "C" int qd_model_params(qd_model_t m, float *d_params, void *stream) {
    using namespace qd;
    if (check_model(m) != QD_OK || !d_params) return fail(QD_ERR_INVALID, "null pointer");
    QD_HIP_CHECK(hipMemcpyAsync(d_params, m->p, QD_MLP_NPARAMS * 4, hipMemcpyDeviceToDevice, (hipStream_t)stream));
    return QD_OK;
}

static int features_launch(qd_tree_t t, const uint64_t *d_q, qd::PairIdx P, uint64_t n_pairs, float *d_feat,
                           hipStream_t s) {
    using namespace qd;
    if (n_pairs == 0) return QD_OK;
    const uint64_t blocks = (n_pairs + (kBlock / 32) - 1) / (kBlock / 32);
    hipLaunchKernelGGL(features_kernel, dim3((uint32_t)blocks), dim3(kBlock), 0, s,
                       reinterpret_cast<const uint4 *>(d_q), reinterpret_cast<const uint4 *>(t->d_or), t->d_child,
                       t->d_parent, t->d_depth, t->d_count, P, n_pairs, d_feat);
    QD_HIP_CHECK(hipGetLastError());
    return QD_OK;
}

extern "C" int qd_model_features(qd_tree_t t, const uint64_t *d_q, const uint32_t *d_pair_q,
                                 const uint32_t *d_pair_node, uint64_t n_pairs, float *d_feat, void *stream) {
    using namespace qd;
    if (!t) return fail(QD_ERR_INVALID, "null tree");
    if (n_pairs && (!d_q || !d_pair_q || !d_pair_node || !d_feat)) return fail(QD_ERR_INVALID, "null pointer");
    return features_launch(t, d_q, PairIdx{d_pair_q, d_pair_node, 0, 1}, n_pairs, d_feat, (hipStream_t)stream);
}

// Forward (and optionally backward) over pairs grouped by query: queries
// q0 .. q0+nq-1 of d_q, pair p belongs to query P.q(p).  With labels y the
// full gradient goes to d_grads (QD_MLP_NPARAMS) and the mean loss to d_loss;
// this path needs the pairs as explicit arrays grouped by query (d_qoff).
// u_pre (nullable): the per-query layer-1 sums u (nq x H), already formed; an
// inference then allocates nothing.
static int mlp_run(qd_model_t m, const uint64_t *d_q, uint32_t q0, uint32_t nq, qd::PairIdx P,
                   const uint64_t *d_qoff, uint64_t qoff_base, const float *d_feat, uint64_t n_pairs, const float *y,
                   float *d_scores, float *d_grads, float *d_loss, hipStream_t s, const float *u_pre = nullptr) {
    using namespace qd;
    const bool train = y != nullptr;
    const uint64_t tiles = (n_pairs + TP - 1) / TP;
    const uint32_t cus = (uint32_t)device_cus();
    const uint32_t gf = (uint32_t)std::min<uint64_t>(tiles, cus);  // forward: one workgroup per CU
    const uint32_t gw = (uint32_t)std::min<uint64_t>(tiles, cus);  // dW2: likewise, each with its own sum
    const uint32_t chunks = train ? l1_chunks(nq, n_pairs) : 0;
    size_t bytes = 0;
    auto take = [&](size_t b) {
        const size_t at = bytes;
        bytes += (b + 255) / 256 * 256;
        return at;
    };
    const size_t o_u = u_pre ? 0 : take((size_t)nq * H * 4);
    size_t o_h1t = 0, o_m1 = 0, o_m2 = 0, o_ds = 0, o_hpart = 0, o_wpart = 0, o_lpart = 0, o_du = 0;
    if (train) {
        o_h1t = take(tiles * TP * 2 * H * 2);
        o_m1 = take(tiles * kMaskWords * 8);
        o_m2 = take(tiles * kMaskWords * 8);
        o_ds = take(tiles * TP * 4);
        o_hpart = take((size_t)gf * kHeadPartLen * 4);
        o_wpart = take((size_t)gw * H * H * 4);
        o_lpart = take((size_t)nq * chunks * kL1PartLen * 4);
        o_du = take((size_t)nq * H * 4);
    }
    char *ws = nullptr;
    if (bytes) QD_HIP_CHECK(hipMallocAsync((void **)&ws, bytes, s));
    const float *u = u_pre ? u_pre : (float *)(ws + o_u);
    uint4 *h1t = (uint4 *)(ws + o_h1t);
    u64 *m1 = (u64 *)(ws + o_m1), *m2 = (u64 *)(ws + o_m2);
    float *ds = (float *)(ws + o_ds), *hpart = (float *)(ws + o_hpart), *wpart = (float *)(ws + o_wpart),
          *lpart = (float *)(ws + o_lpart), *du = (float *)(ws + o_du);
    {
        KernelTimer timer("mlp_forward", s);
        if (!u_pre) hipLaunchKernelGGL(uq_kernel, dim3(nq), dim3(kBlock), 0, s, d_q, q0, m->w, (float *)(ws + o_u));
        if (train)
            hipLaunchKernelGGL(mlp_forward_kernel<true>, dim3(gf), dim3(kMlpBlock), 0, s, u, P, q0, d_feat, n_pairs,
                               m->w, m->w2t, y, nullptr, h1t, m1, m2, ds, hpart);
        else
            hipLaunchKernelGGL(mlp_forward_kernel<false>, dim3(gf), dim3(kMlpBlock), 0, s, u, P, q0, d_feat, n_pairs,
                               m->w, m->w2t, nullptr, d_scores, nullptr, nullptr, nullptr, nullptr, nullptr);
    }
    hipError_t e = hipGetLastError();
    if (train && e == hipSuccess) {
        KernelTimer timer("mlp_backward", s);
        hipLaunchKernelGGL(dw2_kernel, dim3(gw), dim3(kMlpBlock), 0, s, h1t, m2, ds, m->w, tiles, wpart);
        hipLaunchKernelGGL(dw2_sum_kernel, dim3(H), dim3(kBlock), 0, s, wpart, gw, d_grads);
        hipLaunchKernelGGL(layer1_partial_kernel, dim3(nq * chunks), dim3(kMlpBlock), 0, s, m1, m2, ds, d_feat, m->w,
                           d_qoff, qoff_base, n_pairs, chunks, lpart);
        const uint32_t du_blocks = (nq + 3) / 4;
        hipLaunchKernelGGL(sum_parts_kernel, dim3(kL1Cols + kHeadCols + du_blocks), dim3(1024), 0, s, lpart, nq,
                           chunks, hpart, gf, n_pairs, m->w, d_grads, d_loss, du);
        hipLaunchKernelGGL(w1q_grad_kernel, dim3(QD_BITS), dim3(kBlock), 0, s, d_q + (uint64_t)q0 * QD_WORDS, nq, du,
                           d_grads);
        e = hipGetLastError();
    }
    if (ws) (void)hipFreeAsync(ws, s);
    if (e != hipSuccess) return fail(QD_ERR_DEVICE, "mlp kernels: %s", hipGetErrorString(e));
    return QD_OK;
}

extern "C" int qd_model_forward(qd_model_t m, const uint64_t *d_q, uint32_t nq, const uint32_t *d_pair_q,
                                const float *d_feat, uint64_t n_pairs, float *d_scores, void *stream) {
    using namespace qd;
    if (check_model(m) != QD_OK) return QD_ERR_INVALID;
    if (n_pairs == 0) return QD_OK;
    if (!d_q || !d_pair_q || !d_feat || !d_scores || nq == 0) return fail(QD_ERR_INVALID, "null pointer");
    return mlp_run(m, d_q, 0, nq, PairIdx{d_pair_q, nullptr, 0, 1}, nullptr, 0, d_feat, n_pairs, nullptr, d_scores,
                   nullptr, nullptr, (hipStream_t)stream);
}

extern "C" int qd_model_gradients(qd_model_t m, const uint64_t *d_q, uint32_t nq, const uint64_t *d_qoff,
                                  const uint32_t *d_pair_q, const float *d_feat, const float *d_labels,
                                  uint64_t n_pairs, float *d_grads, float *d_loss, void *stream) {
    using namespace qd;
    if (check_model(m) != QD_OK) return QD_ERR_INVALID;
    if (!d_q || !d_qoff || !d_pair_q || !d_feat || !d_labels || !d_grads || nq == 0 || n_pairs == 0)
        return fail(QD_ERR_INVALID, "null pointer or empty batch");
    return mlp_run(m, d_q, 0, nq, PairIdx{d_pair_q, nullptr, 0, 1}, d_qoff, 0, d_feat, n_pairs, d_labels, nullptr,
                   d_grads, d_loss, (hipStream_t)stream);
}

extern "C" int qd_model_adam_step(qd_model_t m, const float *d_grads, float lr, void *stream) {
    using namespace qd;
    if (check_model(m) != QD_OK || !d_grads) return fail(QD_ERR_INVALID, "null pointer");
    m->step++;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)m->step), c2 = 1.f - powf(b2, (float)m->step);
    hipLaunchKernelGGL(adam_kernel, dim3(1024), dim3(kBlock), 0, (hipStream_t)stream, m->p, m->m, m->v, m->w,
                       d_grads, (size_t)QD_MLP_NPARAMS, lr, b1, b2, 1e-8f, c1, c2);
    hipLaunchKernelGGL(transpose_w2_kernel, dim3(H), dim3(H), 0, (hipStream_t)stream, m->w, m->w2t);
    QD_HIP_CHECK(hipGetLastError());
    return QD_OK;
}

// Scores of nodes 0 .. n_scored-1 for every query: d_scores is nq x n_scored.
extern "C" int qd_model_score_tree(qd_model_t m, qd_tree_t t, const uint64_t *d_q, uint32_t nq, uint32_t n_scored,
                                   float *d_scores, void *stream) {
    using namespace qd;
    if (check_model(m) != QD_OK || !t) return fail(QD_ERR_INVALID, "null model or tree");
    if (nq == 0 || n_scored == 0) return QD_OK;
    if (!d_q || !d_scores) return fail(QD_ERR_INVALID, "null pointer");
    if (n_scored > t->n_nodes) return fail(QD_ERR_INVALID, "n_scored %u above the node count", n_scored);
    hipStream_t s = (hipStream_t)stream;
    // chunks of whole queries, about 1M pairs each
    const uint32_t per = std::max<uint32_t>(1, (uint32_t)((1u << 20) / n_scored));
    float *feat = nullptr;
    const uint64_t maxp = (uint64_t)per * n_scored;
    QD_HIP_CHECK(hipMallocAsync((void **)&feat, maxp * NF * 4, s));
    int rc = QD_OK;
    for (uint32_t q0 = 0; q0 < nq && rc == QD_OK; q0 += per) {
        const uint32_t cq = std::min(per, nq - q0);
        const uint64_t npair = (uint64_t)cq * n_scored;
        PairIdx P{nullptr, nullptr, q0, n_scored};
        {
            KernelTimer timer("mlp_features", s);
            rc = features_launch(t, d_q, P, npair, feat, s);
        }
        if (rc == QD_OK)
            rc = mlp_run(m, d_q, q0, cq, P, nullptr, 0, feat, npair, nullptr, d_scores + (uint64_t)q0 * n_scored,
                         nullptr, nullptr, s);
    }
    (void)hipFreeAsync(feat, s);
    return rc;
}

// ---- learned start of the blocked search --------------------------------

namespace qd {
namespace {

// The pair of children of every query's current node: pairs 2i and 2i + 1
// score the similar and the dissimilar child of cur[i] when that node is an
// inner node above max_rows rows; otherwise both name cur[i] (scored, unused).
__global__ void descend_pairs_kernel(const uint32_t *__restrict__ cur, uint32_t nq, const int32_t *__restrict__ child,
                                     const uint32_t *__restrict__ count, uint32_t max_rows,
                                     uint32_t *__restrict__ pq, uint32_t *__restrict__ pn) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nq) return;
    const uint32_t node = cur[i];
    const int32_t a = child[2 * node];
    const bool go = a >= 0 && count[node] > max_rows;
    pq[2 * i] = pq[2 * i + 1] = i;
    pn[2 * i] = go ? (uint32_t)a : node;
    pn[2 * i + 1] = go ? (uint32_t)child[2 * node + 1] : node;
}

// Enter the higher-scoring child (ties: the similar child).
__global__ void descend_pick_kernel(uint32_t *__restrict__ cur, uint32_t nq, const int32_t *__restrict__ child,
                                    const uint32_t *__restrict__ count, uint32_t max_rows,
                                    const float *__restrict__ sc) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nq) return;
    const uint32_t node = cur[i];
    const int32_t a = child[2 * node];
    if (a < 0 || count[node] <= max_rows) return;
    cur[i] = sc[2 * i + 1] > sc[2 * i] ? (uint32_t)child[2 * node + 1] : (uint32_t)a;
}

__global__ void fill_u32_kernel(uint32_t *__restrict__ p, uint32_t n, uint32_t v) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace

// Scratch of one descent: the per-query layer-1 sums, the level's (query,
// node) pairs, their features and scores.
size_t model_descend_bytes(uint32_t nq) {
    const uint64_t np = 2ull * nq;
    return (size_t)nq * H * 4 + np * 8 + np * NF * 4 + np * 4 + 5 * 256;
}

int model_descend(qd_model_t m, qd_tree_t t, const uint64_t *d_q, uint32_t nq, uint32_t max_rows, uint32_t *d_node,
                  char *ws_given, hipStream_t s) {
    if (check_model(m) != QD_OK || !t) return fail(QD_ERR_INVALID, "null model or tree");
    if (nq == 0) return QD_OK;
    const uint64_t np = 2ull * nq;
    char *ws = ws_given;
    if (!ws) QD_HIP_CHECK(hipMallocAsync((void **)&ws, model_descend_bytes(nq), s));
    char *c = ws;
    auto take = [&](size_t b) {
        char *r = c;
        c += (b + 255) / 256 * 256;
        return r;
    };
    float *u = (float *)take((size_t)nq * H * 4);
    uint32_t *pq = (uint32_t *)take(np * 4), *pn = (uint32_t *)take(np * 4);
    float *feat = (float *)take(np * NF * 4), *sc = (float *)take(np * 4);
    const dim3 g((nq + 255) / 256);
    int rc = QD_OK;
    {
        KernelTimer timer("mlp_forward", s);
        hipLaunchKernelGGL(fill_u32_kernel, g, dim3(256), 0, s, d_node, nq, 0u);  // every query starts at the root
        hipLaunchKernelGGL(uq_kernel, dim3(nq), dim3(kBlock), 0, s, d_q, 0u, m->w, u);  // shared by every level
    }
    for (size_t L = 0; L < t->level_max.size() && t->level_max[L] > max_rows && rc == QD_OK; L++) {
        hipLaunchKernelGGL(descend_pairs_kernel, g, dim3(256), 0, s, d_node, nq, t->d_child, t->d_count, max_rows, pq,
                           pn);
        {
            KernelTimer timer("mlp_features", s);
            rc = features_launch(t, d_q, PairIdx{pq, pn, 0, 1}, np, feat, s);
        }
        if (rc == QD_OK)
            rc = mlp_run(m, d_q, 0, nq, PairIdx{pq, pn, 0, 1}, nullptr, 0, feat, np, nullptr, sc, nullptr, nullptr, s,
                         u);
        hipLaunchKernelGGL(descend_pick_kernel, g, dim3(256), 0, s, d_node, nq, t->d_child, t->d_count, max_rows, sc);
    }
    if (rc == QD_OK && hipGetLastError() != hipSuccess) rc = fail(QD_ERR_DEVICE, "model descent: launch failed");
    if (!ws_given) (void)hipFreeAsync(ws, s);
    return rc;
}

}  // namespace qd

// ---- training pairs from traversal traces ------------------------------

namespace qd {
namespace {

// One block per query.  Pass 1 (pair_q == nullptr) counts valid pairs into
// counts[j]; pass 2 writes them at qoff[j] in ascending node order.
__global__ __launch_bounds__(kBlock) void trace_pairs_kernel(const int32_t *__restrict__ parent,
                                                             const uint32_t *__restrict__ begin,
                                                             const uint32_t *__restrict__ count,
                                                             const uint32_t *__restrict__ iperm, uint64_t n_rows,
                                                             const uint32_t *__restrict__ result, uint32_t k,
                                                             const uint32_t *__restrict__ vis, uint32_t n_traced,
                                                             uint32_t *__restrict__ counts,
                                                             const uint64_t *__restrict__ qoff,
                                                             uint32_t *__restrict__ pair_q,
                                                             uint32_t *__restrict__ pair_node,
                                                             float *__restrict__ labels) {
    __shared__ uint32_t pos[QD_MAX_K];
    __shared__ uint32_t wave_cnt[kBlock / 64];
    const uint32_t j = blockIdx.x;
    const uint32_t words = (n_traced + 31) / 32;
    const uint32_t *v = vis + (uint64_t)j * words;
    if (threadIdx.x < k) {
        const uint32_t r = result[(uint64_t)j * k + threadIdx.x];
        pos[threadIdx.x] = r < n_rows ? iperm[r] : 0xFFFFFFFFu;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t out = pair_q ? qoff[j] : 0;
    uint32_t total = 0;
    for (uint32_t base = 1; base < n_traced; base += kBlock) {
        const uint32_t node = base + threadIdx.x;
        bool valid = false;
        float lab = 0.f;
        if (node < n_traced) {
            const int32_t par = parent[node];
            valid = par >= 0 && ((v[par >> 5] >> (par & 31)) & 1u);
            if (valid)
                for (uint32_t r = 0; r < k; r++) {
                    const uint32_t ps = pos[r];
                    if (ps != 0xFFFFFFFFu && ps >= begin[node] && ps - begin[node] < count[node]) lab = 1.f;
                }
        }
        const uint64_t b = ballot(valid);
        if (lane == 0) wave_cnt[w] = (uint32_t)__popcll(b);
        __syncthreads();
        uint32_t before = 0, chunk = 0;
        for (int i = 0; i < kBlock / 64; i++) {
            if (i < w) before += wave_cnt[i];
            chunk += wave_cnt[i];
        }
        if (valid && pair_q) {
            const uint64_t o = out + before + (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
            pair_q[o] = j;
            pair_node[o] = node;
            labels[o] = lab;
        }
        out += chunk;
        total += chunk;
        __syncthreads();
    }
    if (!pair_q && threadIdx.x == 0) counts[j] = total;
}

}  // namespace
}  // namespace qd

extern "C" int qd_trace_pairs(qd_tree_t t, uint32_t nq, uint32_t k, const uint32_t *d_result_idx,
                              const uint32_t *d_visited, uint32_t n_traced, uint32_t *d_pair_q,
                              uint32_t *d_pair_node, float *d_labels, uint64_t capacity, uint64_t *d_qoff,
                              uint64_t *h_n_pairs, void *stream) {
    using namespace qd;
    if (!t || !h_n_pairs) return fail(QD_ERR_INVALID, "null argument");
    if (k < 1 || k > QD_MAX_K) return fail(QD_ERR_INVALID, "k=%u outside 1..%d", k, QD_MAX_K);
    if (n_traced > t->n_nodes) return fail(QD_ERR_INVALID, "n_traced above the node count");
    *h_n_pairs = 0;
    if (nq == 0) return QD_OK;
    if (!d_result_idx || !d_visited || !d_qoff) return fail(QD_ERR_INVALID, "null pointer");
    hipStream_t s = (hipStream_t)stream;
    uint32_t *cnt = nullptr;
    QD_HIP_CHECK(hipMallocAsync((void **)&cnt, (size_t)nq * 4, s));
    hipLaunchKernelGGL(trace_pairs_kernel, dim3(nq), dim3(kBlock), 0, s, t->d_parent, t->d_begin, t->d_count,
                       t->d_iperm, t->n, d_result_idx, k, d_visited, n_traced, cnt, nullptr, nullptr, nullptr,
                       nullptr);
    std::vector<uint32_t> hc(nq);
    std::vector<uint64_t> off(nq + 1, 0);
    hipError_t e = hipMemcpyAsync(hc.data(), cnt, (size_t)nq * 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFreeAsync(cnt, s);
        return fail(QD_ERR_DEVICE, "trace count: %s", hipGetErrorString(e));
    }
    for (uint32_t j = 0; j < nq; j++) off[j + 1] = off[j] + hc[j];
    *h_n_pairs = off[nq];
    if (off[nq] <= capacity && off[nq] > 0) {
        if (!d_pair_q || !d_pair_node || !d_labels) {
            (void)hipFreeAsync(cnt, s);
            return fail(QD_ERR_INVALID, "null pair arrays");
        }
        e = hipMemcpyAsync(d_qoff, off.data(), (nq + 1) * 8, hipMemcpyHostToDevice, s);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(trace_pairs_kernel, dim3(nq), dim3(kBlock), 0, s, t->d_parent, t->d_begin,
                               t->d_count, t->d_iperm, t->n, d_result_idx, k, d_visited, n_traced, cnt, d_qoff,
                               d_pair_q, d_pair_node, d_labels);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    } else if (off[nq] <= capacity) {
        e = hipMemcpyAsync(d_qoff, off.data(), (nq + 1) * 8, hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
    (void)hipFreeAsync(cnt, s);
    if (e != hipSuccess) return fail(QD_ERR_DEVICE, "trace pairs: %s", hipGetErrorString(e));
    return QD_OK;
}

// ---- training loop ------------------------------------------------------

namespace qd {
int knn_tree_impl(qd_tree_t t, const uint64_t *d_q, uint32_t nq, uint32_t k, int order, const float *d_scores,
                  uint32_t n_scored, uint32_t *d_idx, int32_t *d_missed, int32_t *d_extra, float *d_dist,
                  uint32_t *d_qstats, qd_stats *h_stats, void *stream, uint32_t waves_per_cu, uint32_t *d_trace,
                  uint32_t n_traced, uint32_t split);
}

// Traces the exact best-first search of the training queries, forms the
// (query, node, useful) pairs, and runs `epochs` passes of Adam over batches
// of batch_queries queries, in the order h_batch_order gives (a permutation of
// the batch indices; NULL = ascending).  h_losses (nullable) receives the mean
// loss of every step.  Synchronous.
extern "C" int qd_model_train(qd_model_t m, qd_tree_t t, const uint64_t *d_q, uint32_t nq, uint32_t k,
                              uint32_t n_traced, uint32_t epochs, uint32_t batch_queries, float lr,
                              const uint32_t *h_batch_order, float *h_losses, uint64_t *h_n_pairs, void *stream) {
    using namespace qd;
    if (check_model(m) != QD_OK || !t || !d_q) return fail(QD_ERR_INVALID, "null argument");
    if (nq == 0 || batch_queries == 0 || n_traced < 2 || n_traced > t->n_nodes)
        return fail(QD_ERR_INVALID, "bad training shape");
    hipStream_t s = (hipStream_t)stream;
    const uint32_t words = (n_traced + 31) / 32;
    struct Bufs {
        void *p[12] = {};
        ~Bufs() {
            for (void *x : p)
                if (x) (void)hipFree(x);
        }
    } B;
    uint32_t *idx, *vis;
    int32_t *mi, *ex;
    float *di;
    QD_HIP_CHECK(hipMalloc(&B.p[0], (size_t)nq * k * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[1], (size_t)nq * k * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[2], (size_t)nq * k * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[3], (size_t)nq * k * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[4], (size_t)nq * words * 4));
    idx = (uint32_t *)B.p[0];
    mi = (int32_t *)B.p[1];
    ex = (int32_t *)B.p[2];
    di = (float *)B.p[3];
    vis = (uint32_t *)B.p[4];
    int rc = knn_tree_impl(t, d_q, nq, k, QD_ORDER_BEST_FIRST, nullptr, 0, idx, mi, ex, di, nullptr, nullptr, stream, 0,
                           vis, n_traced, 1);
    if (rc != QD_OK) return rc;
    uint64_t np = 0;
    QD_HIP_CHECK(hipMalloc(&B.p[5], (size_t)(nq + 1) * 8));
    uint64_t *qoff = (uint64_t *)B.p[5];
    rc = qd_trace_pairs(t, nq, k, idx, vis, n_traced, nullptr, nullptr, nullptr, 0, qoff, &np, stream);
    if (rc != QD_OK) return rc;
    if (h_n_pairs) *h_n_pairs = np;
    if (np == 0) return fail(QD_ERR_INVALID, "the traced search produced no training pairs");
    QD_HIP_CHECK(hipMalloc(&B.p[6], np * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[7], np * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[8], np * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[9], np * NF * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[10], (size_t)QD_MLP_NPARAMS * 4));
    QD_HIP_CHECK(hipMalloc(&B.p[11], 4));
    uint32_t *pq = (uint32_t *)B.p[6], *pn = (uint32_t *)B.p[7];
    float *lab = (float *)B.p[8], *feat = (float *)B.p[9], *grads = (float *)B.p[10], *loss = (float *)B.p[11];
    rc = qd_trace_pairs(t, nq, k, idx, vis, n_traced, pq, pn, lab, np, qoff, &np, stream);
    if (rc != QD_OK) return rc;
    rc = features_launch(t, d_q, PairIdx{pq, pn, 0, 1}, np, feat, s);
    if (rc != QD_OK) return rc;
    std::vector<uint64_t> hoff(nq + 1);
    QD_HIP_CHECK(hipMemcpy(hoff.data(), qoff, (nq + 1) * 8, hipMemcpyDeviceToHost));
    const uint32_t nb = (nq + batch_queries - 1) / batch_queries;
    uint64_t step = 0;
    for (uint32_t e = 0; e < epochs; e++)
        for (uint32_t bi = 0; bi < nb; bi++) {
            if (abort_requested()) {  // between steps: the queued ones finish first
                (void)hipStreamSynchronize(s);
                return fail(QD_ERR_ABORTED, "training aborted after %llu steps", (unsigned long long)step);
            }
            const uint32_t b = h_batch_order ? h_batch_order[bi] % nb : bi;
            const uint32_t qa = b * batch_queries, qb = std::min(nq, qa + batch_queries);
            const uint64_t p0 = hoff[qa], p1 = hoff[qb];
            float lv = NAN;
            if (p1 > p0) {
                rc = mlp_run(m, d_q, qa, qb - qa, PairIdx{pq + p0, nullptr, 0, 1}, qoff + qa, p0, feat + p0 * NF,
                             p1 - p0, lab + p0, nullptr, grads, loss, s);
                if (rc != QD_OK) return rc;
                rc = qd_model_adam_step(m, grads, lr, stream);
                if (rc != QD_OK) return rc;
                if (h_losses) {
                    QD_HIP_CHECK(hipMemcpyAsync(&lv, loss, 4, hipMemcpyDeviceToHost, s));
                    QD_HIP_CHECK(hipStreamSynchronize(s));
                }
            }
            if (h_losses) h_losses[step] = lv;
            step++;
        }
    QD_HIP_CHECK(hipStreamSynchronize(s));
    return QD_OK;
}
