// Decode attention of one layer (apex_attention_decode): the block whose run time the
// expert prefetch overlaps.
//
// Launches of a call:
//   split_x  (two or more tokens) h cut into bf16 pieces in the matrix cores' operand order.
//   qkv      W_qkv h.  Query rows go to the workspace (fp32); key and value rows are rounded
//            to bf16 and stored at position pos of the caches.
//   split    attn_split, grid (S, G, B): the tiles of 16 cached positions of one key/value
//            head are shared out over S workgroups of four wavefronts for the H / G query
//            heads that use the head.
//   merge    attn_merge (S > 1), grid (H, B): the S partial results of a head merged
//            (log-sum-exp rule) into the attention vector; up to kFewSplits splits of one
//            token are merged by the output projection itself (gemv_merged).
//   out      W_o a.
// One token's projections are gemv (one wavefront per row), a batch's proj_mfma.
// fp32 activations, scores, probabilities and sums on bf16 weights and caches; no float
// atomics and every sum in a fixed order, so results are deterministic.
//
// The matrix cores take bf16 operands, so fp32 activations go through them as three bf16
// pieces of 8 significant bits each, cut off toward zero: x = hi + mid + lo exactly (but
// for parts below the smallest bf16 value), and three products per tile, summed in fp32,
// replace the fp32 multiply-adds without a rounding of the operands.  A result that is
// not finite (an infinite operand times a zero piece) is computed again with fp32
// multiply-adds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "ffn_device.h"
#include "ffn_internal.h"

namespace {

using apex::ffn::bf_hi;
using apex::ffn::bf_lo;
using apex::ffn::dot8;
using apex::ffn::kWave;
using apex::ffn::ld_stream;
using apex::ffn::row_max;
using apex::ffn::row_ror;
using apex::ffn::row_sum;
using apex::ffn::sum_xor16;
using apex::ffn::sum_xor32;
using apex::ffn::wave_sum;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxGroup = 8;               // query heads per key/value head
constexpr int kTile = 16;                  // cached positions per tile
constexpr int kMaxSplits = 256;            // position splits the workspace has room for

__device__ __forceinline__ uint16_t bf16_bits(float v) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
}

__device__ __forceinline__ bool finite(float v) { return fabsf(v) < INFINITY; }

// The three bf16 pieces of 8 fp32 values.
struct Split3 {
    uint4 p[3];   // hi, mid, lo
};
__device__ __forceinline__ Split3 split3(float4 a, float4 b) {
    float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t w[3][4];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t u0 = __float_as_uint(x[2 * i]), u1 = __float_as_uint(x[2 * i + 1]);
            w[q][i] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);   // upper halves of u0, u1
            x[2 * i] -= __uint_as_float(u0 & 0xffff0000u);
            x[2 * i + 1] -= __uint_as_float(u1 & 0xffff0000u);
        }
    Split3 s;
#pragma unroll
    for (int q = 0; q < 3; ++q) s.p[q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
    return s;
}

__device__ __forceinline__ uint4 keep_if(uint4 v, bool c) {
    return make_uint4(c ? v.x : 0u, c ? v.y : 0u, c ? v.z : 0u, c ? v.w : 0u);
}

__device__ __forceinline__ floatx4 mfma(uint4 a, uint4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Where a projection's results go: o[b, r] (out), or the query rows to q and the key and
// value rows to position pos of the caches (qkv).
struct Dest {
    float *out;                       // q or o
    uint16_t *k_cache, *v_cache;      // qkv only
    int G, hd, ctx_max, pos;
    int qrows;                        // rows of `out`: H * hd (qkv) or d
    __device__ __forceinline__ void put(int b, int r, float v) const {
        if (r < qrows) {
            out[size_t(b) * qrows + r] = v;
            return;
        }
        const int kv = r - qrows, n = G * hd;
        const bool is_v = kv >= n;
        const int gr = is_v ? kv - n : kv;
        const int g = gr / hd, dim = gr - g * hd;
        uint16_t *cache = is_v ? v_cache : k_cache;
        cache[((size_t(b) * G + g) * ctx_max + pos) * hd + dim] = bf16_bits(v);
    }
};

// out[b, r] = W[r] . x[b], one wavefront per row, NPL 16-byte chunks of the row per lane in
// flight together; grid (rows / 4, tokens).
template <int NPL>
__global__ __launch_bounds__(kThreads) void gemv(const float *__restrict__ x,
                                                 const uint16_t *__restrict__ w, int K, int R,
                                                 Dest dst) {
    const int b = blockIdx.y;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int r = blockIdx.x * kWaves + wave;
    if (r >= R) return;
    const int nch = K / 8;
    const uint4 *row = reinterpret_cast<const uint4 *>(w + size_t(r) * K);
    const float4 *x4 = reinterpret_cast<const float4 *>(x + size_t(b) * K);
    float acc = 0.f;
    for (int c0 = 0; c0 < nch; c0 += NPL * kWave) {
        uint4 wv[NPL];
        float4 a[NPL], bb[NPL];
#pragma unroll
        for (int n = 0; n < NPL; ++n) {
            const int c = min(c0 + lane + n * kWave, nch - 1);
            wv[n] = row[c];
            a[n] = x4[2 * c];
            bb[n] = x4[2 * c + 1];
        }
#pragma unroll
        for (int n = 0; n < NPL; ++n)
            if (c0 + lane + n * kWave < nch) acc = dot8(wv[n], a[n], bb[n], acc);
    }
    const float v = wave_sum(acc);
    if (lane == 0) dst.put(b, r, v);
}

// Activations as pieces: step s (32 values of K), tile t (16 tokens), piece q and lane l
// hold the 8 values of token 16 t + l % 16 from K = 32 s + 8 (l / 16), so that a wavefront
// reads an operand of the matrix cores as one piece of 1 KB.
__device__ __forceinline__ size_t piece_at(int s, int tiles, int t, int q, int l) {
    return ((size_t(s) * tiles + t) * 3 + q) * kWave + l;
}

// Grid (steps * tiles / 4): the pieces of x, zeros past token B and past K.
__global__ __launch_bounds__(kThreads) void split_x(const float *__restrict__ x, int B, int K,
                                                    int tiles, int n_pieces,
                                                    uint4 *__restrict__ pieces) {
    const int st = blockIdx.x * kWaves + threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (st >= n_pieces) return;
    const int s = st / tiles, t = st - s * tiles;
    const int b = 16 * t + (lane & 15), k = 32 * s + 8 * (lane >> 4);
    float4 u = make_float4(0.f, 0.f, 0.f, 0.f), v = u;
    if (b < B && k < K) {
        const float4 *p = reinterpret_cast<const float4 *>(x + size_t(b) * K + k);
        u = p[0];
        v = p[1];
    }
    const Split3 c = split3(u, v);
#pragma unroll
    for (int q = 0; q < 3; ++q) pieces[piece_at(s, tiles, t, q, lane)] = c.p[q];
}

// Two or more tokens: out[b, r] = W[r] . x[b] on the matrix cores, tokens as M and rows
// as N.  A workgroup owns 16 * RT rows and up to 16 * NT tokens; its eight wavefronts take
// consecutive shares of K, each with U steps (even) of 32 of its weights in flight and the
// pieces of the next step, and their partial sums are added in LDS in wavefront order.  The
// weights go from memory to the operand registers directly (16 rows of 64 bytes per load:
// 4.1 TB/s alone over 50 MB, whole rows 5.5), the pieces come from L2.  Both pass the
// vector cache of the CU, which is what bounds it: with 32 tokens the pieces are 786 KB per
// workgroup (8.1 us alone at R = K = 4096; the weights alone 8.1, both 14.7).
// The products of the hi pieces are summed over two steps in the matrix cores and from
// there in vector registers: over the whole share in the matrix cores, whose sums are cut
// off more coarsely, the projections were 1.4 times as far from a float64 result as fp32
// multiply-adds at K = 4096 (2.2e-7 against 1.6e-7), so they are 0.6 times (0.9e-7).
constexpr int kProjWaves = 8;
template <int NT, int RT, int U>
__global__ __launch_bounds__(kProjWaves *kWave)
    __attribute__((amdgpu_waves_per_eu(2, 2))) void proj_mfma(
    const uint4 *__restrict__ pieces, int tiles, const float *__restrict__ x,
    const uint16_t *__restrict__ w, int B, int K, int R, Dest dst) {
    __shared__ float red[kProjWaves][RT * NT * 4][kWave];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int r0 = blockIdx.x * 16 * RT, t0 = blockIdx.y * NT;
    const int n_steps = (K + 31) / 32;
    const int s_lo = wave * n_steps / kProjWaves, s_hi = (wave + 1) * n_steps / kProjWaves;
    const int kg = 8 * (lane >> 4);
    const uint16_t *wrow[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
        wrow[i] = w + size_t(min(r0 + 16 * i + (lane & 15), R - 1)) * K;
    const floatx4 none = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 total[RT][NT], low[RT][NT], pair[RT][NT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) total[i][t] = low[i][t] = none;
    uint4 xp[2][NT][3];
    const auto load_x = [&](int s, uint4 (&x)[NT][3]) {   // past the share: its last step again
#pragma unroll
        for (int t = 0; t < NT; ++t)   // tiles past the last one repeat it and are dropped
#pragma unroll
            for (int q = 0; q < 3; ++q)
                x[t][q] = pieces[piece_at(min(s, s_hi - 1), tiles, min(t0 + t, tiles - 1), q, lane)];
    };
    for (int s0 = s_lo; s0 < s_hi; s0 += U) {
        uint4 wv[U][RT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(32 * min(s0 + u, s_hi - 1) + kg, K - 8);
#pragma unroll
            for (int i = 0; i < RT; ++i)
                wv[u][i] = ld_stream(reinterpret_cast<const uint4 *>(wrow[i] + k));
        }
        load_x(s0, xp[0]);
        __builtin_amdgcn_sched_barrier(0);   // all weights on the way before the first use
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u + 1 < U) load_x(s0 + u + 1, xp[(u + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            // a step past the share multiplies zeros: no branch that loads could sink into
#pragma unroll
            for (int i = 0; i < RT; ++i) wv[u][i] = keep_if(wv[u][i], s0 + u < s_hi);
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    low[i][t] = mfma(xp[u & 1][t][2], wv[u][i], low[i][t]);
                    low[i][t] = mfma(xp[u & 1][t][1], wv[u][i], low[i][t]);
                    pair[i][t] = mfma(xp[u & 1][t][0], wv[u][i], u & 1 ? pair[i][t] : none);
                    if (u & 1) total[i][t] += pair[i][t];
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                red[wave][4 * (NT * i + t) + c][lane] = total[i][t][c] + low[i][t][c];
    __syncthreads();
    for (int o = threadIdx.x; o < RT * NT * 4 * kWave; o += kProjWaves * kWave) {
        const int j = o / kWave, l = o % kWave, it = j / 4;
        const int r = r0 + 16 * (it / NT) + (l & 15);
        const int b = 16 * (t0 + it % NT) + 4 * (l >> 4) + j % 4;
        if (r >= R || b >= B) continue;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < kProjWaves; ++q) v += red[q][j][l];
        if (!finite(v)) {
            const uint16_t *wr = w + size_t(r) * K;
            const float *xr = x + size_t(b) * K;
            v = 0.f;
            for (int k = 0; k < K; ++k) v = fmaf(__uint_as_float(uint32_t(wr[k]) << 16), xr[k], v);
        }
        dst.put(b, r, v);
    }
}

__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// The attention vector: fp32 [B, K], and its pieces for proj_mfma (two or more tokens).
struct AttnOut {
    float *a;
    uint16_t *pieces;
    int tiles;
    __device__ __forceinline__ void put(int b, int K, int k, float v) const {
        a[size_t(b) * K + k] = v;
        if (!pieces) return;
        const int lane = (b & 15) + 16 * (k % 32 / 8);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint32_t u = __float_as_uint(v);
            pieces[piece_at(k / 32, tiles, b / 16, q, lane) * 8 + k % 8] = uint16_t(u >> 16);
            v -= __uint_as_float(u & 0xffff0000u);
        }
    }
};

// attn_split: positions 0..n_pos-1 of key/value head g in tiles of 16, shared out over
// gridDim.x * 4 wavefronts.  A wavefront keeps the keys and values of its next tile in
// flight while it works on one:
//   scores  on the matrix cores, query heads as M and positions as N, the queries as three
//           bf16 pieces: head i sits in row 4 (i % 4) + i / 4, so lane (i % 4, n) holds the
//           score of head i at position n in register i / 4 and the exponentials of four
//           heads fill the wavefront;
//   softmax the running maximum of a head is common to the wavefront (a rotation through
//           16 lanes); weighted sums are rescaled only in tiles that raise a maximum;
//   values  fp32 multiply-adds, 8 dimensions per lane, the probabilities passed from the
//           score lanes to the lanes of their position through LDS.
// The wavefronts' states are merged in LDS (log-sum-exp rule).  With one split per head the
// result goes to `out` directly; with more, every workgroup writes its weighted sums,
// maximum and normaliser, and attn_merge or gemv_merged merges the splits.
template <int HD, int GR>
__global__ __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(HD == 128 && GR >= 4 ? 2 : 3))) void attn_split(
    const float *__restrict__ q, const uint16_t *__restrict__ k_cache,
    const uint16_t *__restrict__ v_cache, int H, int G, int ctx_max, int n_pos, int per, int more,
    float scale, float *__restrict__ part, float *__restrict__ part_m, float *__restrict__ part_l,
    AttnOut out) {
    constexpr int KS = HD / 32;              // matrix-core steps of a score
    constexpr int LPP = HD / 8;              // lanes per position of a value load
    constexpr int PPI = kWave / LPP;         // positions per value load
    constexpr int VL = kTile / PPI;          // value loads per tile
    constexpr int RH = (GR + 3) / 4;         // score registers in use
    constexpr int GP = GR == 3 ? 4 : GR;     // heads of one position's probabilities in LDS
    __shared__ __align__(16) float p_lds[kWaves][kTile][GP];
    __shared__ float red_m[kWaves][GR], red_l[kWaves][GR];
    __shared__ float red_acc[kWaves][GR][HD];
    const int s = blockIdx.x, g = blockIdx.y, b = blockIdx.z, S = gridDim.x;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int n = lane & 15, lg = lane >> 4;
    const int vpos = lane / LPP, dim0 = 8 * (lane % LPP);
    const int worker = s * kWaves + wave;   // the first `more` wavefronts take a tile more
    const int t_lo = worker * per + min(worker, more);
    const int t_hi = t_lo + per + (worker < more ? 1 : 0);
    const size_t head_base = (size_t(b) * G + g) * ctx_max;
    const uint16_t *kb = k_cache + head_base * HD, *vb = v_cache + head_base * HD;
    const float *qb = q + (size_t(b) * H + g * GR) * HD;

    uint4 kv[KS], vv[VL];   // the tile in work; the next one's loads follow their last use
    const auto load_k = [&](int t) {
        const int j = min(kTile * t + n, n_pos - 1);
#pragma unroll
        for (int u = 0; u < KS; ++u)
            kv[u] = ld_stream(reinterpret_cast<const uint4 *>(kb + size_t(j) * HD + 32 * u + 8 * lg));
    };
    const auto load_v = [&](int t) {
#pragma unroll
        for (int u = 0; u < VL; ++u) {
            const int jv = min(kTile * t + PPI * u + vpos, n_pos - 1);
            vv[u] = ld_stream(reinterpret_cast<const uint4 *>(vb + size_t(jv) * HD + dim0));
        }
    };
    if (t_lo < t_hi) {
        load_k(t_lo);
        load_v(t_lo);
    }

    // query fragments: row n of the matrix operand is head n / 4 + 4 (n % 4)
    Split3 qf[KS];
    {
        const int i = n / 4 + 4 * (n % 4);
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const float4 *p = reinterpret_cast<const float4 *>(qb + size_t(i < GR ? i : 0) * HD +
                                                               32 * u + 8 * lg);
            float4 x0 = p[0], x1 = p[1];
            const float c = i < GR ? scale : 0.f;
            x0 = make_float4(x0.x * c, x0.y * c, x0.z * c, x0.w * c);
            x1 = make_float4(x1.x * c, x1.y * c, x1.z * c, x1.w * c);
            qf[u] = split3(x0, x1);
        }
    }
    float m[RH], l[RH];      // of heads lg + 4 r; l sums the lane's positions only
    float acc[GR][8];        // of positions vpos, vpos + PPI, ... of the tiles
#pragma unroll
    for (int r = 0; r < RH; ++r) {
        m[r] = -INFINITY;
        l[r] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < GR; ++i)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[i][t] = 0.f;

    for (int t = t_lo; t < t_hi; ++t) {
        floatx4 big = floatx4{0.f, 0.f, 0.f, 0.f}, small = big;
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            small = mfma(qf[u].p[2], kv[u], small);
            big = mfma(qf[u].p[0], kv[u], big);
            small = mfma(qf[u].p[1], kv[u], small);
        }
        if (t + 1 < t_hi) load_k(t + 1);
        const int j = kTile * t + n;
        bool up = false;
        float sc[RH], c[RH];
#pragma unroll
        for (int r = 0; r < RH; ++r) {
            const bool on = j < n_pos && lg + 4 * r < GR;
            sc[r] = on ? big[r] + small[r] : -INFINITY;
            if (on && !finite(sc[r])) {
                float v = 0.f;
                for (int x = 0; x < HD; ++x)
                    v = fmaf(qb[size_t(lg + 4 * r) * HD + x] * scale,
                             __uint_as_float(uint32_t(kb[size_t(j) * HD + x]) << 16), v);
                sc[r] = v;
            }
            const float mn = fmaxf(m[r], row_max(sc[r]));
            up = up || mn > m[r];
            c[r] = mn > m[r] ? expf(m[r] - mn) : 1.f;
            const float p = sc[r] == -INFINITY ? 0.f : expf(sc[r] - mn);
            l[r] = l[r] * c[r] + p;
            m[r] = mn;
            if (lg + 4 * r < GP) p_lds[wave][n][lg + 4 * r] = p;
        }
        if (__ballot(up)) {
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const float ci = lane_value(c[i / 4], 16 * (i % 4));
#pragma unroll
                for (int x = 0; x < 8; ++x) acc[i][x] *= ci;
            }
        }
        if (kTile * (t + 1) > n_pos) {   // values of positions past the last one
#pragma unroll
            for (int u = 0; u < VL; ++u)
                if (kTile * t + PPI * u + vpos >= n_pos) vv[u] = make_uint4(0u, 0u, 0u, 0u);
        }
        // one wavefront's LDS operations complete in order: only the compiler is held here
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int u = 0; u < VL; ++u) {
            const uint32_t w[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
            float p[GP];
#pragma unroll
            for (int i = 0; i < GP; ++i) p[i] = p_lds[wave][PPI * u + vpos][i];
#pragma unroll
            for (int i = 0; i < GR; ++i)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    acc[i][2 * x] = fmaf(p[i], bf_lo(w[x]), acc[i][2 * x]);
                    acc[i][2 * x + 1] = fmaf(p[i], bf_hi(w[x]), acc[i][2 * x + 1]);
                }
        }
        if (t + 1 < t_hi) load_v(t + 1);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // the lanes of one dimension, then the wavefronts
#pragma unroll
    for (int i = 0; i < GR; ++i)
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            if (LPP == 8) acc[i][x] += row_ror<8>(acc[i][x]);
            acc[i][x] = sum_xor32(sum_xor16(acc[i][x]));
        }
    if (lane < LPP)
#pragma unroll
        for (int i = 0; i < GR; ++i)
#pragma unroll
            for (int x = 0; x < 8; ++x) red_acc[wave][i][dim0 + x] = acc[i][x];
#pragma unroll
    for (int r = 0; r < RH; ++r) {
        const float lr = row_sum(l[r]);
        if (n == 0 && lg + 4 * r < GR) {
            red_m[wave][lg + 4 * r] = m[r];
            red_l[wave][lg + 4 * r] = lr;
        }
    }
    __syncthreads();
    const size_t head0 = size_t(b) * H + g * GR;
    for (int idx = threadIdx.x; idx < GR * HD; idx += kThreads) {
        const int i = idx / HD, dim = idx % HD;
        float mm = red_m[0][i];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, red_m[w][i]);
        float ll = 0.f, aa = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float mw = red_m[w][i];
            const float cw = mw == -INFINITY ? (red_l[w][i] == 0.f ? 0.f : NAN) : expf(mw - mm);
            ll = fmaf(red_l[w][i], cw, ll);
            aa = fmaf(red_acc[w][i][dim], cw, aa);
        }
        if (S == 1) {
            out.put(b, H * HD, (g * GR + i) * HD + dim, aa / ll);
        } else {
            const size_t at = (head0 + i) * S + s;
            part[at * HD + dim] = aa;
            if (dim == 0) {
                part_m[at] = mm;
                part_l[at] = ll;
            }
        }
    }
}

// attn_merge: grid (H, B).  The S <= 256 splits of one query head merged by the log-sum-exp
// rule: one split's weight per thread, then every thread sums its share of the splits' values
// (S * hd / 256 of them, loaded eight at a time) and the shares meet in LDS.  A launch of its
// own (about 1 us): merged by the split kernel's last workgroup of each head (a store, a count
// and loads past the caches, one after the other) the call took, in us with the same
// projections, Granite-1B one token at 4095 positions 20.4 instead of 14.2, 8 heads of one
// group at 16383 68.5 instead of 20.8; Granite-3B 32 tokens at 1000 36.2 instead of 37.9.
__global__ __launch_bounds__(kThreads) void attn_merge(const float *__restrict__ part,
                                                       const float *__restrict__ part_m,
                                                       const float *__restrict__ part_l, int S,
                                                       int H, int hd, AttnOut out) {
    __shared__ float w[kMaxSplits];
    __shared__ float red[kWaves], sum[kWaves];
    __shared__ float num[kThreads];
    const int head = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
    const int wave = t / kWave, lane = t % kWave;
    const size_t at = (size_t(b) * H + head) * S;
    const float m = t < S ? part_m[at + t] : -INFINITY, l = t < S ? part_l[at + t] : 0.f;
    const float mw = row_max(m);
    const float mx = fmaxf(fmaxf(lane_value(mw, 0), lane_value(mw, 16)),
                           fmaxf(lane_value(mw, 32), lane_value(mw, 48)));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    const float M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    const float wt = m == -INFINITY ? 0.f : expf(m - M);
    w[t] = wt;
    const float den = wave_sum(wt * l);
    if (lane == 0) sum[wave] = den;
    __syncthreads();
    const float D = sum[0] + sum[1] + sum[2] + sum[3];
    const int dim = t % hd, s0 = t / hd, step = kThreads / hd;
    const float *p = part + at * hd + dim;
    float acc = 0.f;
#pragma unroll 8
    for (int s = s0; s < S; s += step) acc = fmaf(w[s], p[size_t(s) * hd], acc);
    num[t] = acc;
    __syncthreads();
    if (t < hd) {
        float v = 0.f;
        for (int g = 0; g < step; ++g) v += num[g * hd + t];
        out.put(b, H * hd, head * hd + t, v / D);
    }
}

// One token with few splits: o[r] = W_o[r] . a, a merged from the splits by every workgroup
// for itself while its rows of W_o are on the way; one wavefront per row.  Nothing here is
// bound by a rate: a launch is a chain of one memory round trip and some arithmetic.  At
// the Granite-1B shape with 1025 positions (launches back to back, us): merge in a launch
// of its own, 32 splits: split 5.0 + merge 2.5 + out 2.7; merge by the last workgroup
// (a store, a count and loads past the caches, one after the other), 17 splits: split 8.6 +
// out 2.8; merged here, 8 splits: 5.2 + 3.7 (17 splits: 4.3 + 5.8, every workgroup
// reads 70 KB of them); the call 14.2 -> 12.8.
constexpr int kFewSplits = 8;
constexpr size_t kFewBytes = 192 << 10;   // of splits that a CU's workgroups read
template <int NPL>
__global__ __launch_bounds__(kThreads) void gemv_merged(
    const float *__restrict__ part, const float *__restrict__ part_m,
    const float *__restrict__ part_l, int S, int H, int hd, const uint16_t *__restrict__ w,
    int R, float *__restrict__ o) {
    extern __shared__ __align__(16) float lds[];   // a [H * hd], then weights [H][kFewSplits]
    const int K = H * hd, nch = K / 8;
    float *weight = lds + K;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int r = blockIdx.x * kWaves + wave;
    const uint4 *row = reinterpret_cast<const uint4 *>(w + size_t(min(r, R - 1)) * K);
    uint4 wv[NPL];
#pragma unroll
    for (int n = 0; n < NPL; ++n) wv[n] = row[min(lane + n * kWave, nch - 1)];
    // this thread's first 4 values of every split
    const float4 *p4 = reinterpret_cast<const float4 *>(part);
    const auto load = [&](int c, float4 (&v)[kFewSplits]) {
        const int i = 4 * c / hd, rest = c - i * (hd / 4);
#pragma unroll
        for (int s = 0; s < kFewSplits; ++s)
            v[s] = p4[(size_t(i) * S + min(s, S - 1)) * (hd / 4) + rest];
    };
    float4 v[kFewSplits];
    load(min(int(threadIdx.x), K / 4 - 1), v);
    for (int i = threadIdx.x; i < H; i += kThreads) {
        float m[kFewSplits], l[kFewSplits], M = -INFINITY, D = 0.f;
#pragma unroll
        for (int s = 0; s < kFewSplits; ++s) {
            m[s] = part_m[size_t(i) * S + min(s, S - 1)];
            l[s] = part_l[size_t(i) * S + min(s, S - 1)];
        }
#pragma unroll
        for (int s = 0; s < kFewSplits; ++s) M = fmaxf(M, m[s]);
#pragma unroll
        for (int s = 0; s < kFewSplits; ++s) {
            m[s] = s < S && m[s] != -INFINITY ? expf(m[s] - M) : 0.f;
            D = fmaf(m[s], l[s], D);
        }
#pragma unroll
        for (int s = 0; s < kFewSplits; ++s) weight[i * kFewSplits + s] = m[s] / D;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < K / 4; c += kThreads) {
        if (c >= kThreads) load(c, v);
        const float *wt = weight + 4 * c / hd * kFewSplits;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int s = 0; s < kFewSplits; ++s) {
            if (s < S) {
                const float ws = wt[s];
                a.x = fmaf(ws, v[s].x, a.x);
                a.y = fmaf(ws, v[s].y, a.y);
                a.z = fmaf(ws, v[s].z, a.z);
                a.w = fmaf(ws, v[s].w, a.w);
            }
        }
        reinterpret_cast<float4 *>(lds)[c] = a;
    }
    __syncthreads();
    if (r >= R) return;
    const float4 *x4 = reinterpret_cast<const float4 *>(lds);
    float acc = 0.f;
#pragma unroll
    for (int n = 0; n < NPL; ++n) {
        const int c = lane + n * kWave;
        if (c < nch) acc = dot8(wv[n], x4[2 * c], x4[2 * c + 1], acc);
    }
    for (int c = lane + NPL * kWave; c < nch; c += kWave)
        acc = dot8(row[c], x4[2 * c], x4[2 * c + 1], acc);
    const float t = wave_sum(acc);
    if (lane == 0) o[r] = t;
}

// Splits of a head's positions: two workgroups per CU (what the registers of the head-128
// kernel leave room for), at least one tile per wavefront.  32 tokens, 8 key/value heads of
// 128, 2000 positions (262 MB of keys and values), us: 1 split 49, 2 46, 4 46, 8 52, 16 65
// (5.7 TB/s at 2; with ordinary instead of non-temporal loads 52); one position per lane
// group and step, unpipelined, with the scores reduced by shuffles: 1 split, 139.
// One split, without the merge, where the loop of a wavefront is then short against it: a
// tile takes it less the fewer workgroups there are.  Call of 32 tokens, 24 heads of 64 in 8
// groups, 200 positions 29.2 -> 26.3 us, 600 33.1 -> 32.3; 16 tokens at 200 24.3 -> 22.6.
int pick_splits(int n_pos, int B, int G, int most) {
    const int want = (512 + B * G - 1) / (B * G);
    const int tiles = (n_pos + kTile - 1) / kTile;
    if (25 * tiles <= kWaves * B * G) return 1;
    return std::max(1, std::min({want, (tiles + kWaves - 1) / kWaves, most}));
}

void launch_gemv(hipStream_t st, const float *x, const uint16_t *w, int B, int K, int R,
                 const Dest &dst) {
    const dim3 grid((R + kWaves - 1) / kWaves, B);
    const int nch = K / 8;
    const auto f = nch <= kWave       ? gemv<1>
                   : nch <= 2 * kWave ? gemv<2>
                   : nch <= 4 * kWave ? gemv<4>
                                      : gemv<8>;
    hipLaunchKernelGGL(f, grid, dim3(kThreads), 0, st, x, w, K, R, dst);
}

template <int NT>
void launch_proj_tiles(hipStream_t st, const uint4 *pieces, int tiles, const float *x,
                       const uint16_t *w, int B, int K, int R, const Dest &dst) {
    // Every workgroup reads all pieces of its tokens (6 bytes a value), at about 40 bytes a
    // cycle and CU: two row tiles per workgroup where one would mean more than a workgroup
    // per CU, else one.  At 32 tokens, K = 4096: R = 6144 22.1 us with two, 27.2 with one;
    // R = 4096 20.2 and 14.7 (one token at a time, W read again for each: 207 and 267).
    const int gy = (tiles + NT - 1) / NT;
    if ((R + 15) / 16 * gy > 256)
        hipLaunchKernelGGL((proj_mfma<NT, 2, NT == 4 ? 4 : 8>), dim3((R + 31) / 32, gy),
                           dim3(kProjWaves * kWave), 0, st, pieces, tiles, x, w, B, K, R, dst);
    else
        hipLaunchKernelGGL((proj_mfma<NT, 1, 8>), dim3((R + 15) / 16, gy),
                           dim3(kProjWaves * kWave), 0, st, pieces, tiles, x, w, B, K, R, dst);
}

// Whether the projection of two or more tokens (R rows of K values) goes to the matrix cores
// (proj_mfma, `split`: with split_x before it) or one token at a time (gemv, which reads W for
// each token, from the caches after the first at about 9.5 TB/s).  Fitted to ten shapes of 2
// to 64 tokens with each projection on either path; where they cross, (B - 1) R is 15000 to
// 38000 up to K = 1024, 10000 to 20000 at 1536 and 2048 and 9000 to 14000 at 4096.  Up to 32
// row tiles the matrix-core kernel leaves most CUs idle and gemv was ahead at all of them.
// A call of 8 tokens at pos 1000, us, matrix cores -> gemv: Granite-1B 23.6 -> 18.5, 8 heads
// of one group at d = 1024 24.7 -> 18.3, OLMoE 36.5 -> 45.0, Mixtral 48.8 -> 96.5.
bool use_mfma(int B, int K, int R, bool split) {
    if (R <= 512 && B <= 64) return false;
    const long long most = K <= 1024 ? 24000 : K <= 2048 ? 10000 : 8000;
    return (B - 1LL) * R > most + (split ? 3000 : 0);
}

void launch_proj(hipStream_t st, const uint4 *pieces, const float *x, const uint16_t *w, int B,
                 int K, int R, const Dest &dst) {
    const int tiles = (B + 15) / 16;
    if (tiles == 1)
        launch_proj_tiles<1>(st, pieces, tiles, x, w, B, K, R, dst);
    else if (tiles == 2)
        launch_proj_tiles<2>(st, pieces, tiles, x, w, B, K, R, dst);
    else
        launch_proj_tiles<4>(st, pieces, tiles, x, w, B, K, R, dst);
}

template <int HD>
void launch_split(int GR, dim3 grid, hipStream_t st, const float *q, const uint16_t *k_cache,
                  const uint16_t *v_cache, int H, int G, int ctx_max, int n_pos, float scale,
                  float *part, float *part_m, float *part_l, const AttnOut &out) {
    const int tiles = (n_pos + kTile - 1) / kTile, workers = grid.x * kWaves;
    const auto f = GR == 1   ? attn_split<HD, 1>
                   : GR == 2 ? attn_split<HD, 2>
                   : GR == 3 ? attn_split<HD, 3>
                   : GR == 4 ? attn_split<HD, 4>
                             : attn_split<HD, 8>;
    hipLaunchKernelGGL(f, grid, dim3(kThreads), 0, st, q, k_cache, v_cache, H, G, ctx_max, n_pos,
                       tiles / workers, tiles % workers, scale, part, part_m, part_l, out);
}

}  // namespace

extern "C" size_t apex_attention_workspace_bytes(int B, int H, int G, int hd, int ctx_max) {
    if (B <= 0 || H <= 0 || G <= 0 || hd <= 0 || ctx_max <= 0) return 256;
    const size_t qb = apex::align_up(size_t(B) * H * hd * sizeof(float), 256);   // q, a
    const size_t pb = size_t(B) * H * kMaxSplits * (hd + 2) * sizeof(float);
    return 2 * qb + apex::align_up(pb, 256);
}

extern "C" apex_status apex_attention_decode(const float *h, const uint16_t *w_qkv,
                                             const uint16_t *w_o, int B, int d, int H, int G,
                                             int hd, uint16_t *k_cache, uint16_t *v_cache,
                                             int ctx_max, int pos, float *o, void *workspace,
                                             size_t workspace_bytes, hipStream_t stream) {
    const char *fn = "apex_attention_decode";
    APEX_REQUIRE(B >= 0, "%s: B=%d must be >= 0", fn, B);
    APEX_REQUIRE(d >= 8 && d % 8 == 0, "%s: d=%d must be a positive multiple of 8", fn, d);
    APEX_REQUIRE(hd == 64 || hd == 128, "%s: head size %d must be 64 or 128", fn, hd);
    APEX_REQUIRE(H >= 1 && G >= 1 && H % G == 0 && H / G <= kMaxGroup,
                 "%s: H=%d must be a multiple of G=%d with at most %d query heads per group",
                 fn, H, G, kMaxGroup);
    APEX_REQUIRE(H / G <= 4 || H / G == 8, "%s: %d query heads per group is not supported",
                 fn, H / G);
    APEX_REQUIRE(ctx_max >= 1 && pos >= 0 && pos < ctx_max, "%s: pos=%d out of [0, %d)", fn,
                 pos, ctx_max);
    if (B == 0) return APEX_OK;
    APEX_REQUIRE(h && w_qkv && w_o && k_cache && v_cache && o && workspace, "%s: NULL pointer",
                 fn);
    APEX_REQUIRE(apex::aligned16(h) && apex::aligned16(w_qkv) && apex::aligned16(w_o) &&
                     apex::aligned16(k_cache) && apex::aligned16(v_cache) &&
                     apex::aligned16(workspace),
                 "%s: inputs, caches and workspace must be 16-byte aligned", fn);
    const size_t need = apex_attention_workspace_bytes(B, H, G, hd, ctx_max);
    if (workspace_bytes < need)
        return apex::fail(APEX_E_CAPACITY, "%s: workspace %zu < %zu bytes", fn, workspace_bytes,
                          need);
    const int n_pos = pos + 1;
    // one token over few positions: up to kFewSplits splits per head, merged by the output
    // projection, as long as its workgroups on one CU (four rows each) read no more than
    // kFewBytes of them
    const int pos_tiles = (n_pos + kTile - 1) / kTile;
    const size_t split_bytes = size_t(H) * hd * sizeof(float) * ((d + 1023) / 1024);
    const int few_splits = std::min({(pos_tiles + kWaves - 1) / kWaves, kFewSplits,
                                     int(std::min(kFewBytes / split_bytes, size_t(kFewSplits)))});
    const bool few = B == 1 && few_splits > 0 && pos_tiles <= few_splits * kWaves * 4;
    // workspace: q, a, then the room of kMaxSplits splits (hd weighted sums, a maximum and a
    // normaliser per head and token).  A batch's pieces, 6 bytes a value and tokens up to whole
    // tiles, take their place there: those of `h` before any split is written, those of `a`
    // behind the splits
    const size_t qb = apex::align_up(size_t(B) * H * hd * sizeof(float), 256);
    const size_t heads = size_t(B) * H, split_room = heads * (hd + 2) * sizeof(float);
    const size_t room = kMaxSplits * split_room;
    const int tiles = (B + 15) / 16;
    const auto piece_bytes = [&](int K) {
        return size_t((K + 31) / 32) * tiles * 3 * kWave * sizeof(uint4);
    };
    const size_t a_bytes = piece_bytes(H * hd);
    float *q = static_cast<float *>(workspace);
    float *a = reinterpret_cast<float *>(static_cast<char *>(workspace) + qb);
    float *part = reinterpret_cast<float *>(static_cast<char *>(workspace) + 2 * qb);
    const bool mfma_out = B > 1 && use_mfma(B, H * hd, d, false);
    const bool mfma_qkv = B > 1 && piece_bytes(d) <= room && use_mfma(B, d, (H + 2 * G) * hd, true);
    uint4 *x_pieces = reinterpret_cast<uint4 *>(part);
    uint4 *a_pieces = reinterpret_cast<uint4 *>(reinterpret_cast<char *>(part) + (room - a_bytes) / 256 * 256);
    const int most = mfma_out ? int((room - a_bytes - 256) / split_room) : kMaxSplits;
    const int S = few ? few_splits : pick_splits(n_pos, B, G, most);
    float *part_m = part + heads * S * hd, *part_l = part_m + heads * S;

    const int R = (H + 2 * G) * hd;
    const Dest qkv{q, k_cache, v_cache, G, hd, ctx_max, pos, H * hd};
    if (mfma_qkv) {
        const int n = (d + 31) / 32 * tiles;
        hipLaunchKernelGGL(split_x, dim3((n + kWaves - 1) / kWaves), dim3(kThreads), 0, stream, h,
                           B, d, tiles, n, x_pieces);
        APEX_HIP(hipGetLastError());
        launch_proj(stream, x_pieces, h, w_qkv, B, d, R, qkv);
    } else {
        launch_gemv(stream, h, w_qkv, B, d, R, qkv);
    }
    APEX_HIP(hipGetLastError());
    const AttnOut out{a, mfma_out ? reinterpret_cast<uint16_t *>(a_pieces) : nullptr, tiles};
    const float scale = 1.f / std::sqrt(float(hd));
    const dim3 grid(S, G, B);
    if (hd == 64)
        launch_split<64>(H / G, grid, stream, q, k_cache, v_cache, H, G, ctx_max, n_pos, scale,
                         part, part_m, part_l, out);
    else
        launch_split<128>(H / G, grid, stream, q, k_cache, v_cache, H, G, ctx_max, n_pos, scale,
                          part, part_m, part_l, out);
    APEX_HIP(hipGetLastError());
    if (S > 1 && !few) {
        hipLaunchKernelGGL(attn_merge, dim3(H, B), dim3(kThreads), 0, stream, part, part_m, part_l,
                           S, H, hd, out);
        APEX_HIP(hipGetLastError());
    }
    const Dest dst{o, nullptr, nullptr, 1, 1, 1, 0, d};
    if (few && S > 1) {
        const int nch = H * hd / 8;
        const size_t lds = (size_t(H) * hd + size_t(H) * kFewSplits) * sizeof(float);
        const auto f = nch <= kWave ? gemv_merged<1> : nch <= 2 * kWave ? gemv_merged<2>
                                  : nch <= 4 * kWave ? gemv_merged<4> : gemv_merged<8>;
        hipLaunchKernelGGL(f, dim3((d + kWaves - 1) / kWaves), dim3(kThreads), lds, stream, part,
                           part_m, part_l, S, H, hd, w_o, d, o);
    } else if (mfma_out) {
        launch_proj(stream, a_pieces, a, w_o, B, H * hd, d, dst);
    } else {
        launch_gemv(stream, a, w_o, B, H * hd, d, dst);
    }
    APEX_HIP(hipGetLastError());
    return APEX_OK;
}
