// Prefetch router (apex_prefetch_route) and original-router top-k (apex_gate_topk).
//
// One workgroup of 16 wavefronts per token.  A wavefront owns 128 values of the hidden
// state (8 per lane of a row of 16 lanes) and streams that piece of four rows of the bf16
// router matrix per 16-byte load, so the workgroup reads the hidden state once and every
// load of a pass (2048 values at most) is requested before the first multiply.  The partial
// dot products are summed over the row's lanes in the vector unit and over the wavefronts in
// LDS.  Softmax, ranking and the selection rules then run in wavefront 0 with one lane per
// expert (E <= 64), exchanging values through registers (DPP, row exchanges, ballots).
// Optionally each token's workgroup then writes `seq` into done[token], after its
// outputs and a system-scope fence, so that a host polling pinned memory learns that the
// outputs are there before the kernel's completion signal reaches it.
#include <hip/hip_runtime.h>

#include <cmath>

#include "common.h"
#include "ffn_device.h"
#include "route_internal.h"

namespace {

constexpr int kWave = 64;
constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxD = 65536;

using apex::ffn::dot8;
using apex::ffn::row_max;
using apex::ffn::row_sum;
using apex::ffn::wave_sum;

__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ float wave_max(float v) {
    v = row_max(v);
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)),
                 fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

// Inclusive prefix sum over the wavefront.
template <int N>
__device__ __forceinline__ float row_shr(float v) {   // the value N lanes back in the row, or 0
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x110 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_prefix(float v, int lane) {
    v += row_shr<1>(v);
    v += row_shr<2>(v);
    v += row_shr<4>(v);
    v += row_shr<8>(v);
    const float a = lane_value(v, 15), b = a + lane_value(v, 31), c = b + lane_value(v, 47);
    return v + (lane < 16 ? 0.f : lane < 32 ? a : lane < 48 ? b : c);
}

// z[e] = W[e, :] . h (+ bias[e]) for all experts, into LDS.  All threads call it.
// A unit of work is 16 chunks of 8 values times 4 experts: one 16-byte load per lane.
// WC (1, 2, 4, 8 or 16) wavefronts share out the groups of 16 chunks, the 16 / WC wavefronts
// with the same chunks the groups of 4 experts, NG of them each per round (at most 8, whose
// loads are in flight together: 128 KB for the workgroup; 16 groups in one round took more
// than the 128 registers a lane has here).  part[WC][64] in LDS.
// One CU reads the whole matrix (256 KB at E = 64, d = 2048), so what bounds the kernel is
// the memory round trip, its vector cache, and the chain behind it.  Against whole rows per
// wavefront, the hidden state read by each, and reductions through the LDS crossbar, us a
// kernel: OLMoE 64 tokens 11.2 -> 9.6, Granite-3B 8.5 -> 6.5, Phi-7B 6.4 -> 4.8, Granite-1B
// 5.3 -> 4.5, Mixtral 32 tokens 4.9 -> 3.9, d = 256 with 8 experts 3.0 -> 2.3.
template <int WC, int NG>
__device__ void token_logits(const float *__restrict__ h, const uint16_t *__restrict__ W,
                             const float *__restrict__ bias, int d, int E, float (*part)[64],
                             float *z_lds) {
    const float4 *h4 = reinterpret_cast<const float4 *>(h);
    // a buffer: base and length in scalar registers, so that a load takes one offset register
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(W), 0, E * d * 2,
                                                        0x00027000);
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int wc = wave % WC, we = wave / WC;
    constexpr int WE = kWaves / WC;
    const int nch = d / 8, sub = lane & 15, er = lane >> 4;
#pragma unroll 1
    for (int e0 = 4 * we; e0 < E; e0 += 4 * WE * NG) {   // one round, or two
        float acc[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g] = 0.f;
#pragma unroll 1
        for (int c0 = 16 * wc; c0 < nch; c0 += 16 * WC) {
            const bool on = c0 + sub < nch;
            const int c = on ? c0 + sub : nch - 1;
            uint4 w[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g)   // experts past E repeat the last one and are dropped
                w[g] = __builtin_bit_cast(
                    uint4, __builtin_amdgcn_raw_buffer_load_b128(
                               rsrc, (min(e0 + 4 * WE * g + er, E - 1) * nch + c) * 16, 0, 0));
            float4 a = h4[2 * c], b = h4[2 * c + 1];
            if (!on) a = b = make_float4(0.f, 0.f, 0.f, 0.f);
            __builtin_amdgcn_sched_barrier(0);   // all loads on the way before the first use
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (on) acc[g] = dot8(w[g], a, b, acc[g]);
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float s = row_sum(acc[g]);
            const int e = e0 + 4 * WE * g + er;
            if (sub == 0 && e < E) part[wc][e] = s;
        }
    }
    __syncthreads();
    if (wave != 0) return;
    float z[WC];   // added pairwise: one after the other they rounded up to 15 times
#pragma unroll
    for (int q = 0; q < WC; ++q) z[q] = part[q][lane];
#pragma unroll
    for (int n = WC / 2; n > 0; n /= 2)
#pragma unroll
        for (int q = 0; q < n; ++q) z[q] += z[q + n];
    if (lane < E) z_lds[lane] = z[0] + (bias ? bias[lane] : 0.f);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Position of expert `lane` when experts are ordered by descending logit, lower id
// first on equal logits, counting only experts whose bit is set in `mask` (no bit at or
// beyond E).  The logits are read from LDS four at a time, every lane at the same address
// (a broadcast): against other lanes' logits read with readlane (register to scalar, one
// at a time) the router took 6.20 -> 5.51 us at the Granite-1B shape and 11.34 -> 10.63
// at OLMoE's, with the same ranks.  z_lds is 16-byte aligned and holds 64 entries.
__device__ __forceinline__ int masked_rank(const float *z_lds, float z, int E, int lane,
                                           unsigned long long mask) {
    int r = 0;
    const float4 *z4 = reinterpret_cast<const float4 *>(z_lds);
    for (int j4 = 0; j4 < (E + 3) / 4; ++j4) {
        const float4 q = z4[j4];
        const int j = 4 * j4;
        const unsigned long long mb = mask >> j;
        r += ((mb & 1ull) && (q.x > z || (q.x == z && j < lane))) ? 1 : 0;
        r += ((mb & 2ull) && (q.y > z || (q.y == z && j + 1 < lane))) ? 1 : 0;
        r += ((mb & 4ull) && (q.z > z || (q.z == z && j + 2 < lane))) ? 1 : 0;
        r += ((mb & 8ull) && (q.w > z || (q.w == z && j + 3 < lane))) ? 1 : 0;
    }
    return r;
}

// Marks token b's outputs as written: every store of this wavefront first reaches the
// system (host memory included), then done[b] = seq, written by lane 0 (a vector store).
__device__ __forceinline__ void signal_done(int32_t *done, int32_t seq, int b, int lane) {
    if (!done) return;
    __threadfence_system();
    if (lane == 0) __hip_atomic_store(done + b, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ float logit_of(float tau) {
    if (tau <= 0.f) return -INFINITY;
    if (tau >= 1.f) return INFINITY;
    return logf(tau / (1.f - tau));
}

template <int WC, int NG>
__global__ __launch_bounds__(kThreads) void prefetch_route_kernel(
    const float *__restrict__ h_pre, const uint16_t *__restrict__ w_pf,
    const float *__restrict__ b_pf, int d, int E, int k, int k_max, int policy, float tau,
    int static_delta, const float *__restrict__ cdf_w, const float *__restrict__ cdf_theta,
    int32_t *__restrict__ pf_idx, int32_t *__restrict__ pf_count, float *__restrict__ pf_prob,
    int32_t *__restrict__ done, int32_t seq) {
    __shared__ __align__(16) float z_lds[APEX_MAX_EXPERTS];
    __shared__ float part[WC][64];
    __shared__ float sorted_q[APEX_MAX_EXPERTS];
    __shared__ int sorted_id[APEX_MAX_EXPERTS];

    const int b = blockIdx.x;
    token_logits<WC, NG>(h_pre + size_t(b) * d, w_pf, b_pf, d, E, part, z_lds);

    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (wave != 0) return;   // selection is one wavefront's work; no barriers follow

    const bool live = lane < E;
    const float z = live ? z_lds[lane] : -INFINITY;
    const float mx = wave_max(z);
    const float p = live ? expf(z - mx) : 0.f;
    const float q = p / wave_sum(p);
    const unsigned long long all = (E == 64) ? ~0ull : ((1ull << E) - 1ull);
    const int r = masked_rank(z_lds, z, E, lane, all);
    if (live) {
        sorted_q[r] = q;
        sorted_id[r] = lane;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const float qs = live ? sorted_q[lane] : 0.f;

    int m;
    if (policy == APEX_SEL_CUMPROB) {
        const float S = wave_prefix(qs, lane);   // in ranked order
        const unsigned long long hit = __ballot(live && S >= tau);
        const int m_star = hit ? __ffsll(static_cast<long long>(hit)) : E;
        m = min(max(m_star, k), k_max);
    } else if (policy == APEX_SEL_ORDINAL_CDF) {
        const float s = wave_sum(live ? cdf_w[lane] * qs : 0.f);
        const float thr = logit_of(tau);
        const bool ok = (lane <= E - k) && (cdf_theta[lane <= E - k ? lane : 0] - s >= thr);
        const unsigned long long hit = __ballot(ok);
        const int delta_hat = hit ? __ffsll(static_cast<long long>(hit)) - 1 : E - k;
        m = min(k + delta_hat, k_max);
    } else if (policy == APEX_SEL_STATIC) {
        m = min(k + static_delta, k_max);
    } else {
        m = 0;   // APEX_SEL_NONE
    }
    if (lane < k_max) pf_idx[size_t(b) * k_max + lane] = lane < m ? sorted_id[lane] : -1;
    if (lane == 0) pf_count[b] = m;
    if (pf_prob && live) pf_prob[size_t(b) * E + lane] = q;
    signal_done(done, seq, b, lane);
}

template <int WC, int NG>
__global__ __launch_bounds__(kThreads) void gate_topk_kernel(
    const float *__restrict__ h_post, const uint16_t *__restrict__ w_g,
    const float *__restrict__ b_g, int d, int E, int k, int mode,
    const uint8_t *__restrict__ avail, int avail_stride, int32_t *__restrict__ route_idx,
    float *__restrict__ route_gate, int32_t *__restrict__ exec_idx,
    float *__restrict__ exec_gate, float *__restrict__ gate_prob, int32_t *__restrict__ done,
    int32_t seq) {
    __shared__ __align__(16) float z_lds[APEX_MAX_EXPERTS];
    __shared__ float part[WC][64];

    const int b = blockIdx.x;
    token_logits<WC, NG>(h_post + size_t(b) * d, w_g, b_g, d, E, part, z_lds);

    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (wave != 0) return;

    const bool live = lane < E;
    const float z = live ? z_lds[lane] : -INFINITY;
    const float mx = wave_max(z);
    const float p = live ? expf(z - mx) : 0.f;
    const float psum = wave_sum(p);
    const unsigned long long all = (E == 64) ? ~0ull : ((1ull << E) - 1ull);

    const int r = masked_rank(z_lds, z, E, lane, all);
    const bool sel_r = live && r < k;
    const float rsum = wave_sum(sel_r ? p : 0.f);
    const size_t row = size_t(b) * k;
    if (sel_r) {
        route_idx[row + r] = lane;
        route_gate[row + r] = p / rsum;
    }
    if (mode == APEX_MODE_EXACT) {
        if (sel_r) {
            exec_idx[row + r] = lane;
            exec_gate[row + r] = p / rsum;
        }
    } else {
        const bool a = live && avail[size_t(b) * avail_stride + lane] != 0;
        const unsigned long long amask = __ballot(a);
        const int ra = masked_rank(z_lds, z, E, lane, amask);
        const bool sel = a && ra < k;
        const int n_sel = __popcll(__ballot(sel));
        const float xsum = wave_sum(sel ? p : 0.f);
        if (sel) {
            exec_idx[row + ra] = lane;
            exec_gate[row + ra] = p / xsum;
        }
        if (lane >= n_sel && lane < k) {
            exec_idx[row + lane] = -1;
            exec_gate[row + lane] = 0.f;
        }
    }
    if (gate_prob && live) gate_prob[size_t(b) * E + lane] = p / psum;
    signal_done(done, seq, b, lane);
}

// Shape of token_logits: as many wavefronts as there are groups of 16 chunks (up to 16) side
// by side along d, the others along the experts.
struct LogitShape {
    int wc, ng;   // ng: groups of 4 experts per wavefront and round, rounded up to 1, 2, 4, 6, 8
};
LogitShape logit_shape(int d, int E) {
    const int groups = (d / 8 + 15) / 16;
    int wc = 1;
    while (wc < groups && wc < kWaves) wc *= 2;
    const int we = kWaves / wc, all = (E + 4 * we - 1) / (4 * we);
    const int ng = all > 8 ? (all + 1) / 2 : all;
    return {wc, ng <= 2 ? ng : ng <= 4 ? 4 : ng <= 6 ? 6 : 8};
}

// The kernel of a shape; F<WC, NG>::run() launches it.
template <template <int, int> class F, class... A>
void launch_shape(LogitShape s, A... a) {
#define APEX_SHAPE(WC_)                                                                    \
    switch (s.ng) {                                                                        \
        case 1: F<WC_, 1>::run(a...); break;                                               \
        case 2: F<WC_, 2>::run(a...); break;                                               \
        case 4: F<WC_, 4>::run(a...); break;                                               \
        case 6: F<WC_, 6>::run(a...); break;                                               \
        default: F<WC_, 8>::run(a...); break;                                              \
    }
    // E <= 64: one group of experts per wavefront with one along d, two with two, four with four
    if (s.wc == 1) {
        F<1, 1>::run(a...);
    } else if (s.wc == 2) {
        s.ng == 1 ? F<2, 1>::run(a...) : F<2, 2>::run(a...);
    } else if (s.wc == 4) {
        s.ng == 1 ? F<4, 1>::run(a...) : s.ng == 2 ? F<4, 2>::run(a...) : F<4, 4>::run(a...);
    } else if (s.wc == 8) {
        APEX_SHAPE(8)
    } else {
        APEX_SHAPE(16)
    }
#undef APEX_SHAPE
}
template <int WC, int NG>
struct Route {
    template <class... A>
    static void run(int B, hipStream_t st, A... a) {
        hipLaunchKernelGGL((prefetch_route_kernel<WC, NG>), dim3(B), dim3(kThreads), 0, st, a...);
    }
};
template <int WC, int NG>
struct Gate {
    template <class... A>
    static void run(int B, hipStream_t st, A... a) {
        hipLaunchKernelGGL((gate_topk_kernel<WC, NG>), dim3(B), dim3(kThreads), 0, st, a...);
    }
};

apex_status check_router_args(const char *fn, const float *h, const uint16_t *w, int B, int d,
                              int E, int k) {
    APEX_REQUIRE(B >= 0, "%s: B=%d must be >= 0", fn, B);
    APEX_REQUIRE(E >= 1, "%s: E=%d must be >= 1", fn, E);
    if (E > APEX_MAX_EXPERTS)
        return apex::fail(APEX_E_UNSUPPORTED, "%s: E=%d exceeds %d", fn, E, APEX_MAX_EXPERTS);
    APEX_REQUIRE(k >= 1 && k <= E, "%s: k=%d out of [1, E=%d]", fn, k, E);
    APEX_REQUIRE(d >= 8 && d % 8 == 0, "%s: d=%d must be a positive multiple of 8", fn, d);
    if (d > kMaxD) return apex::fail(APEX_E_UNSUPPORTED, "%s: d=%d exceeds %d", fn, d, kMaxD);
    if (B == 0) return APEX_OK;
    APEX_REQUIRE(h && w, "%s: NULL input pointer", fn);
    APEX_REQUIRE(apex::aligned16(h) && apex::aligned16(w), "%s: inputs must be 16-byte aligned",
                 fn);
    return APEX_OK;
}

}  // namespace

namespace apex {

apex_status prefetch_route(const float *h_pre, const uint16_t *w_pf, const float *b_pf, int B,
                           int d, int E, int k, int k_max, int policy, float tau,
                           int static_delta, const float *cdf_w, const float *cdf_theta,
                           int32_t *pf_idx, int32_t *pf_count, float *pf_prob, int32_t *done,
                           int32_t seq, hipStream_t stream) {
    const char *fn = "apex_prefetch_route";
    apex_status st = check_router_args(fn, h_pre, w_pf, B, d, E, k);
    if (st != APEX_OK) return st;
    APEX_REQUIRE(k_max >= k && k_max <= E, "%s: k_max=%d out of [k=%d, E=%d]", fn, k_max, k, E);
    APEX_REQUIRE(policy == APEX_SEL_CUMPROB || policy == APEX_SEL_ORDINAL_CDF ||
                     policy == APEX_SEL_STATIC || policy == APEX_SEL_NONE,
                 "%s: unknown policy %d", fn, policy);
    APEX_REQUIRE(policy == APEX_SEL_STATIC || policy == APEX_SEL_NONE ||
                     (tau >= 0.f && tau <= 1.f),
                 "%s: tau=%g out of [0, 1]", fn, double(tau));
    APEX_REQUIRE(policy != APEX_SEL_STATIC || static_delta >= 0, "%s: static_delta=%d < 0", fn,
                 static_delta);
    APEX_REQUIRE(policy != APEX_SEL_ORDINAL_CDF || (cdf_w && cdf_theta),
                 "%s: ORDINAL_CDF needs cdf_w and cdf_theta", fn);
    if (B == 0) return APEX_OK;
    APEX_REQUIRE(pf_idx && pf_count, "%s: NULL output pointer", fn);
    launch_shape<Route>(logit_shape(d, E), B, stream, h_pre, w_pf, b_pf, d, E, k, k_max, policy, tau,
                        static_delta, cdf_w, cdf_theta, pf_idx, pf_count, pf_prob, done, seq);
    APEX_HIP(hipGetLastError());
    return APEX_OK;
}

apex_status gate_topk(const float *h_post, const uint16_t *w_g, const float *b_g, int B, int d,
                      int E, int k, int mode, const uint8_t *avail, int avail_stride,
                      int32_t *route_idx, float *route_gate, int32_t *exec_idx, float *exec_gate,
                      float *gate_prob, int32_t *done, int32_t seq, hipStream_t stream) {
    const char *fn = "apex_gate_topk";
    apex_status st = check_router_args(fn, h_post, w_g, B, d, E, k);
    if (st != APEX_OK) return st;
    APEX_REQUIRE(mode == APEX_MODE_EXACT || mode == APEX_MODE_STALL_FREE, "%s: unknown mode %d",
                 fn, mode);
    if (mode == APEX_MODE_STALL_FREE) {
        APEX_REQUIRE(avail_stride == 0 || avail_stride >= E,
                     "%s: avail_stride=%d must be 0 or >= E", fn, avail_stride);
        APEX_REQUIRE(B == 0 || avail, "%s: STALL_FREE needs avail", fn);
    }
    if (B == 0) return APEX_OK;
    APEX_REQUIRE(route_idx && route_gate && exec_idx && exec_gate, "%s: NULL output pointer", fn);
    launch_shape<Gate>(logit_shape(d, E), B, stream, h_post, w_g, b_g, d, E, k, mode, avail,
                       avail_stride, route_idx, route_gate, exec_idx, exec_gate, gate_prob, done, seq);
    APEX_HIP(hipGetLastError());
    return APEX_OK;
}

}  // namespace apex

extern "C" apex_status apex_prefetch_route(const float *h_pre, const uint16_t *w_pf,
                                           const float *b_pf, int B, int d, int E, int k,
                                           int k_max, int policy, float tau, int static_delta,
                                           const float *cdf_w, const float *cdf_theta,
                                           int32_t *pf_idx, int32_t *pf_count, float *pf_prob,
                                           hipStream_t stream) {
    return apex::prefetch_route(h_pre, w_pf, b_pf, B, d, E, k, k_max, policy, tau, static_delta,
                                cdf_w, cdf_theta, pf_idx, pf_count, pf_prob, nullptr, 0, stream);
}

extern "C" apex_status apex_gate_topk(const float *h_post, const uint16_t *w_g, const float *b_g,
                                      int B, int d, int E, int k, int mode,
                                      const uint8_t *avail, int avail_stride, int32_t *route_idx,
                                      float *route_gate, int32_t *exec_idx, float *exec_gate,
                                      float *gate_prob, hipStream_t stream) {
    return apex::gate_topk(h_post, w_g, b_g, B, d, E, k, mode, avail, avail_stride, route_idx,
                           route_gate, exec_idx, exec_gate, gate_prob, nullptr, 0, stream);
}
